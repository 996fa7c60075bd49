"""The flexible-tile GEMM against the 256x256 one: a sequence alone (few rows, small tiles)
must give bitwise what it gives packed behind a long one (many rows, 256x256 tiles), since
every tile forms each output with the same MFMA chain.  Row counts sit on the edges of the
32-, 64-, 128-, 160- and 256-row tiles; the shapes make the dispatch pick every tile (wide,
shallow gate/up and lm_head; a deep down projection; 3584-column o-proj).  The long packed
run itself is compared with the oracle by the other parity tests' models."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2608_14498_amd import binding as rb
from paper_2608_14498_amd import configs, inputs
from paper_2608_14498_amd.runtime import DeviceModel, to_device

pytestmark = pytest.mark.gpu

WIDE = configs.ModelShape(n_layers=2, d_model=128, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn_dim=20480,
                          vocab=152064, dtype="bf16")
BROAD = configs.ModelShape(n_layers=1, d_model=3584, n_q_heads=8, n_kv_heads=2, head_dim=128, ffn_dim=192,
                           vocab=1003, dtype="bf16")
# q/k/v of 4608 columns, a narrow gate/up and lm_head: totals of a few thousand rows end in a
# ragged round of 256x256 tiles
ROUNDS = configs.ModelShape(n_layers=1, d_model=512, n_q_heads=28, n_kv_heads=4, head_dim=128, ffn_dim=3008,
                            vocab=20011, dtype="bf16")


def _prefix(dm, lens, ids):
    T = sum(lens)
    cu = [0] + [int(x) for x in np.cumsum(lens)]
    hidden = torch.empty((T, dm.shape.d_model), dtype=torch.float32, device=dm.device)
    K, V, h = dm.prefix(cu, ids, None, hidden_out=hidden)
    return cu, K, V, h, hidden


@pytest.mark.parametrize("model,layout,long,lens", [
    (WIDE, 0, 4300, [1, 32, 33, 64, 65, 129, 160, 161, 257, 470]),
    (replace(WIDE, dtype="f16"), rb.RP_WO_TRANSPOSED | rb.RP_W_DOWN_TRANSPOSED, 4300, [31, 96, 128, 200, 320]),
    (BROAD, 0, 7600, [40, 500, 1000, 1500]),
    (BROAD, rb.RP_WO_TRANSPOSED | rb.RP_W_DOWN_TRANSPOSED, 7600, [130, 1499])])
def test_small_tiles_give_the_bits_of_the_large_one(model, layout, long, lens):
    w = configs.custom(model, [1], [0], [0], index=83)
    dm = DeviceModel(inputs.make_weights(w, norm="random", bias=True), max(lens + [long]) + 1, weight_layout=layout)
    rng = np.random.default_rng(7)
    far = rng.integers(0, model.vocab, long, dtype=np.int32)
    for n in lens:
        own = rng.integers(0, model.vocab, n, dtype=np.int32)
        print("rows", n, flush=True)
        ids1 = to_device(own, dm.device)
        cu1, K1, V1, h1, x1 = _prefix(dm, [n], ids1)
        ids2 = to_device(np.concatenate([far, own]), dm.device)
        cu2, K2, V2, h2, x2 = _prefix(dm, [long, n], ids2)
        assert torch.equal(K1, K2[:, long:]) and torch.equal(V1, V2[:, long:])
        assert torch.equal(x1, x2[long:]) and torch.equal(h1[0], h2[1])
        assert torch.isfinite(x1).all()
        if n > 1:
            # scoring: the few rows alone, and among the long sequence's
            few = torch.arange(1, n, dtype=torch.int32, device=dm.device)
            most = torch.arange(long - 1500, long + n, dtype=torch.int32, device=dm.device)
            for flags in (0, rb.RP_SUFFIX_FUSED_LOGPROB):
                a = dm.prompt_logprobs(cu1, ids1, x1, few, flags=flags)
                b = dm.prompt_logprobs(cu2, ids2, x2, most, flags=flags)
                assert torch.equal(a, b[-(n - 1):]), flags
    dm.close()


@pytest.mark.parametrize("model,layout,totals", [
    # q/k/v cut by rows (4688, 5743), by columns (4899, 7642); gate/up by columns (3700, 8650),
    # by rows (4150, 5450); lm_head by rows (1100 of 20011 columns) and columns (1700) below
    (ROUNDS, 0, [3700, 4150, 4688, 4899, 5450, 5743, 7642, 8650]),
    (replace(ROUNDS, dtype="f16"), 0, [4688, 4899]),
    # o and down (3584 columns) by rows (5954, 6587), by columns (6165, 9963)
    (BROAD, 0, [5954, 6165, 6587, 9963]),
    (BROAD, rb.RP_WO_TRANSPOSED | rb.RP_W_DOWN_TRANSPOSED, [5954, 6165, 9963])])
def test_a_cut_last_round_gives_the_bits_of_whole_launches(model, layout, totals):
    w = configs.custom(model, [1], [0], [0], index=84)
    dm = DeviceModel(inputs.make_weights(w, norm="random", bias=True), max(totals) + 1, weight_layout=layout)
    rng = np.random.default_rng(8)
    for total in totals:
        print("rows", total, flush=True)
        # short sequences run on the flexible tiles alone; packed they share the cut launches
        lens = [1500] * (total // 1500) + [total % 1500]
        ids = [rng.integers(0, model.vocab, n, dtype=np.int32) for n in lens]
        all_ids = to_device(np.concatenate(ids), dm.device)
        cu, K, V, h, x = _prefix(dm, lens, all_ids)
        for i, own in enumerate(ids):
            _, K1, V1, h1, x1 = _prefix(dm, [lens[i]], to_device(own, dm.device))
            a, b = cu[i], cu[i + 1]
            assert torch.equal(K[:, a:b], K1) and torch.equal(V[:, a:b], V1), i
            assert torch.equal(x[a:b], x1) and torch.equal(h[i], h1[0]), i
        for n in (1100, 1700):
            pos = torch.arange(1, n + 1, dtype=torch.int32, device=dm.device)
            pos[pos == 1500] = 1499  # not the first token of the second sequence
            for flags in (0, rb.RP_SUFFIX_FUSED_LOGPROB):
                whole = dm.prompt_logprobs(cu, all_ids, x, pos, flags=flags)
                parts = [dm.prompt_logprobs(cu, all_ids, x, p.contiguous(), flags=flags) for p in pos.split(400)]
                assert torch.equal(whole, torch.cat(parts)), flags
    dm.close()
