"""The flexible-tile GEMM against the 256x256 one: a sequence alone (few rows, small tiles)
must give bitwise what it gives packed before a long one (many rows, 256x256 tiles), since
every tile forms each output with the same MFMA chain.  Row counts sit on the edges of the
32-, 64-, 128-, 160- and 256-row tiles.  The library is asked which kernel and tile each launch
takes, and a test fails where the tiles that it names are not compared with the 256x256 kernel.
The long packed run itself is compared with the oracle by the other parity tests' models."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2608_14498_amd import binding as rb
from paper_2608_14498_amd import configs, inputs
from paper_2608_14498_amd.runtime import DeviceModel, to_device
from tests.test_dispatch_cpu import gemm_form

pytestmark = pytest.mark.gpu

WIDE = configs.ModelShape(n_layers=2, d_model=128, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn_dim=20480,
                          vocab=152064, dtype="bf16")
BROAD = configs.ModelShape(n_layers=1, d_model=3584, n_q_heads=8, n_kv_heads=2, head_dim=128, ffn_dim=192,
                           vocab=1003, dtype="bf16")
# q/k/v of 4608 columns, a narrow gate/up and lm_head: totals of a few thousand rows end in a
# ragged round of 256x256 tiles
ROUNDS = configs.ModelShape(n_layers=1, d_model=512, n_q_heads=28, n_kv_heads=4, head_dim=128, ffn_dim=3008,
                            vocab=20011, dtype="bf16")


TRANSPOSED = rb.RP_WO_TRANSPOSED | rb.RP_W_DOWN_TRANSPOSED


def _forms(m, rows, layout):
    """(form, flexible tile) of each GEMM of a prefix layer over this many rows."""
    hq, qkv = m.n_q_heads * m.head_dim, (m.n_q_heads + 2 * m.n_kv_heads) * m.head_dim
    return {"qkv": gemm_form(m.dtype, rows, qkv, m.d_model, "rope"),
            "o": gemm_form(m.dtype, rows, m.d_model, hq, "add", trans=bool(layout & rb.RP_WO_TRANSPOSED)),
            "gate_up": gemm_form(m.dtype, rows, m.ffn_dim, m.d_model, "swiglu"),
            "down": gemm_form(m.dtype, rows, m.d_model, m.ffn_dim, "add", trans=bool(layout & rb.RP_W_DOWN_TRANSPOSED))}


def _head_form(m, rows, flags):
    return gemm_form(m.dtype, rows, m.vocab, m.d_model, "lse" if flags & rb.RP_SUFFIX_FUSED_LOGPROB else "store_f32")


def _prefix(dm, lens, ids):
    T = sum(lens)
    cu = [0] + [int(x) for x in np.cumsum(lens)]
    hidden = torch.empty((T, dm.shape.d_model), dtype=torch.float32, device=dm.device)
    K, V, h = dm.prefix(cu, ids, None, hidden_out=hidden)
    return cu, K, V, h, hidden


# tiles: those (100 RF + 10 SW + NS) that some length alone takes where the packed launch runs
# 256x256 tiles over its rows
@pytest.mark.parametrize("model,layout,long,lens,tiles", [
    (WIDE, 0, 4300, [1, 32, 33, 64, 65, 129, 160, 161, 257, 470],
     {"gate_up": {255, 454, 554, 542}, "lm_head": {246, 445, 542}}),
    (replace(WIDE, dtype="f16"), 0, 4300, [31, 96, 128, 200, 320], {"gate_up": {255, 454, 554}, "lm_head": {246, 445, 542}}),
    (BROAD, 0, 7600, [40, 500, 1000, 1500], {"qkv": {246, 445}, "o": {246, 445, 843}, "down": {246, 445, 843}}),
    (BROAD, TRANSPOSED, 7600, [130, 1000, 1499], {"o": {246, 445, 843}, "down": {246, 445, 843}}),
    (replace(BROAD, dtype="f16"), TRANSPOSED, 7600, [130, 1000, 1499], {"o": {246, 445, 843}, "down": {246, 445, 843}})])
def test_small_tiles_give_the_bits_of_the_large_one(model, layout, long, lens, tiles):
    w = configs.custom(model, [1], [0], [0], index=83)
    dm = DeviceModel(inputs.make_weights(w, norm="random", bias=True), max(lens + [long]) + 1, weight_layout=layout)
    rng = np.random.default_rng(7)
    far = rng.integers(0, model.vocab, long, dtype=np.int32)
    seen = {name: set() for name in ("qkv", "o", "gate_up", "down", "lm_head")}

    def note(name, alone, packed):  # the rows of the short sequence are the first: those of a cut's head
        if alone[0] == "flex" and packed[0] in ("256", "cut rows", "cut columns"):
            seen[name].add(alone[1])

    for n in lens:
        own = rng.integers(0, model.vocab, n, dtype=np.int32)
        alone, packed = _forms(model, n, layout), _forms(model, n + long, layout)
        print("rows", n, alone, packed, flush=True)
        for name in alone:
            note(name, alone[name], packed[name])
        ids1 = to_device(own, dm.device)
        cu1, K1, V1, h1, x1 = _prefix(dm, [n], ids1)
        ids2 = to_device(np.concatenate([own, far]), dm.device)
        cu2, K2, V2, h2, x2 = _prefix(dm, [n, long], ids2)
        assert torch.equal(K1, K2[:, :n]) and torch.equal(V1, V2[:, :n])
        assert torch.equal(x1, x2[:n]) and torch.equal(h1[0], h2[0])
        assert torch.isfinite(x1).all()
        if n > 1:
            # scoring: the few rows alone, and before rows of the long sequence
            few = torch.arange(1, n, dtype=torch.int32, device=dm.device)
            most = torch.cat([few, torch.arange(n + 1, n + 1501, dtype=torch.int32, device=dm.device)])
            for flags in (0, rb.RP_SUFFIX_FUSED_LOGPROB):
                note("lm_head", _head_form(model, n - 1, flags), _head_form(model, n + 1499, flags))
                a = dm.prompt_logprobs(cu1, ids1, x1, few, flags=flags)
                b = dm.prompt_logprobs(cu2, ids2, x2, most, flags=flags)
                assert torch.equal(a, b[:n - 1]), flags
    dm.close()
    for name, want in tiles.items():
        assert seen[name] >= want, (name, seen[name])


R, C = "cut rows", "cut columns"


@pytest.mark.parametrize("model,layout,totals", [
    (ROUNDS, 0, {3700: {"gate_up": C}, 4150: {"gate_up": R}, 4688: {"qkv": R}, 4899: {"qkv": C},
                 5450: {"gate_up": R, "qkv": C}, 5743: {"qkv": R}, 7642: {"qkv": C}, 8650: {"gate_up": C}}),
    (replace(ROUNDS, dtype="f16"), 0, {4688: {"qkv": R}, 4899: {"qkv": C}}),
    (BROAD, 0, {5954: {"o": R, "down": R}, 6165: {"o": C, "down": C}, 6587: {"o": R, "down": R}, 9963: {"o": C, "down": C}}),
    (BROAD, TRANSPOSED, {5954: {"o": R, "down": R}, 6165: {"o": C, "down": C}, 9963: {"o": C, "down": C}})])
def test_a_cut_last_round_gives_the_bits_of_whole_launches(model, layout, totals):
    # the lm_head's cuts are of 1100 and 1700 rows below
    for total, want in totals.items():
        forms = _forms(model, total, layout)
        assert {k: forms[k][0] for k in want} == want, (total, forms)
    if model.vocab == ROUNDS.vocab:
        for flags in (0, rb.RP_SUFFIX_FUSED_LOGPROB):
            assert [_head_form(model, n, flags)[0] for n in (1100, 1700, 400)] == [R, C, "flex"]
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
