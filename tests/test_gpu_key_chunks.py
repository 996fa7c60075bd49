"""Attention over a long first key segment in key chunks: a response alone (its chunks on
workgroups of their own, then merged) must give bitwise what it gives in a batch whose blocks
fill the chip (all chunks in one workgroup).  Parity with the oracle is the other tests'.  Response
lengths sit on the edges of the chunk rule (blocks of 128 packed rows, chunks of 256 keys, 1024 keys and more cut) and
of the 4- and 8-wave blocks.  The library is asked which form each launch takes, so that the two
sides of a comparison are known to differ."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2608_14498_amd import configs, inputs
from paper_2608_14498_amd.runtime import DeviceModel, to_device
from tests.test_dispatch_cpu import suffix_chunks

pytestmark = pytest.mark.gpu

# the memory of 8 K splits of the down projection holds the partials of 7 chunks
MODEL = configs.ModelShape(n_layers=1, d_model=512, n_q_heads=8, n_kv_heads=2, head_dim=64, ffn_dim=8192, vocab=515,
                           dtype="bf16")
F16 = replace(MODEL, dtype="f16")
WIDE_HEADS = replace(MODEL, d_model=1024, n_q_heads=6, n_kv_heads=3, head_dim=128)
FIVE_CHUNKS = replace(WIDE_HEADS, d_model=512, dtype="f16")  # memory for 5


@pytest.mark.parametrize("model,prefix,lens,fill", [
    (MODEL, [512, 1023, 1024, 1501, 8192], [1, 16, 17, 32, 33, 48, 64, 65, 96, 97, 129, 300], 256),
    (F16, [8192, 1501], [16, 48, 129, 300], 256),
    (WIDE_HEADS, [2047, 1025], [1, 42, 43, 64, 85, 200], 200),
    (replace(WIDE_HEADS, dtype="f16"), [8192, 1501], [1, 42, 43, 64, 85, 200], 250),
    (FIVE_CHUNKS, [2047, 1025], [1, 42, 43, 64, 85, 200], 200),
    (MODEL, [1793, 1100], [8200, 31, 64], 6)])
def test_chunks_alone_and_in_a_batch(model, prefix, lens, fill):
    """fill: responses in the batch, enough of them that a workgroup takes all chunks.  The
    8200-token responses put theirs in 8-wave blocks."""
    w = configs.custom(model, [1], [0], [0], index=85)
    dm = DeviceModel(inputs.make_weights(w, norm="random", bias=True), max(prefix) + max(lens) + 1)
    g = torch.Generator(device="cuda").manual_seed(3)
    K, V = dm.alloc_kv(sum(prefix))
    K.normal_(0, 0.5, generator=g)
    V.normal_(0, 0.5, generator=g)
    h = torch.empty((len(prefix), model.d_model), device=dm.device).normal_(0, 1, generator=g)
    pcu = [0] + [int(x) for x in np.cumsum(prefix)]
    rng = np.random.default_rng(4)
    want = (lens * fill)[:fill]
    of = sorted(int(x) for x in rng.integers(0, len(prefix), fill))
    ids = [rng.integers(0, model.vocab, n, dtype=np.int32) for n in want]
    scu = [0] + [int(x) for x in np.cumsum(want)]
    assert suffix_chunks(dm.handle, prefix, want, of) < 0  # one workgroup takes all chunks
    whole = dm.suffix_grouped(pcu, of, scu, K, V, h, to_device(np.concatenate(ids), dm.device))
    assert torch.isfinite(whole).all()
    seen, split = set(), 0
    for i, (n, p) in enumerate(zip(want, of)):
        if (n, p) in seen:
            continue
        seen.add((n, p))
        chunks = suffix_chunks(dm.handle, prefix[p], [n])
        print("response", n, "prefix", prefix[p], "chunks", chunks, flush=True)
        assert chunks >= 1  # a lone response: its chunks on workgroups of their own
        split += chunks > 1
        k, v = (t[:, pcu[p]:pcu[p + 1]].contiguous() for t in (K, V))
        own = dm.suffix([0, prefix[p]], [0, n], k, v, h[p:p + 1].contiguous(), to_device(ids[i], dm.device))
        assert torch.equal(own, whole[scu[i]:scu[i + 1]]), (n, prefix[p])
    assert 2 * split >= len(seen), split  # at least half: split against folded
    dm.close()
