"""The forms a decode step takes by batch size give one sequence the same bits: alone it runs
one wave per 1024-key chunk (deep ring, chunk merge), in a large batch three chunks per
workgroup, with one record (the result written directly) or several.  Where both forms convert
to fp16 a single rounding can fall otherwise once in some 2^13 values, so that model's sequences
are all compared.  The gate/up projection that sums its K chunks itself (7B: two of them) gives
the bits of the split-K partials that it takes the place of."""
import ctypes
from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle
from paper_2608_14498_amd import binding as rb
from paper_2608_14498_amd import configs, inputs
from paper_2608_14498_amd.runtime import DeviceModel, to_device
from tests.gpu_helpers import max_abs
from tests.test_dispatch_cpu import decode_deep

pytestmark = pytest.mark.gpu

WIDE_F = configs.ModelShape(n_layers=2, d_model=256, n_q_heads=8, n_kv_heads=4, head_dim=128, ffn_dim=12800,
                            vocab=1003, dtype="bf16")
F16_D64 = configs.ModelShape(n_layers=2, d_model=256, n_q_heads=16, n_kv_heads=8, head_dim=64, ffn_dim=512,
                             vocab=1003, dtype="f16")


@pytest.mark.parametrize("model,cap,edges,alone", [
    (WIDE_F, 2200, [0, 1, 31, 32, 33, 1023, 1024, 1056, 2047, 2048, 2199], 11),
    (replace(WIDE_F, dtype="f16"), 4200, [159, 160, 161, 3071, 3072, 3073, 4199], 7),
    (F16_D64, 3000, [0, 127, 1025, 2999], 63),   # one record
    (F16_D64, 3100, [0, 127, 1025, 3099], 63)])  # two
def test_alone_and_in_a_batch_the_same_bits(model, cap, edges, alone):
    B = 63
    w = configs.custom(model, [1], [0], [1], index=86)
    hw = inputs.make_weights(w, norm="random", bias=True)
    kv_len = np.resize(np.array(edges, np.int32), B)
    dec = inputs.make_decode(w, batch=B, kv_len=kv_len, cap=cap)
    dm = DeviceModel(hw, cap + 1)
    ck, cv = to_device(dec.cache_k, dm.device), to_device(dec.cache_v, dm.device)
    lens, ids = to_device(dec.kv_len, dm.device), to_device(dec.token_ids, dm.device)

    def step(rows):
        logits = torch.empty((len(rows), model.vocab), dtype=torch.float32, device=dm.device)
        nxt = dm.decode(ck[:, rows].contiguous(), cv[:, rows].contiguous(), lens[rows].contiguous(),
                        ids[rows].contiguous(), logits=logits)
        return logits, nxt

    assert decode_deep(dm.handle, 1, cap) and not decode_deep(dm.handle, B, cap)
    lg, nx = step(list(range(B)))
    assert torch.isfinite(lg).all()
    assert torch.equal(nx.long(), lg.argmax(1))
    print("model", model.dtype, model.head_dim, "cap", cap, flush=True)
    differ = []
    for b in range(alone):
        l1, n1 = step([b])
        if not (torch.equal(l1[0], lg[b]) and int(n1[0]) == int(nx[b])):
            differ.append((b, int(kv_len[b])))
    assert not differ
    n = min(4, len(edges))
    lo = oracle.decode_step(hw.as_f32(), model, inputs.to_f32(dec.cache_k[:, :n]), inputs.to_f32(dec.cache_v[:, :n]),
                            dec.kv_len[:n], dec.token_ids[:n])[0]
    # 16-bit decode logits of two layers: 2e-2, the bound of the decode parity tests
    assert max_abs(lg[:n].cpu().numpy(), lo) <= 2e-2
    dm.close()


# gate/up with K summed in chunks in the kernel, and as split-K partials added by the SwiGLU kernel
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("K,chunks", [(512, 2), (704, 2), (768, 3), (896, 3), (3584, 2)])
def test_chunked_gate_up_gives_the_bits_of_its_partials(dtype, K, chunks):
    """704 and 896: the last chunk is shorter (6 + 5 and 5 + 5 + 4 slabs).  F = 18944 takes the 7B
    weights' two chunks."""
    f = rb.lib().rp_test_gate_up
    f.restype, f.argtypes = ctypes.c_int32, [ctypes.c_void_p] + [ctypes.c_int32] * 4 + [ctypes.c_void_p] * 5
    t = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    g = torch.Generator(device="cuda").manual_seed(5)
    F = 18944 if K == 3584 else 12864
    gate, up = (torch.randn((F, K), generator=g, device="cuda").mul_(K ** -0.5).to(t) for _ in range(2))
    stream = torch.cuda.current_stream().cuda_stream
    for M in (1, 31, 32, 33, 63, 64):
        x = torch.randn((M, K), generator=g, device="cuda").to(t)
        part = torch.full((chunks, M, 2 * F), float("nan"), device="cuda")
        out = [torch.full((M, F), float("nan"), device="cuda", dtype=t) for _ in range(2)]
        print("rows", M, flush=True)
        for p, o in zip((None, part), out):
            got = f(stream, rb._DTYPES[dtype], M, F, K, x.data_ptr(), gate.data_ptr(), up.data_ptr(),
                    None if p is None else p.data_ptr(), o.data_ptr())
            assert got == chunks
        torch.cuda.synchronize()
        assert torch.equal(out[0], out[1]), M
        a, b = x.double() @ gate.double().T, x.double() @ up.double().T
        want = a / (1 + torch.exp(-a)) * b
        # fp32 sums of K terms and one rounding to 16 bits (8 or 11 significant bits)
        assert float((out[0].double() - want).norm() / want.norm()) <= {"bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dtype]
