"""Which kernels a call's launches take, asked of the library without a GPU: the rules of the
dispatch have to hold over the shapes of all models, not only at the sizes they were timed at."""
import ctypes
from dataclasses import replace

import pytest

from paper_2608_14498_amd import binding as rb
from paper_2608_14498_amd import configs
from tests.test_abi_cpu import make

SMALL = configs.ModelShape(n_layers=2, d_model=512, n_q_heads=6, n_kv_heads=3, head_dim=128, ffn_dim=1536, vocab=4096,
                           dtype="bf16")
SMALL64 = replace(SMALL, n_q_heads=8, n_kv_heads=2, head_dim=64, ffn_dim=1024, dtype="f16")
TWO_WAYS = replace(SMALL, ffn_dim=2048)  # a down projection in two K splits


def suffix_chunks(handle, prefix, lens, of=None):
    """Key-chunk slots of the suffix attention of responses `lens` over one prefix, or over prefixes
    `prefix` [of[i]] (negative: a workgroup takes all chunks)."""
    arr = lambda v: (ctypes.c_int32 * len(v))(*v)
    f = rb.lib().rp_test_suffix_chunks
    f.restype = ctypes.c_int32
    f.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_void_p, ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p]
    cums = []
    for sizes in ([prefix] if of is None else prefix, lens):
        cu = [0]
        for n in sizes:
            cu.append(cu[-1] + n)
        cums.append(arr(cu))
    return f(handle, len(cums[0]) - 1, cums[0], len(lens), arr(of or [0] * len(lens)), cums[1])


@pytest.mark.parametrize("model", [SMALL, SMALL64, TWO_WAYS, configs.QWEN7B_SLICE, configs.QWEN32B_SLICE])
def test_a_lone_response_spreads_a_long_prefix_over_workgroups(model):
    """At least the chunks that the prefix's length asks for (one per 4096 keys, eight at most),
    each on a workgroup of its own: the workspace holds their partials for every model."""
    h, keep = make(model, 60000)
    try:
        for prefix in (300, 4096, 8191, 8192, 12288, 16384, 30000, 32768, 50000):
            for n in (1, 48, 64, 300, 900):
                got = suffix_chunks(h, prefix, [n])
                assert got >= max(1, min(8, prefix // 4096)), (prefix, n, got)
    finally:
        rb.rp_destroy(h)


def _heads(hq, hkv, d_model, ffn, head_dim=128, dtype="bf16"):
    return replace(SMALL, n_layers=1, n_q_heads=hq, n_kv_heads=hkv, d_model=d_model, ffn_dim=ffn, head_dim=head_dim,
                   dtype=dtype)


SIX, TWELVE, WIDE, HALF = (_heads(6, 3, 1024, 8192), _heads(12, 2, 1024, 8192), _heads(28, 4, 3584, 18944),
                           _heads(16, 2, 1024, 8192, 64, "f16"))


# batches whose two forms differ by a fifth and more: us of the attention, one workgroup for all
# chunks / a workgroup for each
@pytest.mark.parametrize("model,prefix,lens,whole", [
    (TWELVE, 16384, [700] * 8, False),    # 881 / 654: 528 blocks, a second round of 16
    (TWELVE, 32768, [1400] * 8, False),   # 2803 / 2398
    (TWELVE, 16384, [3000] * 2, False),   # 913 / 708
    (WIDE, 16384, [300] * 8, False),      # 885 / 655
    (WIDE, 1500, [48], False),            # 36 / 23
    (HALF, 32768, [300] * 8, False),      # 628 / 462
    (SIX, 1024, [128] * 64, True),        # 56 / 102: 384 blocks
    (SIX, 1024, [200] * 40, True),        # 57 / 109
    (HALF, 1024, [128] * 16, True),       # 27 / 49
    (TWELVE, 1024, [40] * 128, True),     # 63 / 141
    (WIDE, 4096, [40] * 128, True),       # 482 / 695
    (HALF, 8192, [40] * 128, True)])      # 298 / 411
def test_chunks_take_the_faster_form(model, prefix, lens, whole):
    h, keep = make(model, 60000)
    try:
        got = suffix_chunks(h, prefix, lens)
        assert abs(got) > 1 and (got < 0) == whole, got
    finally:
        rb.rp_destroy(h)


@pytest.mark.parametrize("model", [configs.QWEN7B_SLICE, configs.QWEN32B_SLICE])
def test_suffix_partials_share_one_memory(model):
    """The attention's partials lie in the GEMMs' memory: up to seven chunks a longer prefix asks
    for no more workspace (R responses' tokens and the logits alone count)."""
    h, keep = make(model, 60000)
    try:
        want = {p: rb.rp_suffix_workspace_bytes(h, 1, [0, p], [0, 256]) for p in (300, 4096, 8192, 16384, 30000)}
        assert len(set(want.values())) == 1, want
        assert rb.rp_suffix_workspace_bytes(h, 1, [0, 40000], [0, 256]) >= want[300]
    finally:
        rb.rp_destroy(h)


EPI = dict(store_f32=1, add=2, swiglu=3, lse=4, partials=5, rope=6)
FORMS = ["none", "f32", "skinny", "flex", "256", "cut rows", "cut columns"]


def gemm_form(dtype, M, N, K, epi, splitk=1, trans=False):
    """(form, flexible tile as 100 RF + 10 SW + NS or 0) of a GEMM launch."""
    f = rb.lib().rp_test_gemm_form
    f.restype, f.argtypes = ctypes.c_int32, [ctypes.c_int32] * 7 + [ctypes.c_void_p]
    tile = ctypes.c_int32()
    form = f(rb._DTYPES[dtype], M, N, K, int(trans), EPI[epi], splitk, ctypes.byref(tile))
    return FORMS[form], tile.value


@pytest.mark.parametrize("model", [configs.QWEN7B_SLICE, configs.QWEN32B_SLICE])
@pytest.mark.parametrize("epi", ["lse", "store_f32"])
def test_a_row_tail_does_not_read_the_lm_head_again(model, epi):
    """A cut by rows reads B twice: of the lm_head, 1 GB for the few rows of the last round, which
    took 3 to 6% longer than the launch left whole (772 to 926 rows, 7B)."""
    for rows in range(65, 4000, 3):
        assert gemm_form("bf16", rows, model.vocab, model.d_model, epi)[0] != "cut rows", rows


def decode_deep(handle, batch, cap):
    """Whether a decode step's attention runs one wave per 1024-key chunk."""
    f = rb.lib().rp_test_decode_deep
    f.restype, f.argtypes = ctypes.c_int32, [ctypes.c_void_p, ctypes.c_int32, ctypes.c_int32]
    return bool(f(handle, batch, cap))


@pytest.mark.parametrize("model,batch,cap,deep", [
    (TWELVE, 64, 1000, False), (TWELVE, 1, 200, False),  # one record: no merge where it is written directly
    (WIDE, 16, 1100, False), (WIDE, 32, 2048, False), (TWELVE, 32, 3072, False), (HALF, 16, 3072, False),
    (WIDE, 16, 3072, True), (WIDE, 1, 4000, True), (TWELVE, 16, 6000, True), (HALF, 4, 9000, True),
    (WIDE, 64, 4000, False)])  # more chunks than compute units
def test_decode_attention_takes_the_faster_form(model, batch, cap, deep):
    h, keep = make(model, 60000)
    try:
        assert decode_deep(h, batch, cap) == deep
    finally:
        rb.rp_destroy(h)
