"""The fp32 matrix-core kernels at their edges: tiles of 32 rows, keys and columns, K that is
no multiple of the 32-deep loads (8-deep chunks split over four waves), head_dim 128, and
non-finite values of later tokens, which must not reach earlier ones, and scores of -inf."""
import numpy as np
import pytest
import torch

from paper_2608_14498_amd import binding as rb
from paper_2608_14498_amd import configs, inputs
from paper_2608_14498_amd.runtime import DeviceModel, to_device
from tests.gpu_helpers import gpu_run, max_abs, oracle_run, rel_err

pytestmark = pytest.mark.gpu

D64 = configs.ModelShape(n_layers=2, d_model=72, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn_dim=40, vocab=101,
                         dtype="f32")
D128 = configs.ModelShape(n_layers=2, d_model=264, n_q_heads=3, n_kv_heads=1, head_dim=128, ffn_dim=104, vocab=1001,
                          dtype="f32")


@pytest.mark.parametrize("model", [D64, D128])
@pytest.mark.parametrize("layout", [0, rb.RP_WO_TRANSPOSED | rb.RP_W_DOWN_TRANSPOSED])
def test_f32_tile_edges_match_oracle(model, layout):
    P, S = [1, 31, 32, 33, 64, 300], [33, 32, 31, 1, 0, 65]
    w = configs.custom(model, P, [0, 8, 0, 30, 64, 256], S, index=84)
    hw = inputs.make_weights(w, norm="random", bias=True)
    bt = inputs.make_batch(w)
    Ko, Vo, Ho, lpo = oracle_run(w, hw, bt)
    if layout:
        dm = DeviceModel(hw, 512, weight_layout=layout)
        cu_p, cu_s = [int(x) for x in bt.cu_prefix], [int(x) for x in bt.cu_suffix]
        K, V, h = dm.prefix(cu_p, to_device(bt.token_ids, dm.device), to_device(bt.visual, dm.device))
        lp = dm.suffix(cu_p, cu_s, K, V, h, to_device(bt.response_ids, dm.device))
        K, V, H, lp = (t.cpu().numpy() for t in (K, V, h, lp))
        dm.close()
    else:
        K, V, H, lp = gpu_run(w, hw, bt)
    # fp32 sums of at most 300 terms over two layers: the bounds of the tiny fp32 model
    assert rel_err(K, Ko) <= 1e-5 and rel_err(V, Vo) <= 1e-5 and rel_err(H, Ho) <= 1e-5
    assert max_abs(lp, lpo) <= 1e-4


@pytest.mark.parametrize("model", [D64, D128])
@pytest.mark.parametrize("at", [40, 63])
def test_f32_non_finite_token_leaves_earlier_rows(model, at):
    n = 70
    w = configs.custom(model, [n], [n], [0], index=85)
    dm = DeviceModel(inputs.make_weights(w, norm="random", bias=True), 128)
    bt = inputs.make_batch(w)
    ids = to_device(bt.token_ids, dm.device)

    def run(vis):
        hidden = torch.empty((n, model.d_model), dtype=torch.float32, device=dm.device)
        K, V, _ = dm.prefix([0, n], ids, vis, hidden_out=hidden)
        return K, V, hidden

    vis = to_device(bt.visual, dm.device)
    K, V, x = run(vis)
    bad = vis.clone()
    bad[at] = float("nan")
    Kb, Vb, xb = run(bad)
    # (the rows of the bad token's tile take another order of additions: not bitwise)
    for a, b in ((K[:, :at], Kb[:, :at]), (V[:, :at], Vb[:, :at]), (x[:at], xb[:at])):
        assert torch.isfinite(b).all()
        assert float((a - b).abs().max() / a.abs().max()) <= 1e-5
    assert not torch.isfinite(xb[at:]).any()
    dm.close()


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("first,last", [(32, 64), (32, 95), (64, 300), (1, 301)])
def test_f32_keys_of_score_minus_infinity_weigh_nothing(head_dim, first, last):
    """Prefix keys first .. last - 1 hold -inf in the dimension of the slowest rotation, where every
    query is positive: their scores are -inf, whole 32-key tiles of them, and the result is that of
    scores of -1e30."""
    n = 301
    model = configs.ModelShape(n_layers=1, d_model=72, n_q_heads=2, n_kv_heads=1, head_dim=head_dim, ffn_dim=40,
                               vocab=101, dtype="f32")
    w = configs.custom(model, [n], [0], [33], index=87)
    hw = inputs.make_weights(w, norm="random", bias=True)
    lw = hw.layers[0]
    dim = head_dim // 2 - 1  # rotates by n theta^(2 / D - 1): 5e-4 at most
    for h in range(2):
        r = h * head_dim + np.array([dim, dim + head_dim // 2])
        lw["wq"][r] = 0
        lw["bq"][r] = [1, 0]
    bt = inputs.make_batch(w)
    dm = DeviceModel(hw, 512)
    K, V, hl = dm.prefix([0, n], to_device(bt.token_ids, dm.device), None)

    def run(value):
        k = K.clone()
        k[:, first:last, :, dim] = value
        return dm.suffix([0, n], [0, 33], k, V, hl, to_device(bt.response_ids, dm.device))

    want, got = run(-1e30), run(float("-inf"))
    assert torch.isfinite(want).all()
    # fp32 sums of at most 334 terms, in the same order (keys of weight 0 add zeros)
    assert torch.equal(want, got)
    dm.close()
