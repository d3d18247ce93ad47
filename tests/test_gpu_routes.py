"""GPU parity of routes through the entry points that the per-kernel files do not take: index lists that end with their last
entry, on every kernel that reads one; values that are not finite; a mask made on the device in front of the 64-wide kernel."""
import numpy as np
import pytest

from oracle import laud_oracle as O
from paper_2308_15949_amd import inputs as I
from test_gpu_body import close, oparams, shortcut_params
from test_gpu_parity import G, TOL, check_dyn  # noqa: F401

pytestmark = pytest.mark.gpu


def exact_list(t, mask):
    """The ascending ids of the active patches in a tensor of exactly that many entries, and their number."""
    ids = np.flatnonzero(mask).astype(np.int32)
    return t.from_numpy(ids).cuda(), t.tensor([len(ids)], dtype=t.int32, device="cuda")


@pytest.mark.parametrize("case", [
    # N, H, W, C, m, S, dtype
    (1, 56, 56, 256, 64, 4, I.F32),       # small tiles
    (2, 7, 7, 2048, 512, 1, I.BF16),
    (5, 56, 56, 256, 64, 4, I.BF16),      # 64-wide kernel
    (22, 14, 14, 1024, 256, 2, I.BF16),   # register-weight first 1x1, fused 3x3 -> 1x1
    (40, 28, 28, 512, 128, 4, I.BF16),    # tiled kernels
    (22, 14, 14, 1024, 256, 14, I.BF16),  # patches that are whole samples, on the last two
    (40, 28, 28, 512, 128, 28, I.BF16),
    (22, 28, 28, 24, 40, 28, I.F32),
    (17, 28, 28, 64, 72, 28, I.BF16),     # whole samples on narrow maps, which other patches run the first 1x1 of densely
    (21, 28, 28, 512, 136, 28, I.BF16),   # ... long reductions: 2 x 258 tiles of 64 x 128, one round of 128 x 64 ...
    (9, 28, 28, 520, 136, 28, I.BF16),    # ... and 2 x 111: one round
    (66, 7, 7, 520, 584, 1, I.BF16),      # 51 x 5 tiles: every pixel; 52 x 5: listed
    (67, 7, 7, 520, 584, 1, I.BF16),
])
@pytest.mark.parametrize("active", [1, 0.3])
def test_list_of_exact_length(G, case, active):  # noqa: F811
    t, L, D = G.torch, G.L, G.D
    N, H, W, C, m, S, dt = case
    x = I.feature_map(7000 + C, N, H, W, C, dt)
    hb = I.bottleneck_params(7100 + C, C, m, C, dt, relu_out=True)
    if active == 1:  # one entry, the grid's last patch
        mask = np.zeros((N, H // S, W // S), np.uint8)
        mask[-1, -1, -1] = 1
    else:
        mask = I.bernoulli_mask(7200 + H, (N, H // S, W // S), active)
    idx, cnt = exact_list(t, mask)
    xd, db = D.to_device(x, dt), D.DeviceBottleneck(hb)
    fx = L.fmap_of(xd)
    L.laud_dyn_bottleneck(xd, fx, db.desc, S, idx, cnt, xd, D.workspace(L.workspace_size(L.binding.OP_DYN_BOTTLENECK, fx, db.desc, S)))
    t.cuda.synchronize()
    check_dyn(D.to_host(xd), x, hb, S, mask)


@pytest.mark.parametrize("case", [
    (3, 16, 16, 64, 64, 256, 2, 4), (8, 112, 112, 64, 64, 256, 2, 8),
    (30, 56, 55, 64, 104, 104, 2, 28), (30, 28, 28, 512, 256, 1024, 2, 14),  # whole samples
])
def test_projection_list_of_exact_length(G, case):  # noqa: F811
    t, L, D = G.torch, G.L, G.D
    N, H, W, ci, m, co, stride, S = case
    x = I.feature_map(7300 + H, N, H, W, ci, I.BF16)
    hb = I.bottleneck_params(7400 + H, ci, m, co, I.BF16, relu_out=True, s3_gain=0.5)
    wsc, ssc, tsc = shortcut_params(7500 + H, ci, co, I.BF16)
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    mask = I.bernoulli_mask(7600 + H, (N, Ho // S, Wo // S), 0.4)
    ref = O.dyn_projection_bottleneck(x, oparams(hb), wsc, ssc, tsc, stride, S, mask)
    idx, cnt = exact_list(t, mask)
    xd, db = D.to_device(x, I.BF16), D.DeviceBottleneck(hb)
    fx, out = L.fmap_of(xd), t.full(ref.shape, 7.0, dtype=t.bfloat16, device="cuda")
    L.laud_dyn_projection_bottleneck(xd, fx, db.desc, D.to_device(wsc, I.BF16), t.from_numpy(ssc).cuda(), t.from_numpy(tsc).cuda(),
                                     stride, S, idx, cnt, out, D.workspace(L.dyn_projection_workspace(fx, db.desc, stride)))
    t.cuda.synchronize()
    close(D.to_host(out), ref, TOL[I.BF16])


@pytest.mark.parametrize("case", [
    # N, H, W, C, m, S, dtype
    (1, 56, 56, 256, 64, 4, I.BF16),      # small tiles
    (5, 56, 56, 256, 64, 4, I.BF16),      # 64-wide kernel
    (2, 14, 14, 1024, 256, 2, I.BF16),    # small tiles
    (22, 14, 14, 1024, 256, 2, I.BF16),   # fused 3x3 -> 1x1
    (40, 28, 28, 512, 128, 4, I.BF16),    # tiled kernels
])
def test_nan_stays_nan_without_output_relu(G, case):  # noqa: F811
    """One NaN in an active pixel, whatever kernel the batch size selects: the first 1x1's ReLU makes that pixel's h1 zero, the
    residual add gives NaN at that one value of the output, and without an output ReLU it stays NaN."""
    t, L, D = G.torch, G.L, G.D
    N, H, W, C, m, S, dt = case
    x = I.feature_map(7700 + C, N, H, W, C, dt)
    x[N - 1, H - 2, 3, 5] = np.nan
    hb = I.bottleneck_params(7800 + C, C, m, C, dt, relu_out=False)
    mask = I.bernoulli_mask(7900 + H, (N, H // S, W // S), 0.5)
    mask[N - 1, (H - 2) // S, 3 // S] = 1
    idx, cnt = exact_list(t, mask)
    xd, db = D.to_device(x, dt), D.DeviceBottleneck(hb)
    assert int(t.isnan(xd).sum()) == 1
    fx = L.fmap_of(xd)
    L.laud_dyn_bottleneck(xd, fx, db.desc, S, idx, cnt, xd, D.workspace(L.workspace_size(L.binding.OP_DYN_BOTTLENECK, fx, db.desc, S)))
    t.cuda.synchronize()
    got = xd.float().cpu().numpy()
    assert np.argwhere(~np.isfinite(got)).tolist() == [[N - 1, H - 2, 3, 5]] and np.isnan(got[N - 1, H - 2, 3, 5])


@pytest.mark.parametrize("use_keep", [False, True])
@pytest.mark.parametrize("case", [(5, 56, 56, 4), (13, 40, 28, 2)])
def test_masker_into_the_64_wide_kernel_out_of_place(G, case, use_keep):  # noqa: F811
    """The list is made by the launch before: the 64-wide kernel's tiles and its copying workgroups both read it."""
    t, L, D = G.torch, G.L, G.D
    N, H, W, S = case
    x = I.feature_map(8000 + H, N, H, W, 256, I.BF16)
    hb = I.bottleneck_params(8100 + H, 256, 64, 256, I.BF16, relu_out=True)
    w = I.masker_weights(8200, 256)
    ref0 = O.mask_logits(x, S, w, 0.0)
    bias = I.bias_for_ratio(ref0, 0.4, window=ref0.size // 8)[0]
    keep = np.ones(N, np.uint8)
    keep[[0, -2]] = 0
    mask = O.threshold(ref0 + bias) * (keep[:, None, None] if use_keep else 1)
    xd, db = D.to_device(x, I.BF16), D.DeviceBottleneck(hb)
    fx, n = L.fmap_of(xd), mask.size
    mk, idx, cnt = t.zeros(n, dtype=t.uint8, device="cuda"), t.zeros(n, dtype=t.int32, device="cuda"), t.zeros(1, dtype=t.int32, device="cuda")
    out, ws = t.full_like(xd, 7.0), D.workspace(L.workspace_size(L.binding.OP_DYN_BOTTLENECK, fx, db.desc, S))
    ws.fill_(0xFF)
    L.laud_masker_dyn_bottleneck(xd, fx, db.desc, S, t.from_numpy(w).cuda(), bias, t.from_numpy(keep).cuda() if use_keep else None,
                                 mk, idx, cnt, None, None, out, ws)
    t.cuda.synchronize()
    assert np.array_equal(mk.cpu().numpy().reshape(mask.shape), mask)
    assert np.array_equal(D.to_host(xd), x)
    check_dyn(D.to_host(out), x, hb, S, mask)


@pytest.mark.parametrize("shape", [(1, 64, 80), (2, 37, 46)])
def test_stem_infinite_pixel_stays_in_its_windows(G, shape):  # noqa: F811
    """An infinite value of the image makes the windows that cover it infinite (or zero, behind the ReLU) and no other: not the
    ones beside it, whose padded reduction reads the next pixel too."""
    t, L, D = G.torch, G.L, G.D
    N, H, W = shape
    g = np.random.default_rng(7950 + H)
    x = I.round_to(g.standard_normal((N, H, W, 3), dtype=np.float32), I.BF16)
    for y, xx, c in ((5, 7, 0), (5, 30, 2), (H - 1, W - 1, 1), (20, 19, 0), (21, W - 12, 1)):
        x[N - 1, y, xx, c] = np.inf
    w7 = I.round_to(g.standard_normal((64, 7, 7, 3), dtype=np.float32) * np.float32(np.sqrt(2.0 / 147)), I.BF16)
    assert np.all(w7 != 0)
    s, b = (1 + 0.1 * g.standard_normal(64)).astype(np.float32), (0.1 * g.standard_normal(64)).astype(np.float32)
    # a conv value is infinite where it meets an infinite value with a positive weight; -inf, and the NaN of inf - inf, end as 0
    # behind the ReLU
    inf = np.isinf(x).astype(np.float32)
    plus, minus = O.conv2d(inf, np.maximum(w7, 0), 2, 3) > 0, O.conv2d(inf, np.maximum(-w7, 0), 2, 3) > 0
    conv = O.relu(O.affine(O.conv2d(np.where(np.isinf(x), 0, x), w7, 2, 3), s, b))
    finite = O.maxpool3x3_s2(np.where(minus, 0.0, conv))
    want_inf = O.maxpool3x3_s2((plus & ~minus).astype(np.float32)) > 0
    assert want_inf.any() and not want_inf.all()
    out = t.full(finite.shape, 7.0, dtype=t.bfloat16, device="cuda")
    L.laud_stem(D.to_device(x, I.BF16), N, H, W, I.BF16, D.to_device(w7, I.BF16), t.from_numpy(s).cuda(), t.from_numpy(b).cuda(),
                64, out, D.workspace(L.stem_workspace(N, H, W, 64, I.BF16)))
    t.cuda.synchronize()
    got = D.to_host(out)
    assert np.array_equal(np.isposinf(got), want_inf)
    close(np.where(want_inf, 0, got), np.where(want_inf, 0, finite), TOL[I.BF16])
