"""GPU parity of the tiled kernel for many rows (csrc/laud_pipe.h) on each bf16 tile of the block modes (which shapes meet which:
REACHES in test_memory_bounds.py, whose cases have the same sizes): ragged rows, columns and reductions (not
whole 64-channel slices), patches that straddle tiles, lists that fill a fraction of the capacity, the projection of the fused
masker, strides.  Tolerance: that of the parity tests."""
import numpy as np
import pytest

from oracle import laud_oracle as O
from paper_2308_15949_amd import inputs as I
from test_gpu_body import close, oparams, shortcut_params
from test_gpu_group_se import check_group_se, run_group_se
from test_gpu_parity import G, TOL, check_dyn, run_dyn  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    # N, H, W, C, m, S, ratio, relu_out: the 3x3's tile and what it meets
    (21, 28, 28, 72, 40, 4, 0.5, True),     # 128 x 64 throughout; one slice and a bit a tap
    (29, 23, 25, 64, 64, 1, 0.9, False),    # whole slices, odd maps
    (9, 28, 28, 200, 136, 7, 0.5, True),    # 64 x 128, six slices deep, two column tiles
    (26, 28, 28, 80, 136, 4, 0.6, False),   # 128 x 128
    (26, 28, 28, 80, 136, 28, 0.1, True),   # whole samples, few of them
    (21, 28, 28, 72, 40, 14, 1.0, True),
    (100, 7, 7, 520, 136, 1, 0.3, True),    # first 1x1 on 64 x 128, every pixel and listed samples
    (100, 7, 7, 520, 136, 7, 0.3, False),
    (100, 7, 7, 136, 520, 1, 0.3, True),    # last 1x1 on 64 x 128, 128 x 128 and (with listed pixels on 128 x 128 ahead) 128 x 256
    (32, 28, 28, 136, 328, 4, 0.3, False),
    (16, 28, 28, 1032, 456, 4, 0.2, True),
])
@pytest.mark.parametrize("dtype", [I.BF16, I.F32])
def test_dyn_block(G, case, dtype):  # noqa: F811
    N, H, W, C, m, S, ratio, relu = case
    x = I.feature_map(9000 + m, N, H, W, C, dtype)
    hb = I.bottleneck_params(9100 + m, C, m, C, dtype, relu_out=relu)
    hb.t1 = (np.abs(hb.t1) + 0.25).astype(np.float32)  # positive conv1 shift: the 3x3's padding must be on h1
    mask = I.bernoulli_mask(9200 + S, (N, H // S, W // S), ratio)
    mask[-1, -1, -1] = 1
    check_dyn(run_dyn(G, x, hb, S, mask, False), x, hb, S, mask)


@pytest.mark.parametrize("case", [(14, 14, 14, 1032, 264, 2), (40, 21, 21, 104, 72, 3), (23, 28, 28, 40, 56, 4), (3, 30, 30, 4096, 264, 2)])
def test_masker_projection(G, case):  # noqa: F811
    """128 x 128 and 128 x 64 tiles; the first column tile takes the projection of all its rows."""
    t, L, D = G.torch, G.L, G.D
    N, H, W, C, m, S = case
    x = I.feature_map(9300 + C, N, H, W, C, I.BF16)
    hb = I.bottleneck_params(9400 + C, C, m, C, I.BF16, relu_out=True)
    w = I.masker_weights(9500, C)
    ref0 = O.mask_logits(x, S, w, 0.0)
    bias = I.bias_for_ratio(ref0, 0.4, window=ref0.size // 8)[0]
    mask = O.threshold(ref0 + bias)
    xd, db = D.to_device(x, I.BF16), D.DeviceBottleneck(hb)
    fx, n = L.fmap_of(xd), mask.size
    mk, idx, cnt = t.zeros(n, dtype=t.uint8, device="cuda"), t.zeros(n, dtype=t.int32, device="cuda"), t.zeros(1, dtype=t.int32, device="cuda")
    logits = t.zeros(n, dtype=t.float32, device="cuda")
    ws = D.workspace(L.workspace_size(L.binding.OP_DYN_BOTTLENECK, fx, db.desc, S))
    ws.fill_(0xFF)
    L.laud_masker_dyn_bottleneck(xd, fx, db.desc, S, t.from_numpy(w).cuda(), bias, None, mk, idx, cnt, None, logits, xd, ws)
    t.cuda.synchronize()
    assert np.array_equal(mk.cpu().numpy().reshape(mask.shape), mask)
    got = logits.cpu().numpy().reshape(mask.shape)  # float32 sums of C products
    assert np.abs(got - (ref0 + bias)).max() <= 2e-5 * max(1.0, np.abs(ref0).max())
    check_dyn(D.to_host(xd), x, hb, S, mask)


@pytest.mark.parametrize("case", [
    # N, H, W, c_in, m, c_out, stride: 128 x 256 shortcut with a fraction of a slice; 3x3 on the small tiles (267 of them) and 128 x 128
    (32, 28, 28, 8, 64, 264, 1), (7, 57, 55, 72, 136, 96, 2), (9, 129, 127, 16, 72, 80, 1),
    # 3x3 on 64 x 128 (more tiles than the small ones take, one round) and 256 x 128 (two rounds of 128 x 128, one of these)
    (9, 57, 55, 72, 136, 96, 2), (9, 121, 123, 16, 72, 80, 2),
    # last 1x1 on 64 x 128, 128 x 128 and 128 x 256
    (6, 28, 28, 16, 456, 136, 1), (16, 28, 28, 16, 328, 136, 1), (8, 28, 28, 16, 456, 1032, 1),
])
def test_static_first_block(G, case):  # noqa: F811
    t, L, D = G.torch, G.L, G.D
    N, H, W, ci, m, co, stride = case
    x = I.feature_map(9600 + ci, N, H, W, ci, I.BF16)
    hb = I.bottleneck_params(9700 + m, ci, m, co, I.BF16, relu_out=True, s3_gain=0.5)
    hb.t1 = (np.abs(hb.t1) + 0.25).astype(np.float32)
    wsc, ssc, tsc = shortcut_params(9800 + co, ci, co, I.BF16)
    ref = O.projection_bottleneck(x, oparams(hb), wsc, ssc, tsc, stride)
    xd = D.to_device(x, I.BF16)
    fx, db = L.fmap_of(xd), D.DeviceBottleneck(hb)
    out = t.full(ref.shape, 7.0, dtype=xd.dtype, device="cuda")
    ws = D.workspace(L.static_bottleneck_workspace(fx, db.desc, stride))
    ws.fill_(0xFF)
    L.laud_static_bottleneck(xd, fx, db.desc, D.to_device(wsc, I.BF16), t.from_numpy(ssc).cuda(), t.from_numpy(tsc).cuda(), stride, out, ws)
    t.cuda.synchronize()
    close(D.to_host(out), ref, TOL[I.BF16])


@pytest.mark.parametrize("case", [(3, 1, 56), (2, 56, 56), (1, 56, 3)])
def test_copy_of_whole_samples(G, case):  # noqa: F811
    """Out of place with whole samples as patches: the copy is shared out by pixel rows."""
    t, L, D = G.torch, G.L, G.D
    N, kept, H = case[0], case[1] % 2, case[2]
    x = I.feature_map(9900 + H, N, H, H, 256, I.BF16)
    hb = I.bottleneck_params(9910, 256, 64, 256, I.BF16, relu_out=True)
    mask = np.zeros((N, 1, 1), np.uint8)
    mask[N // 2] = kept
    got = run_dyn(G, x, hb, H, mask, False)
    if kept:
        check_dyn(got, x, hb, H, mask)
    else:
        assert np.array_equal(got, x)


@pytest.mark.parametrize("case", [
    # N, H, W, C, g, S, ratio: one and several column tiles, the last with 8, 16 and 48 channels; fewer and more tiles than workgroups
    (5, 56, 56, 64, 64, 4, 0.5), (12, 28, 28, 144, 16, 2, 0.9), (22, 14, 14, 440, 8, 7, 0.3), (9, 41, 37, 48, 8, 1, 0.5),
    (13, 56, 56, 104, 8, 8, 1.0), (4, 28, 28, 832, 32, 28, 0.5),
])
def test_group_conv(G, case):  # noqa: F811
    N, H, W, C, g, S, ratio = case
    x = I.feature_map(9950 + C, N, H, W, C, I.BF16)
    hb = I.bottleneck_params(9960 + C, C, C, C, I.BF16, True, group_width=g)
    mask = I.bernoulli_mask(9970 + S, (N, H // S, W // S), ratio)
    mask[0, 0, 0] = mask[-1, -1, -1] = 1
    check_group_se(run_group_se(G, x, hb, g, None, S, mask, True), x, hb, g, None, S, mask)
