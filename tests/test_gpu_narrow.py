"""GPU parity of the kernel of the 64-wide bf16 blocks (csrc/laud_narrow.hip: c_mid = 64, c_out = 256, more than 14336 rows) at
the edges of its 128-row tiles, of the workgroups' walk over them and of the map, and of the one-kernel stem (csrc/laud_static.hip)
at the edges of its strips and steps.  Tolerance: that of the bf16 parity tests (two bf16 roundings of intermediates, one of the
result)."""
import numpy as np
import pytest

from oracle import laud_oracle as O
from paper_2308_15949_amd import inputs as I
from test_gpu_body import close, oparams, shortcut_params
from test_gpu_parity import G, TOL, check_dyn, run_dyn  # noqa: F401

pytestmark = pytest.mark.gpu


def patch_mask(kind, seed, shape):
    mk = np.zeros(shape, np.uint8)
    if kind == "ones":
        mk[:] = 1
    elif kind == "corners":     # one patch per tile row and column edge, far from a full tile
        mk[0, 0, 0] = mk[-1, -1, -1] = 1
    elif kind == "first":       # everything in the first sample: tiles of one XCD's eighth only
        mk[0] = 1
    elif kind == "bern":
        mk = I.bernoulli_mask(seed, shape, 0.5)
    return mk


@pytest.mark.parametrize("case", [
    # N, H, W, S, mask, relu_out
    (1, 128, 112, 4, "bern", True),      # 14336 rows: the last size of the small tiles
    (1, 103, 140, 1, "ones", False),     # 14420 rows, ragged last tile, odd height
    (1, 121, 119, 1, "bern", True),      # 14399 rows, odd in both directions
    (5, 56, 56, 7, "bern", False),       # patches of 49 pixels straddle tiles
    (5, 56, 56, 56, "first", True),      # whole samples
    (5, 56, 56, 2, "corners", True),     # eight rows: one tile
    (5, 56, 56, 4, "zeros", True),
    (12, 56, 56, 8, "ones", True),       # 294 tiles: more than one per workgroup
    (25, 56, 56, 4, "bern", False),
])
@pytest.mark.parametrize("inplace", [True, False])
def test_narrow_dyn_block(G, case, inplace):  # noqa: F811
    N, H, W, S, kind, relu = case
    x = I.feature_map(5000 + H + S, N, H, W, 256, I.BF16)
    hb = I.bottleneck_params(5100 + S, 256, 64, 256, I.BF16, relu_out=relu)
    hb.t1 = (np.abs(hb.t1) + 0.25).astype(np.float32)  # positive conv1 shift: the 3x3's padding must be on h1
    mask = patch_mask(kind, 5200 + H, (N, H // S, W // S))
    check_dyn_or_copy(run_dyn(G, x, hb, S, mask, inplace), x, hb, S, mask)


def check_dyn_or_copy(got, x, hb, S, mask):
    if mask.any():
        check_dyn(got, x, hb, S, mask)
    else:
        assert np.array_equal(got, x)


STATIC_CASES = [
    (1, 241, 239, 2), (12, 112, 112, 2), (21, 112, 112, 2),  # in front of a stride: fewer tiles than compute units, up to two and three a workgroup
    (612, 7, 7, 1), (1400, 7, 7, 1), (20000, 1, 1, 1),       # maps too small for the rectangles of laud_first.hip
]


@pytest.mark.parametrize("case", STATIC_CASES)
def test_narrow_static_first_block(G, case):  # noqa: F811
    t, L, D = G.torch, G.L, G.D
    N, H, W, stride = case
    x = I.feature_map(5300 + H, N, H, W, 64, I.BF16)
    hb = I.bottleneck_params(5400 + H, 64, 64, 256, I.BF16, relu_out=True, s3_gain=0.5)
    hb.t1 = (np.abs(hb.t1) + 0.25).astype(np.float32)
    wsc, ssc, tsc = shortcut_params(5500 + H, 64, 256, I.BF16)
    ref = O.projection_bottleneck(x, oparams(hb), wsc, ssc, tsc, stride)
    xd = D.to_device(x, I.BF16)
    fx, db = L.fmap_of(xd), D.DeviceBottleneck(hb)
    out = t.full(ref.shape, 7.0, dtype=xd.dtype, device="cuda")
    ws = D.workspace(L.static_bottleneck_workspace(fx, db.desc, stride))
    ws.fill_(0xFF)
    L.laud_static_bottleneck(xd, fx, db.desc, D.to_device(wsc, I.BF16), t.from_numpy(ssc).cuda(), t.from_numpy(tsc).cuda(), stride, out, ws)
    t.cuda.synchronize()
    assert np.array_equal(D.to_host(xd), x)
    close(D.to_host(out), ref, TOL[I.BF16])


@pytest.mark.parametrize("case", [
    (1, 1, 1), (1, 7, 300), (1, 27, 30), (1, 29, 34),   # one pixel; one strip cut along x; one past a strip and past a step
    (300, 20, 20),                                      # more strips than compute units
    (90, 90, 46),                                       # four strips an image, the last ragged
    # two workgroups a compute unit, 512: more strips than that, of two steps, of four strips an image; three strips a workgroup, three steps
    (600, 20, 20), (140, 90, 46), (1100, 13, 66),
])
def test_stem_one_kernel(G, case):  # noqa: F811
    t, L, D = G.torch, G.L, G.D
    N, H, W = case
    g = np.random.default_rng(5600 + H)
    x = I.round_to(g.standard_normal((N, H, W, 3), dtype=np.float32), I.BF16)
    w7 = I.round_to(g.standard_normal((64, 7, 7, 3), dtype=np.float32) * np.float32(np.sqrt(2.0 / 147)), I.BF16)
    s, b = (1 + 0.1 * g.standard_normal(64)).astype(np.float32), (0.1 * g.standard_normal(64)).astype(np.float32)
    ref = O.stem(x, w7, s, b)
    out = t.full(ref.shape, 7.0, dtype=t.bfloat16, device="cuda")
    L.laud_stem(D.to_device(x, I.BF16), N, H, W, I.BF16, D.to_device(w7, I.BF16), t.from_numpy(s).cuda(), t.from_numpy(b).cuda(),
                64, out, D.workspace(L.stem_workspace(N, H, W, 64, I.BF16)))
    t.cuda.synchronize()
    close(D.to_host(out), ref, TOL[I.BF16])


@pytest.mark.parametrize("case", [
    # N, H, W, c_out: edges of the matrix-core 3x3 stem (even width from 4 on, channels in 32s, 32 output pixels a tile)
    (1, 1, 4, 32), (2, 2, 2, 32), (1, 3, 6, 32), (2, 5, 62, 32), (2, 6, 64, 64), (3, 7, 66, 32), (2, 9, 65, 32), (2, 8, 66, 40),
    (70, 240, 4, 32),  # more tiles than waves
])
def test_stem3x3_matrix_cores(G, case):  # noqa: F811
    t, L, D = G.torch, G.L, G.D
    N, H, W, co = case
    g = np.random.default_rng(5700 + W)
    x = I.round_to(g.standard_normal((N, H, W, 3), dtype=np.float32), I.BF16)
    w3 = I.round_to(g.standard_normal((co, 3, 3, 3), dtype=np.float32) * np.float32(np.sqrt(2.0 / 27)), I.BF16)
    s, b = (1 + 0.1 * g.standard_normal(co)).astype(np.float32), (0.1 * g.standard_normal(co)).astype(np.float32)
    ref = O.stem3x3(x, w3, s, b)
    out = t.full(ref.shape, 7.0, dtype=t.bfloat16, device="cuda")
    L.laud_stem3x3(D.to_device(x, I.BF16), N, H, W, I.BF16, D.to_device(w3, I.BF16), t.from_numpy(s).cuda(), t.from_numpy(b).cuda(), co, out)
    t.cuda.synchronize()
    close(D.to_host(out), ref, TOL[I.BF16])
