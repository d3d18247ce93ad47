"""GPU parity of the split-reduction kernels that take launches with few rows (csrc/laud_skinny.hip), at the edges of their
tiles (16, 32 and 64 rows / columns), of the reduction slices, and of the rules that choose between them and the tiled
kernels."""
import numpy as np
import pytest

import test_gpu_body as body
from oracle import laud_oracle as O
from paper_2308_15949_amd import inputs as I
from test_gpu_parity import G, TOL, assert_close, check_dyn, oracle_params, run_dyn  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    # N, H, W, C, m, S, dtype
    (1, 1, 1, 8, 8, 1, I.BF16),          # one row
    (1, 1, 17, 24, 16, 1, I.F32),        # 17 rows: one past a 16-row tile, three column tiles with a ragged last
    (1, 4, 4, 136, 72, 2, I.BF16),       # 16 rows; K tails in the last slice (136 = 2 x 64 + 8, 72 = 64 + 8)
    (1, 3, 11, 520, 40, 1, I.F32),       # 33 rows, seventeen slices of the first 1x1: more than one per wave
    (1, 7, 7, 2048, 512, 1, I.BF16),     # 72 slices of the 3x3 on eight waves
    (3, 14, 14, 1024, 256, 2, I.BF16),   # 588 rows, 32 x 32 tiles
    (9, 14, 14, 1024, 256, 2, I.BF16),   # 1764 rows, 32 x 64 tiles
    (21, 14, 14, 1024, 256, 2, I.BF16),  # 4116 rows: past the line to the register-weight kernels
    (1, 128, 128, 16, 8, 4, I.BF16),     # 256 tiles of 64 x 64: the last size of the split-reduction first 1x1
    (1, 128, 132, 16, 8, 4, I.BF16),     # 264 tiles: past it
    (1, 56, 64, 32, 16, 8, I.F32),
    (1, 104, 128, 16, 8, 4, I.BF16),     # 208 tiles: the last size of the last 1x1 (a residual is read) ...
    (1, 88, 152, 16, 8, 4, I.BF16),      # ... 209
    (1, 112, 128, 16, 8, 4, I.BF16),     # 224 tiles: the last size of a 3x3 of nine slices ...
    (1, 120, 120, 16, 8, 4, I.BF16),     # ... 225
    (1, 96, 96, 16, 72, 4, I.BF16),      # 288 tiles: the last size of a 3x3 of more slices ...
    (1, 80, 116, 16, 72, 4, I.BF16),     # ... 290
    (1, 128, 256, 16, 8, 4, I.F32),      # 512 tiles: the last size of a float32 3x3 ...
    (1, 108, 304, 16, 8, 4, I.F32),      # ... 513
    (1, 104, 128, 520, 64, 4, I.BF16),   # 208 tiles: the last size of a first 1x1 of more than eight slices ...
    (1, 88, 152, 520, 64, 4, I.BF16),    # ... 209
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("inplace", [True, False])
def test_few_rows_dyn_block(G, case, inplace):  # noqa: F811
    N, H, W, C, m, S, dt = case
    x = I.feature_map(4000 + C + H, N, H, W, C, dt)
    hb = I.bottleneck_params(4100 + C, C, m, C, dt, relu_out=bool(m % 16))
    hb.t1 = (np.abs(hb.t1) + 0.25).astype(np.float32)  # positive conv1 shift: the 3x3's padding must be on h1
    mask = I.bernoulli_mask(4200 + H + S, (N, H // S, W // S), 0.5)
    mask.reshape(-1)[0] = 1
    check_dyn(run_dyn(G, x, hb, S, mask, inplace), x, hb, S, mask)


@pytest.mark.parametrize("case", [(1, 4, 4, 136, 72, 2, I.BF16), (1, 2, 17, 24, 16, 1, I.F32), (1, 14, 14, 1024, 256, 7, I.BF16),
                                  (2, 12, 12, 2048, 128, 4, I.BF16)])
@pytest.mark.parametrize("use_keep", [False, True])
def test_few_rows_fused_masker(G, case, use_keep):  # noqa: F811
    t, L, D = G.torch, G.L, G.D
    N, H, W, C, m, S, dt = case
    x = I.feature_map(4300 + C, N, H, W, C, dt)
    hb = I.bottleneck_params(4400 + C, C, m, C, dt, True)
    w = I.masker_weights(4500 + C, C)
    ref0 = O.mask_logits(x, S, w, 0.0)
    bias = I.bias_for_ratio(ref0, 0.5, window=max(2, ref0.size // 8))[0]
    keep = np.ones(N, np.uint8)
    keep[-1] = 0
    mask = O.threshold(ref0 + bias)
    if use_keep:
        mask = mask * keep[:, None, None]
    xd, db = D.to_device(x, dt), D.DeviceBottleneck(hb)
    fx, n = L.fmap_of(xd), mask.size
    mk, idx = t.full((n,), 9, dtype=t.uint8, device="cuda"), t.zeros(n, dtype=t.int32, device="cuda")
    cnt, lg = t.zeros(1, dtype=t.int32, device="cuda"), t.zeros(n, dtype=t.float32, device="cuda")
    ws = D.workspace(L.workspace_size(L.binding.OP_DYN_BOTTLENECK, fx, db.desc, S))
    ws.fill_(0xFF)
    L.laud_masker_dyn_bottleneck(xd, fx, db.desc, S, t.from_numpy(w).cuda(), bias, t.from_numpy(keep).cuda() if use_keep else None,
                                 mk, idx, cnt, None, None if use_keep else lg, xd, ws)
    t.cuda.synchronize()
    assert np.array_equal(mk.cpu().numpy().reshape(mask.shape), mask)
    assert np.array_equal(idx.cpu().numpy()[:int(cnt.item())], np.flatnonzero(mask))
    if not use_keep:
        assert_close(lg.cpu().numpy().reshape(ref0.shape), ref0 + bias, 2e-5, "logits")
    check_dyn(D.to_host(xd), x, hb, S, mask)


@pytest.mark.parametrize("case", [(22, 14, 14, 320, 256, 1024, 1, 2, I.BF16, True, "bern"),
                                  (17, 32, 32, 40, 256, 1024, 2, 4, I.BF16, True, "bern")])
def test_dense_first_conv_before_fused_kernel(case):
    """A dynamic first block whose input width the register-weight first 1x1 does not take, with enough rows for the fused
    3x3 -> 1x1 kernel and no caller-packed weights: the call re-orders them itself, whichever way its first 1x1 runs."""
    body.test_dyn_projection_block(case)


# shortcut and first 1x1 in one launch: N, H, W, c_in, m, c_out, stride, S, dtype
PAIR_CASES = [
    (1, 1, 1, 8, 8, 16, 1, 1, I.BF16),          # one row each
    (1, 9, 7, 40, 24, 72, 2, 1, I.F32),         # 20 and 63 rows, ragged columns on both sides
    (1, 3, 11, 520, 40, 136, 2, 1, I.BF16),     # nine slices: more than one per wave
    (1, 14, 14, 1024, 512, 2048, 2, 1, I.BF16),  # 32 x 32 tiles
    (3, 14, 14, 512, 256, 1024, 1, 2, I.BF16),  # 32 x 64
    (1, 48, 64, 32, 64, 256, 1, 4, I.BF16),     # 64 x 64
    (2, 28, 28, 96, 64, 256, 1, 4, I.F32),      # float32, 64 x 64
    # 192 + 64 tiles of 64 x 64 in one launch, 200 + 100 in two.  In float32: over a million outputs of eight mid channels
    # in bf16, the roundings of h2 (eight products of up to 2^-9 each, of either sign: 8 x 0.2 %), of the shortcut and of the output
    # (2^-9 each) add up to 2 % of |ref| + rms at the worst, in one launch and in two (whose outputs are equal bit for bit).
    (1, 64, 64, 16, 8, 192, 1, 4, I.F32), (1, 64, 100, 16, 8, 128, 1, 4, I.F32),
]


@pytest.mark.parametrize("case", PAIR_CASES)
def test_few_rows_shortcut_and_first_conv(case):
    body.test_dyn_projection_block((*case, True, "bern"))
    N, H, W, ci, m, co, stride, _, dt = case
    body.test_static_projection_block((N, H, W, ci, m, co, stride, dt))
