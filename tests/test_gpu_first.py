"""GPU parity of the one-kernel static first block (csrc/laud_first.hip: 64 -> 64 -> 256 channels, bf16, no stride, more than 1024
output pixels) at the edges of its rectangles, of the map and of the workgroups' walk over them.  Tolerance: that of the bf16 parity
tests (two bf16 roundings of intermediates, one of the result)."""
import numpy as np
import pytest

from oracle import laud_oracle as O
from paper_2308_15949_amd import inputs as I
from test_gpu_body import close, oparams, shortcut_params
from test_gpu_parity import G, TOL  # noqa: F401

pytestmark = pytest.mark.gpu


CASES = [
    (2, 41, 25), (2, 23, 31),       # odd in both directions, ragged rectangles
    (1, 1, 1100), (1, 1100, 1), (3, 2, 300), (2, 300, 5),   # rectangles of one row, of one column, limited by their halo and by their height
    (1, 56, 56), (5, 56, 56), (1, 121, 119),                # the shape of ResNet stage 1: fewer rectangles than compute units
    (13, 56, 56), (9, 57, 83), (2, 150, 149),               # two a workgroup
    (768, 4, 4),                                            # mostly empty ones, three a workgroup: input and h2 buffers come round again
    (20, 56, 56), (37, 56, 56), (65, 56, 56),               # up to three, five and eight a workgroup, the last eighth of them ragged
]


@pytest.mark.parametrize("case", [(1, 32, 32), *CASES])  # 1024 rows: the last size of the small tiles
def test_first_block(G, case):  # noqa: F811
    t, L, D = G.torch, G.L, G.D
    N, H, W = case
    x = I.feature_map(5900 + H, N, H, W, 64, I.BF16)
    hb = I.bottleneck_params(5910 + H, 64, 64, 256, I.BF16, relu_out=True, s3_gain=0.5)
    hb.t1 = (np.abs(hb.t1) + 0.25).astype(np.float32)  # positive conv1 shift: the 3x3's padding must be on h1
    wsc, ssc, tsc = shortcut_params(5920 + H, 64, 256, I.BF16)
    ref = O.projection_bottleneck(x, oparams(hb), wsc, ssc, tsc, 1)
    xd = D.to_device(x, I.BF16)
    fx, db = L.fmap_of(xd), D.DeviceBottleneck(hb)
    out = t.full(ref.shape, 7.0, dtype=xd.dtype, device="cuda")
    ws = D.workspace(L.static_bottleneck_workspace(fx, db.desc, 1))
    args = (D.to_device(wsc, I.BF16), t.from_numpy(ssc).cuda(), t.from_numpy(tsc).cuda(), 1)
    L.laud_static_bottleneck(xd, fx, db.desc, *args, out, ws)
    t.cuda.synchronize()
    assert np.array_equal(D.to_host(xd), x)
    close(D.to_host(out), ref, TOL[I.BF16])
    again = t.full(ref.shape, 9.0, dtype=xd.dtype, device="cuda")
    L.laud_static_bottleneck(xd, fx, db.desc, *args, again, ws)
    t.cuda.synchronize()
    assert t.equal(out, again)  # no order of sums that a run may change
