"""GPU parity of a dynamic first block whose output map passes what 32-bit offsets reach (64 -> 256 -> 1024 channels on samples of 128 x
128, bf16: x and h1 stay below 2 GiB, the output takes 33.5 MB a sample)."""
import numpy as np
import pytest

from oracle import laud_oracle as O
from paper_2308_15949_amd import binding as B
from paper_2308_15949_amd import inputs as I
from test_gpu_body import close, oparams, shortcut_params
from test_gpu_parity import G, TOL  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [64, 65, 129])  # the last size of 32-bit offsets, the first past it, and one whose offsets would come round
def test_dyn_projection_block_with_an_output_past_2_gib(G, N):  # noqa: F811
    """One image N times: every sample gets the first one's bits, and those are the oracle's within the bf16 tolerance."""
    t, L, D = G.torch, G.L, G.D
    H, S, dt = 128, 4, I.BF16
    x = I.feature_map(7100, 1, H, H, 64, dt)
    hb = I.bottleneck_params(7101, 64, 256, 1024, dt, relu_out=True, s3_gain=0.5)
    wsc, ssc, tsc = shortcut_params(7102, 64, 1024, dt)
    mask = I.bernoulli_mask(7103, (1, H // S, H // S), 0.3)
    ref = O.dyn_projection_bottleneck(x, oparams(hb), wsc, ssc, tsc, 1, S, mask)
    xd = D.to_device(x, dt).expand(N, H, H, 64).contiguous()
    fx, db = L.fmap_of(xd), D.DeviceBottleneck(hb)
    npatch = N * mask.size
    idx = t.zeros(npatch, dtype=t.int32, device="cuda")
    cnt = t.zeros(1, dtype=t.int32, device="cuda")
    L.laud_layer_skip_compact(t.from_numpy(np.tile(mask.reshape(-1), N)).cuda(), npatch, idx, cnt,
                              D.workspace(L.workspace_size(B.OP_COMPACT, fx, None, npatch)))
    out = t.full((N, H, H, 1024), 7.0, dtype=xd.dtype, device="cuda")
    L.laud_dyn_projection_bottleneck(xd, fx, db.desc, D.to_device(wsc, dt), t.from_numpy(ssc).cuda(), t.from_numpy(tsc).cuda(), 1, S, idx, cnt,
                                     out, D.workspace(L.dyn_projection_workspace(fx, db.desc, 1)))
    t.cuda.synchronize()
    close(D.to_host(out[:1]), ref, TOL[dt])
    first = out[0].view(t.int16)
    assert all(t.equal(out[n].view(t.int16), first) for n in range(1, N))
