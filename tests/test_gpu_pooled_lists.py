"""GPU parity of the launch that pools, decides and lists a masker's patches by itself (csrc/laud_mask.hip: k_pool_compact) where it holds less
than a whole block of them, and of masks that are written over the gates they are decided with."""
import numpy as np
import pytest

from paper_2308_15949_amd import inputs as I
from test_gpu_parity import G, test_masker_dyn_bottleneck as masker_block  # noqa: F401

pytestmark = pytest.mark.gpu

# N, H, W, C, m, S, dtype, relu_out, and the threads of the block: widths whose 3x3 leaves the list to a launch of its own
# (tests/test_memory_bounds.py: that they do)
PARTIAL = [
    ((1, 32, 32, 16, 1280, 4, I.BF16, True), 64),      # one full wave
    ((1, 32, 28, 16, 1424, 4, I.BF16, True), 64),      # ... 56 patches
    ((1, 36, 32, 16, 1152, 4, I.BF16, False), 128),    # 72: a second wave of eight
    ((13, 7, 7, 16, 1920, 1, I.BF16, True), 640),      # 637 patches of one pixel
    ((12, 14, 14, 32, 520, 2, I.BF16, True), 640),     # 588 of 2 x 2
    ((5, 32, 32, 1024, 256, 4, I.BF16, True), 320),    # in front of the fused 3x3 -> 1x1
    ((5, 56, 56, 256, 64, 4, I.BF16, True), 1024),     # 980, of the 64-wide blocks
]


@pytest.mark.parametrize("case", [c for c, _ in PARTIAL])
@pytest.mark.parametrize("use_keep", [False, True])
def test_lists_of_less_than_a_block(G, case, use_keep):  # noqa: F811
    masker_block(G, case, True, use_keep)


# ... and those whose list is made in the 3x3 (k_skinny), with the threads of its workgroups: one, two and four patches a thread
IN_3X3 = [
    ((1, 7, 7, 16, 8, 1, I.BF16, True), 512), ((1, 32, 32, 16, 8, 1, I.BF16, True), 512), ((1, 32, 32, 16, 384, 1, I.BF16, True), 256),
    ((2, 14, 14, 16, 8, 2, I.F32, True), 512), ((4, 32, 32, 16, 8, 2, I.BF16, True), 512), ((3, 36, 32, 16, 72, 2, I.BF16, False), 256),
    ((2, 32, 32, 16, 8, 4, I.F32, False), 512), ((7, 32, 36, 16, 8, 4, I.BF16, True), 256), ((13, 32, 32, 16, 8, 4, I.BF16, True), 256),
]


@pytest.mark.parametrize("case", [c for c, _ in IN_3X3])
@pytest.mark.parametrize("use_keep", [False, True])
def test_lists_made_in_the_3x3(G, case, use_keep):  # noqa: F811
    masker_block(G, case, True, use_keep)


# N, S: maps of S x S, one patch a sample, so that mask and gates have the same bytes
IN_PLACE = [(40, 1), (40, 2), (40, 4), (1000, 4), (1100, 4), (3000, 2), (4500, 1), (70, 3)]


@pytest.mark.parametrize("N,S", IN_PLACE)
def test_masks_written_over_their_gates(G, N, S):  # noqa: F811
    t, L, D = G.torch, G.L, G.D
    C, m, dt = 16, 8, I.BF16
    x = D.to_device(I.feature_map(7200 + S, N, S, S, C, dt), dt)
    db, fx, w = D.DeviceBottleneck(I.bottleneck_params(7201, C, m, C, dt, True)), L.fmap_of(x), t.from_numpy(I.masker_weights(7202, C)).cuda()
    gates = t.from_numpy(I.bernoulli_mask(7203 + N, (N,), 0.6)).cuda()
    got = []
    for in_place in (False, True):
        mask, keep = (gates.clone(),) * 2 if in_place else (t.full((N,), 9, dtype=t.uint8, device="cuda"), gates)
        idx, cnt, so = (t.full((k,), -7, dtype=t.int32, device="cuda") for k in (N, 1, N + 1))
        lg, out = t.zeros(N, device="cuda"), t.zeros_like(x)
        L.laud_masker_dyn_bottleneck(x, fx, db.desc, S, w, 0.1, keep, mask, idx, cnt, so, lg, out, D.workspace(L.workspace_size(L.binding.OP_DYN_BOTTLENECK, fx, db.desc, S)))
        t.cuda.synchronize()
        got.append((mask, idx, cnt, so, lg, out))
    assert 0 < int(got[0][2]) < int(gates.sum())
    assert all(t.equal(a, b) for a, b in zip(*got))
    assert np.array_equal(np.flatnonzero(got[0][0].cpu().numpy()), got[0][1].cpu().numpy()[:int(got[0][2])])
