"""One context's inferences across rebuilds: the captured sweeps are replayed only while every buffer they read is
where it was.  The build between has more edge slots but no more (keyframe, voxel) pairs, so that with the first
build's reserve only buffers without one have to grow."""
import pytest

from paper_2006_03512_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _scene(seed, w, h, grid):
    f = 0.9 * w
    return S.random_scene(seed, grid=grid, voxel=2.0 / max(grid), n_frames=1,
                          intr=S.Intrinsics(w, h, f, f, (w - 1) / 2, (h - 1) / 2))


@pytest.mark.parametrize("keyframes", [False, True])
def test_rebuild_with_moved_buffers(keyframes):
    from paper_2006_03512_amd import RayMRF
    a, b = _scene(51, 320, 240, (96, 90, 80)), _scene(52, 640, 480, (48, 45, 40))
    sig = torch.tensor(a.sigma_table, dtype=torch.float32, device="cuda")
    th = torch.from_numpy(a.prior_logit()).cuda()

    def infer(m):
        (m.infer_keyframe_avg if keyframes else m.infer)(th, sig, 3)
        return m.marginals()[1]

    m = RayMRF()
    st = m.build(a, keyframe_average=keyframes, reserve_frames=4)
    slots, pairs = st.n_slots, st.n_keyframe_pairs
    assert slots >= 1 << 20   # lists of runs
    want = infer(m)
    st = m.build(b, keyframe_average=keyframes)
    assert st.n_slots > slots and st.n_keyframe_pairs <= pairs
    m.accuracy(torch.zeros(st.n_voxels, device="cuda"))   # the build is used, but not for an inference
    m.build(a, keyframe_average=keyframes, reserve_frames=4)
    assert torch.equal(infer(m), want)
    m.close()
