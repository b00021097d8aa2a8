"""The bytes of a forward sweep that the statistics state are those of its kernels, on graphs kept as lists of edges
and as runs."""
import pytest

from paper_2006_03512_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,runs", [(64, 48, False), (320, 240, True)])
def test_sweep_bytes_are_the_kernels(w, h, runs):
    from paper_2006_03512_amd import RayMRF
    sc = S.random_scene(61, grid=(96, 90, 40), voxel=0.02, n_frames=1,
                        intr=S.Intrinsics(w, h, 0.9 * w, 0.9 * w, (w - 1) / 2, (h - 1) / 2))
    m = RayMRF()
    st = m.build(sc)
    assert (st.n_slots >= 1 << 20) == runs
    m.infer(torch.from_numpy(sc.prior_logit()).cuda(), torch.tensor(sc.sigma_table, dtype=torch.float32).cuda(), 2)
    kernels = m.profile_sweeps(reps=1, include_backward=False)
    assert any(k["name"].startswith("run_sum_k") for k in kernels) == runs
    # the kernels leave out the totals that the ray phase gathers (4 bytes a touched voxel) and tiles without a ray
    rest = st.fwd_bytes_per_sweep - sum(k["bytes_per_launch"] for k in kernels) - 4 * st.n_touched_voxels
    assert rest >= 0 and rest % 36 == 0 and rest < 36 * st.n_tiles
    m.close()
