"""Depth messages in every tile class: tiles of up to 16, 64, ... 512 steps (staged in LDS) and longer
ones (walked by a thread per ray), images that are no multiple of a tile, rays without voxels, and each
output asked for alone.  Bounds as in the parity test of the depth messages (1e-4 on probabilities)."""
import numpy as np
import pytest
from test_gpu_depth_rules import _check_depth
from test_gpu_tuning import _long_ray_scenes

from paper_2006_03512_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _scenes():
    out = _long_ray_scenes()
    sc = S.random_scene(24, grid=(90, 70, 40), voxel=0.02, n_frames=2,
                        intr=S.Intrinsics(27, 19, 22.0, 22.0, 13.0, 9.0))
    sc.depth[:, 3:9, 5:14] = 0.0   # rays without a measurement, whole tiles among them
    return out + [sc, S.random_scene(25, grid=(9, 8, 7), voxel=0.1)]


@pytest.mark.parametrize("k", range(5))
def test_depth_messages_per_tile_class(oracle, k):
    from paper_2006_03512_amd.mrf import RayMRF
    sc = _scenes()[k]
    G = oracle.build_graph(sc)
    theta = sc.prior_logit()
    ref = oracle.infer(G, theta.astype(np.float64), sc.sigma_table, 2)
    m = RayMRF()
    m.build(sc)
    m.infer(torch.from_numpy(theta).cuda(), torch.from_numpy(sc.sigma_table.astype(np.float32)).cuda(), 2)
    out = m.depth_distribution()
    _check_depth(G, ref.lam, ref.g, out)
    L = m._L
    prob, mode = torch.empty_like(out["prob"]), torch.empty_like(out["mode_step"])
    mean = torch.empty_like(out["mean_depth"])
    for p, q, r in ((prob, None, None), (None, mode, None), (None, None, mean)):   # one output at a time
        a = [None if x is None else x.data_ptr() for x in (p, q, r)]
        assert L.mrf_depth_distribution(m.handle, *a, None) == 0
    torch.cuda.synchronize()
    assert torch.equal(prob, out["prob"]) and torch.equal(mode, out["mode_step"])
    assert torch.equal(mean.nan_to_num(-1.0), out["mean_depth"].nan_to_num(-1.0))
    m.close()
