"""Depth messages of rays longer than a tile's LDS image holds (more than 512 voxels, up to the longest a graph
takes), a wave per ray: every class of such tiles, images cut at both edges, rays without voxels beside long ones,
exact and per-keyframe averaged messages.  Bounds as in the parity test of the depth messages."""
import numpy as np
import pytest
from test_gpu_depth_rules import _check_depth

from paper_2006_03512_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CLASSES = (640, 768, 1024, 1536, 2048)


def _scene():
    """Two frames of 27x19 pixels down the diagonal of a flat grid, tiles of a column alike in depth: the columns'
    rays cross from a few to about 2000 voxels."""
    K, g = S.Intrinsics(27, 19, 2000.0, 2000.0, 13.0, 9.0), S.Grid(1100, 1000, 40, 0.004)
    poses = np.array([S.look_at((0.05, 0.03, 0.083), (4.3, 3.9, 0.083)), S.look_at((0.1, 0.02, 0.081), (4.2, 3.9, 0.083))])
    steps = np.array([30, 560, 700, 900, 1300, 1800, 1960])          # voxels of the rays of the 7 columns of tiles
    rng = np.random.default_rng(2)
    z = np.repeat(steps, 4)[:27] * 0.004 / 1.42 * rng.uniform(0.97, 1.0, (2, 19, 27))
    z[:, 5:8, ::3] = 0.0
    p = S.BuildParams(z_min=0.05, z_max=8.0, trunc_nsigma=3.0, trunc_c0=0.002, trunc_c2=0.0, table_dmax=8.0)
    tab = np.full(64, 0.01)
    return S.Scene("long", z.astype(np.float32), poses, K, g, np.zeros((0, 2, 3)), p, tab, 0.02, 2)


@pytest.mark.parametrize("keyframes", [False, True])
def test_depth_messages_of_long_rays(oracle, keyframes):
    from paper_2006_03512_amd.mrf import RayMRF
    sc = _scene()
    G = oracle.build_graph(sc)
    n = np.zeros((2, 20, 28), int)
    n[:, :19, :27] = np.diff(G.row_ptr).reshape(2, 19, 27)
    longest = n.reshape(2, 5, 4, 7, 4).max((2, 4))
    assert {CLASSES[int(np.searchsorted(CLASSES, t))] for t in longest.ravel() if t > 512} == set(CLASSES)
    rng = np.random.default_rng(1)
    theta = (sc.prior_logit() + rng.normal(0, 0.5, sc.grid.n_voxels)).astype(np.float32)
    th64 = theta.astype(np.float64)
    m = RayMRF()
    m.build(sc, keyframe_average=keyframes)
    args = torch.from_numpy(theta).cuda(), torch.from_numpy(sc.sigma_table.astype(np.float32)).cuda(), 2
    if keyframes:
        ref = oracle.infer_keyframe_average(G, th64, sc.sigma_table, 2, *oracle.edge_keyframes_and_lengths(G, sc))
        m.infer_keyframe_avg(*args)
    else:
        ref = oracle.infer(G, th64, sc.sigma_table, 2)
        m.infer(*args)
    out = m.depth_distribution()
    _check_depth(G, ref.lam, ref.g, out)
    prob, mean = out["prob"].cpu().numpy().astype(np.float64), out["mean_depth"].cpu().numpy().astype(np.float64)
    ray = np.repeat(np.arange(G.n_rays), np.diff(G.row_ptr))
    want = np.bincount(ray, weights=prob * 0.5 * (G.t_in + G.t_out), minlength=G.n_rays)
    # float32 probabilities (2^-24 each) and residuals Z - d of up to 8 m
    got = np.diff(G.row_ptr) > 0
    assert np.all(np.abs(mean - want)[got] <= 2.0 ** -23 * 8.0 + 2.0 ** -24 * 8.0) and np.all(np.isnan(mean[~got]))
    m.close()
