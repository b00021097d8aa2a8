"""Rays that cross faces of several axes at once, or almost: cameras on lattice points (and next to them) looking along
an axis with slopes of few bits, so that whole diagonals of the image have equal or integer slopes, a row and a column
run parallel to an axis, and rays end on faces.  Counts, voxel ids and chords are the oracle's exactly, where images
are walked in parts (up to 8192 tiles), where they are walked whole, and in both with lists sorted either way."""
import numpy as np
import pytest

from paper_2006_03512_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

AXES = {"z": np.eye(3), "x": np.array([[0, 0, 1], [1, 0, 0], [0, 1, 0.0]]), "-y": np.array([[1, 0, 0], [0, 0, -1], [0, 1, 0.0]])}


def _scene(w, h, grid, voxel, origin, seed):
    rng = np.random.default_rng(seed)
    f = float(2 ** int(np.ceil(np.log2(w / 2))))        # slopes k / f, with the principal point on a pixel
    K = S.Intrinsics(w, h, f, f, float(w // 2), float(h // 2))
    g = S.Grid(*grid, voxel, origin)
    o, n = np.array(origin), np.array(grid)
    poses, depth = [], []
    for R in AXES.values():
        fwd = R[:, 2]
        for eps in (0.0, 2.0 ** -30, 2.0 ** -50):       # on the lattice, and off it by a little
            at = n // 2 - np.rint(fwd).astype(int) * (n // 2 - 1)
            T = np.eye(4)
            T[:3, :3] = R
            T[:3, 3] = (o + at * voxel) * (1.0 + eps) + eps * np.array([1.0, -1.0, 0.5])
            poses.append(T)
            far = 0.8 * voxel * float(np.abs(n @ fwd))
            z = rng.uniform(0.2, 1.0, (h, w)) * far
            k = rng.integers(1, int(far / voxel), (h, w)) * voxel     # surfaces on faces
            depth.append(np.where(rng.random((h, w)) < 0.5, k, z))
    p = S.BuildParams(z_min=0.0, z_max=100.0, trunc_nsigma=2.0, trunc_c0=voxel * 0.5, trunc_c2=0.0, table_dmax=8.0)
    return S.Scene("ties", np.array(depth, np.float32), np.array(poses), K, g, np.zeros((0, 2, 3)), p, np.full(64, 0.05),
                   0.1, 2)


# images of 9 frames: 9 x 30 and 9 x 1020 tiles
@pytest.mark.parametrize("w,h", [(24, 20), (136, 120)])
@pytest.mark.parametrize("grid,voxel,origin", [((32, 32, 32), 0.125, (0.0, -2.0, 1.0)), ((41, 30, 37), 0.1, (-1.3, 0.7, 0.0)),
                                               ((90, 84, 100), 0.03, (-1.35, 0.0, 12.0))])
def test_tied_rays_are_the_oracles(oracle, w, h, grid, voxel, origin):
    from paper_2006_03512_amd import RayMRF
    sc = _scene(w, h, grid, voxel, origin, 5)
    G = oracle.build_graph(sc)
    assert G.n_edges > 20 * G.n_rays * 0.05
    m = RayMRF()
    st = m.build(sc, keep_chords=True)
    assert (st.n_tiles <= 8192) == (w == 24)
    np.testing.assert_array_equal(m.count(sc)[1].sum(), G.n_edges)
    m.build(sc, keep_chords=True)
    inc = {k: v.cpu().numpy() for k, v in m.export_incidence().items()}
    np.testing.assert_array_equal(inc["row_ptr"], G.row_ptr)
    np.testing.assert_array_equal(inc["col"], G.col)
    np.testing.assert_array_equal(inc["t_in"], G.t_in)
    np.testing.assert_array_equal(inc["t_out"], G.t_out)
    np.testing.assert_array_equal(inc["vptr"], G.vptr)
    np.testing.assert_array_equal(inc["vedge"], G.vedge)
    m.close()
