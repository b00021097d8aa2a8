"""Batches of many scenes: the scene of a voxel and of a brick-major key is found for every scene, those without an
edge and the last among them, on graphs kept as lists of edges and as runs."""
import dataclasses

import numpy as np
import pytest

from paper_2006_03512_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,size", [(1, (16, 12)), (2, (16, 12)), (37, (16, 12)), (300, (24, 20))])
def test_batch_is_its_scenes_one_after_the_other(oracle, n, size):
    from paper_2006_03512_amd import RayMRF
    w, h = size
    scs = [S.random_scene(200 + i, grid=(9 + i % 23, 8 + i % 17, 7 + i % 11), voxel=0.1, n_frames=1 + i % 2,
                          intr=S.Intrinsics(w, h, 18.0, 18.0, (w - 1) / 2, (h - 1) / 2)) for i in range(n)]
    p0 = max((s.params for s in scs), key=lambda p: p.z_max)
    for i, s in enumerate(scs):
        s.params = p0
        if i % 7 == 3:
            scs[i] = dataclasses.replace(s, depth=np.zeros_like(s.depth))
    m = RayMRF()
    st = m.build(scs)
    assert (st.n_slots >= 1 << 20) == (n == 300)
    inc = {k: v.cpu().numpy() for k, v in m.export_incidence().items()}
    th = np.concatenate([s.prior_logit() for s in scs])
    m.infer(torch.from_numpy(th).cuda(), torch.from_numpy(scs[0].sigma_table.astype(np.float32)).cuda(), 1)
    p = m.marginals()[0].cpu().numpy()
    r0 = v0 = e0 = 0
    for s in scs:
        G = oracle.build_graph(s)
        R, V, E = G.n_rays, G.n_voxels, G.n_edges
        np.testing.assert_array_equal(inc["row_ptr"][r0:r0 + R + 1] - e0, G.row_ptr)
        np.testing.assert_array_equal(inc["col"][e0:e0 + E] - v0, G.col)
        np.testing.assert_array_equal(inc["vptr"][v0:v0 + V + 1] - e0, G.vptr)
        np.testing.assert_array_equal(inc["vedge"][e0:e0 + E] - e0, G.vedge)
        ref = oracle.infer(G, s.prior_logit().astype(np.float64), scs[0].sigma_table, 1) if E else None
        want = ref.p if E else 1 / (1 + np.exp(-s.prior_logit().astype(np.float64)))
        assert np.abs(p[v0:v0 + V] - want).max() <= 1e-4   # the marginals' bar
        r0, v0, e0 = r0 + R, v0 + V, e0 + E
    assert e0 == st.n_edges and v0 == st.n_voxels
    m.close()
