"""A batch with more runs than their numbers have bits for keeps lists of edges: the bits are lowered with those of the
slot groups, so that six scenes of 1e6 edge slots pass the limit.  Voxel -> ray lists as the oracle's, beliefs
as the exported messages give them, gradients as those of the lists of runs, frames added to the last scene."""
import dataclasses

import numpy as np
import pytest

from paper_2006_03512_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _scenes(log2):
    # pixels wider than the voxels: hardly two rays of a tile cross a voxel; in an order in which the last scene is a
    # group of its own, also without its last frame
    out = [S.random_scene(300 + i, grid=(200, 190, 100), voxel=0.02, n_frames=3,
                          intr=S.Intrinsics(64, 48, 45.0, 45.0, 31.5, 23.5)) for i in (0, 1, 4, 5, 2, 3)]
    for s in out:
        s.params = dataclasses.replace(out[0].params, group_slots_log2=log2)
    return out


def _run(m, st, sigma):
    rng = np.random.default_rng(3)
    theta = torch.from_numpy(rng.normal(-2, 0.5, st.n_voxels).astype(np.float32)).cuda()
    dL = torch.from_numpy(rng.normal(0, 1, st.n_voxels).astype(np.float32)).cuda()
    m.infer(theta, sigma, 2, keep_checkpoints=True)
    logit, grads = m.marginals()[1], m.backward(dL)
    inc = {k: v.cpu().numpy() for k, v in m.export_incidence().items()}
    ell = m.export_edges()["ell"].cpu().numpy().astype(np.float64)
    want, mag = theta.cpu().numpy().astype(np.float64), np.zeros(st.n_voxels)
    np.add.at(want, inc["col"], ell)
    np.add.at(mag, inc["col"], np.abs(ell))
    err = np.abs(logit.cpu().numpy() - want)
    # one rounding to FP32, and FP64 sums of up to max degree terms
    assert np.all(err <= 2.0 ** -23 * np.abs(want) + 2.0 ** -52 * st.max_voxel_degree * (mag + 10))
    lists = any(k["name"] == "seg_sum_k" for k in m.profile_sweeps(reps=1, include_backward=False))
    return inc, [logit, *grads], lists


def test_more_runs_than_numbers_keeps_lists_of_edges(oracle):
    from paper_2006_03512_amd import RayMRF
    m = RayMRF()
    slots, _ = m.count(_scenes(0))
    log2 = int(np.ceil(np.log2(slots.reshape(6, 3).sum(1).max() + 1)))
    scs = _scenes(log2)
    sigma = torch.from_numpy(scs[0].sigma_table.astype(np.float32)).cuda()
    st = m.build(_scenes(0))
    assert st.n_slots >= 1 << 20 and st.n_slot_groups == 1
    want_inc, want, lists = _run(m, st, sigma)
    assert not lists
    part = scs[:-1] + [dataclasses.replace(scs[-1], depth=scs[-1].depth[:-1], T_wc=scs[-1].T_wc[:-1])]
    got = []
    for added in (False, True):
        st = m.build(part if added else scs)
        if added:
            st = m.add_frames(scs[-1].depth[-1:], scs[-1].T_wc[-1:])
        assert st.n_slot_groups > 1
        inc, res, lists = _run(m, st, sigma)
        assert lists   # more than 2^log2 runs
        for k in inc:
            np.testing.assert_array_equal(inc[k], want_inc[k])
        got.append(res)
    for a, b in zip(*got):   # the same lists, so the same sums
        assert torch.equal(a, b)
    v0 = e0 = 0
    for s in scs:
        G = oracle.build_graph(s)
        np.testing.assert_array_equal(want_inc["vptr"][v0:v0 + G.n_voxels + 1] - e0, G.vptr)
        np.testing.assert_array_equal(want_inc["vedge"][e0:e0 + G.n_edges] - e0, G.vedge)
        v0, e0 = v0 + G.n_voxels, e0 + G.n_edges
    # sums of FP64 terms in another order: within the parity bar of the gradients
    for a, b in zip(got[0][1:], want[1:]):
        assert float((a - b).norm()) <= 1e-3 * float(b.norm())
    m.close()
