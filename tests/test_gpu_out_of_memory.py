"""An inference whose checkpoints do not fit the device fails and takes with it the last inference's, whose buffers
made room: there is nothing left to differentiate or export, and the next inference is as any other."""
import pytest

from paper_2006_03512_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("keyframes", [False, True])
def test_checkpoints_that_do_not_fit(keyframes):
    from paper_2006_03512_amd import RayMRF
    from paper_2006_03512_amd._lib import MRF_ENOMEM, MRF_ESTATE, MRFError
    sc = S.make_fd()
    m = RayMRF()
    st = m.build(sc, keyframe_average=keyframes)
    th = torch.from_numpy(sc.prior_logit()).cuda()
    sig = torch.tensor(sc.sigma_table, dtype=torch.float32, device="cuda")
    infer = m.infer_keyframe_avg if keyframes else m.infer
    infer(th, sig, 3, keep_checkpoints=True)
    dL = torch.ones_like(th)
    want = [m.marginals()[1], *m.backward(dL)]
    size = 8 * st.n_keyframe_pairs if keyframes else 4 * st.n_slots
    with pytest.raises(MRFError) as e:
        infer(th, sig, min(2 ** 31 - 1, 2 ** 43 // size), keep_checkpoints=True)   # 8 TB
    assert e.value.code == MRF_ENOMEM
    with pytest.raises(MRFError) as e:
        m.backward(dL)
    assert e.value.code == MRF_ESTATE
    infer(th, sig, 3, keep_checkpoints=True)
    for a, b in zip([m.marginals()[1], *m.backward(dL)], want):
        assert torch.equal(a, b)
    m.close()
