"""Inferences of one context on several streams run in the order of the calls, on the caller's stream."""
import pytest

from paper_2006_03512_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("keyframes", [False, True])
def test_inferences_on_two_streams_keep_their_order(keyframes):
    from paper_2006_03512_amd import RayMRF
    sc = S.make_fd()
    m = RayMRF()
    m.build(sc, keyframe_average=keyframes)
    sig = torch.tensor(sc.sigma_table, dtype=torch.float32, device="cuda")
    th = [torch.from_numpy(sc.prior_logit()).cuda() + 0.1 * i for i in range(2)]

    def infer(i, stream=None):
        (m.infer_keyframe_avg if keyframes else m.infer)(th[i], sig, 6, stream=stream)

    want = []
    for i in range(2):
        infer(i)
        want.append(m.marginals()[1])
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for k in range(6):   # the other stream each time, no synchronisation between the calls
        for i in range(2):
            infer(i, streams[(k + i) % 2])
        last = streams[(k + 1) % 2]
        with torch.cuda.stream(last):
            got = m.marginals(stream=last)[1]
        last.synchronize()
        assert torch.equal(got, want[1])
    m.close()
