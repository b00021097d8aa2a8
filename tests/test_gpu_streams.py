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


@pytest.mark.parametrize("keyframes", [False, True])
def test_eager_sweeps_captured_by_the_caller_after_a_graph(keyframes):
    """A caller's own capture of the sweeps (plain schedule), after and between replays of the library's graph:
    every replay gives the eager result for the inputs that are then in place."""
    from paper_2006_03512_amd import RayMRF
    sc = S.make_fd()
    m = RayMRF()
    m.build(sc, keyframe_average=keyframes)
    sig = torch.tensor(sc.sigma_table, dtype=torch.float32, device="cuda")
    th = [torch.from_numpy(sc.prior_logit()).cuda() + 0.1 * i for i in range(3)]
    infer = m.infer_keyframe_avg if keyframes else m.infer
    want = {}
    for schedule in ("plain", "graph"):   # the last launch before the capture is a replay
        m.set_schedule(schedule)
        for i, t in enumerate(th):
            infer(t, sig, 4)
            want[schedule, i] = m.marginals()[1]
    x = th[0].clone()
    torch.cuda.synchronize()
    m.set_schedule("plain")
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=stream):
        infer(x, sig, 4, stream=stream)
        got = m.marginals(stream=stream)[1]
    m.set_schedule("graph")
    for i in (1, 2, 0, 1):
        x.copy_(th[i])
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want["plain", i])
        infer(th[2 - i], sig, 4)   # eager work between the replays
        assert torch.equal(m.marginals()[1], want["graph", 2 - i])
        torch.cuda.synchronize()
    m.close()
