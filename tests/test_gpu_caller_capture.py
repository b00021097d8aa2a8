"""Inferences and reverse passes recorded in a capture of the caller's: every replay gives the eager result for the
inputs that are then in place, under either schedule, with the library's own graph launched between the replays."""
import pytest

from paper_2006_03512_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("schedule", ["plain", "graph"])
@pytest.mark.parametrize("keyframes", [False, True])
def test_replays_of_a_captured_training_step(schedule, keyframes):
    from paper_2006_03512_amd import RayMRF
    sc = S.make_fd()
    m = RayMRF()
    m.build(sc, keyframe_average=keyframes)
    m.set_schedule(schedule)
    sig = torch.tensor(sc.sigma_table, dtype=torch.float32, device="cuda")
    th = [torch.from_numpy(sc.prior_logit()).cuda() + 0.1 * i for i in range(3)]
    dL = torch.ones_like(th[0])

    def step(x, stream=None):
        (m.infer_keyframe_avg if keyframes else m.infer)(x, sig, 4, keep_checkpoints=True, stream=stream)
        return [m.marginals(stream=stream)[1], *m.backward(dL, stream=stream)]

    want = [step(t) for t in th]   # and every buffer allocated
    x = th[2].clone()
    torch.cuda.synchronize()
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=stream):
        got = step(x, stream)
    for i in (1, 2, 0, 1):
        x.copy_(th[i])
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(got, want[i]):
            assert torch.equal(a, b)
        for a, b in zip(step(th[2 - i]), want[2 - i]):   # eager work between the replays
            assert torch.equal(a, b)
        torch.cuda.synchronize()
    m.close()
