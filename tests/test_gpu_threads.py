"""Contexts in several threads at once, each on a stream of its own: builds with their readbacks, captures of the
sweeps, inferences, reverse passes and added frames give what one thread alone gets."""
import threading

import pytest

from paper_2006_03512_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _work(seed, stream, rounds):
    from paper_2006_03512_amd import RayMRF
    sc = S.random_scene(seed, grid=(48, 40, 30 + seed % 7), voxel=0.05, n_frames=3,
                        intr=S.Intrinsics(64 + 4 * (seed % 3), 48, 55.0, 55.0, 31.5, 23.5))
    out = []
    with torch.cuda.stream(stream):
        th = torch.from_numpy(sc.prior_logit()).cuda()
        sig = torch.tensor(sc.sigma_table, dtype=torch.float32, device="cuda")
        dL = torch.ones_like(th)
        m = RayMRF()
        for k in range(rounds):
            m.upload(sc)
            m.build_resident(keyframe_average=True, stream=stream)
            m.infer(th, sig, 2 + k % 3, keep_checkpoints=True, stream=stream)
            got = [m.marginals(stream=stream)[1], *m.backward(dL, stream=stream)]
            m.add_frames(sc.depth[:1], sc.T_wc[:1], stream=stream)
            m.infer_keyframe_avg(th, sig, 2 + k % 2, stream=stream)
            got.append(m.marginals(stream=stream)[1])
            stream.synchronize()
            out.append([g.cpu() for g in got])
        m.close()
    return out


def test_threads_do_not_disturb_each_other():
    n, rounds = 4, 6
    want = [_work(400 + i, torch.cuda.Stream(), rounds) for i in range(n)]
    got, errors = [None] * n, []

    def run(i, stream):
        try:
            got[i] = _work(400 + i, stream, rounds)
        except Exception as e:   # reported by the main thread
            errors.append((i, repr(e)))

    threads = [threading.Thread(target=run, args=(i, torch.cuda.Stream())) for i in range(n)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for a, b in zip(got, want):
        for x, y in zip(a, b):
            for p, q in zip(x, y):
                assert torch.equal(p, q)
