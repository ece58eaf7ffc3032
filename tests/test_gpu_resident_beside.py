"""On-chip enforcement beside other work: calls of two streams in flight, each stream's enforcement
and solves next to the other's, at the largest model that is held on chip, one that is held with one
workgroup per CU, and one past the limit; and a batch next to solves.  Every result is bitwise what
the call gives alone."""
import numpy as np
import pytest

from tests.gpu_util import dev, need_gpu, torch

pytestmark = pytest.mark.gpu


def _model(n, seed):
    rng = np.random.default_rng(seed + n)
    F = rng.uniform(0.0, 1.0, (n, n + 1)) * (rng.uniform(size=(n, n + 1)) < 0.5)
    F[:, n] += 0.01
    F /= F.sum(axis=1, keepdims=True)
    eps = dev(rng.uniform(0.1, 0.9, n))
    return dev(F), dev(rng.uniform(0.5, 2.0, n)), dev(rng.integers(100, 10000, n).astype(float)), eps, 1.0 - eps


def _streams(count):
    out = [torch.cuda.Stream() for _ in range(count)]
    for s in out:
        s.wait_stream(torch.cuda.current_stream())
    return out


@pytest.mark.parametrize("n", [1300, 1984, 2000])
def test_two_streams_of_enforcement_and_solves(n):
    need_gpu()
    import paper_2511_04277_amd as rad
    models = [_model(n, k) for k in (1, 2)]
    bufs = [(torch.empty_like(m[0]), torch.empty_like(m[0]), rad.Factors(n, "fp64", m[0].device)) for m in models]

    def call(m, b):
        b[0].copy_(m[0])
        rad.enforce_vf_(b[0], m[1], m[2], max_iter=20, want_stats=False)
        rad.gebhart_ref(b[0], m[3], m[4], out=b[1], factors=b[2], want_stats=False)

    want = []
    for m, b in zip(models, bufs):
        call(m, b)
        want.append((b[0].clone(), b[1].clone()))
    streams = _streams(2)
    for _ in range(10):
        for s, m, b in zip(streams, models, bufs):
            with torch.cuda.stream(s):
                call(m, b)
    torch.cuda.synchronize()
    for b, w in zip(bufs, want):
        assert torch.equal(b[0], w[0]) and torch.equal(b[1], w[1])


def test_batch_beside_solves():
    need_gpu()
    import paper_2511_04277_amd as rad
    models = [_model(n, 3) for n in (1984, 1500, 900, 900, 400, 130)]
    start = [m[0].clone() for m in models]
    batch = rad.Batch([{"F": m[0], "area": m[1], "n_rays": m[2], "eps": [m[3]], "rho": [m[4]]} for m in models],
                      precision="fp64")
    F, _, _, eps, rho = _model(2000, 4)
    B, fac = torch.empty_like(F), rad.Factors(2000, "fp64", F.device)

    def run():
        for m, f in zip(models, start):
            m[0].copy_(f)
        batch.run(enforce_iters=20)

    run()
    rad.gebhart_ref(F, eps, rho, out=B, factors=fac, want_stats=False)
    want, want_b = [m[0].clone() for m in models] + [b.clone() for bs in batch.B for b in bs], B.clone()
    one, other = _streams(2)
    for _ in range(6):
        with torch.cuda.stream(one):
            run()
        with torch.cuda.stream(other):
            for _ in range(4):
                rad.gebhart_ref(F, eps, rho, out=B, factors=fac, want_stats=False)
    torch.cuda.synchronize()
    assert torch.equal(B, want_b)
    for a, w in zip([m[0] for m in models] + [b for bs in batch.B for b in bs], want):
        assert torch.equal(a, w)


def test_grids_of_two_threads_take_turns():
    """Enforcement with statistics (the host waits) from two threads, each with a stream of its own."""
    import threading

    need_gpu()
    import paper_2511_04277_amd as rad
    models = [_model(n, 5) for n in (1984, 1700)]
    want, got, failed = [], [[], []], []
    for m in models:
        f = m[0].clone()
        want.append((f, rad.enforce_vf_(f, m[1], m[2], tol=1e-6, max_iter=40)))
    torch.cuda.synchronize()

    def work(k):
        try:
            m = models[k]
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(8):
                    f = m[0].clone()
                    got[k].append((f, rad.enforce_vf_(f, m[1], m[2], tol=1e-6, max_iter=40)))
                torch.cuda.current_stream().synchronize()
        except Exception as e:  # noqa: BLE001
            failed.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed
    for k in (0, 1):
        for f, st in got[k]:
            assert torch.equal(f, want[k][0]) and st == want[k][1]


def test_calls_in_the_shared_scratch_end():
    """rad_enforce_vf_noalloc from two streams at once: undefined results, but every call ends, and the
    next ones are right."""
    need_gpu()
    from paper_2511_04277_amd import _lib as L
    lib = L.lib()
    models = [_model(n, 6) for n in (1200, 700)]

    def call(f, m, stream):
        assert lib.rad_enforce_vf_noalloc(f.data_ptr(), f.shape[0], f.stride(0), m[1].data_ptr(), m[2].data_ptr(),
                                          L.RAD_KAPPA_FRACVAR, 0.0, 30, None, stream.cuda_stream) == 0

    alone = []
    for m in models:
        alone.append(m[0].clone())
        call(alone[-1], m, torch.cuda.current_stream())
        torch.cuda.synchronize()
    streams = _streams(2)
    for _ in range(6):
        for s, m in zip(streams, models):
            with torch.cuda.stream(s):
                call(m[0].clone(), m, s)
    torch.cuda.synchronize()
    for m, want in zip(models, alone):
        f = m[0].clone()
        call(f, m, torch.cuda.current_stream())
        torch.cuda.synchronize()
        assert torch.equal(f, want)
