"""Inputs that the on-chip enforcement refuses, at the largest grids and with workgroups that start at
different times (solves of another stream hold the chip): a bad entry in the first, in an off-diagonal
and in the last tile pair, a bad space entry, a row without exchange, a bad area.  The documented code
comes back, F is as it was, the next call works, and in a batch the other models keep their bits and
the codes are those of the streamed enforcement."""
import numpy as np
import pytest

from tests.gpu_util import dev, need_gpu, torch

pytestmark = pytest.mark.gpu


def _nan_first(F, area):
    F[1, 0] = np.nan


def _nan_corner(F, area):
    F[0, F.shape[0] - 1] = np.nan


def _negative_last(F, area):
    n = F.shape[0]
    F[n - 1, n - 2] = -1.0


def _negative_space(F, area):
    F[-1, -1] = -1.0


def _empty_row(F, area):
    F[2, :] = 0.0
    F[:, 2] = 0.0


def _bad_area(F, area):
    area[-1] = 0.0


def _bad_area_and_entry(F, area):
    """The areas are checked before the first sweep."""
    _bad_area(F, area)
    _negative_last(F, area)


def _empty_row_and_bad_entry(F, area):
    """The entry belongs to row blocks other than the row's: a bad entry counts first."""
    _empty_row(F, area)
    F[-2, -3] = -1.0


SPOILS = [(_nan_first, -2), (_nan_corner, -2), (_negative_last, -2), (_negative_space, -2), (_empty_row, -3),
          (_empty_row_and_bad_entry, -2), (_bad_area, -1), (_bad_area_and_entry, -1)]


def _model(n, seed):
    rng = np.random.default_rng(seed + n)
    F = rng.uniform(0.0, 1.0, (n, n + 1)) * (rng.uniform(size=(n, n + 1)) < 0.5)
    F[:, n] += 0.01
    F /= F.sum(axis=1, keepdims=True)
    return F, rng.uniform(0.5, 2.0, n), rng.integers(100, 10000, n).astype(float)


class _Solves:
    """Solves in flight on a stream of their own."""

    def __init__(self, n=1500):
        import paper_2511_04277_amd as rad
        F, _, _ = _model(n, 90)
        eps = np.full(n, 0.5)
        self.call = lambda: rad.gebhart_ref(self.F, self.eps, self.eps, out=self.B, factors=self.fac, want_stats=False)
        self.F, self.eps = dev(F), dev(eps)
        self.B, self.fac = torch.empty_like(self.F), rad.Factors(n, "fp64", self.F.device)
        self.stream = torch.cuda.Stream()
        self.stream.wait_stream(torch.cuda.current_stream())

    def start(self, count):
        with torch.cuda.stream(self.stream):
            for _ in range(count):
                self.call()


def _bits(t):
    return t.contiguous().view(torch.int64)


@pytest.mark.parametrize("n", [300, 1300, 1984])
def test_single_call(n):
    need_gpu()
    import paper_2511_04277_amd as rad
    from paper_2511_04277_amd._lib import RadError
    F, area, rays = _model(n, 1)
    solves = _Solves()
    want = dev(F)
    rad.enforce_vf_(want, dev(area), dev(rays), max_iter=4)
    for spoil, code in SPOILS:
        for busy in (0, 3):
            f, a = F.copy(), area.copy()
            spoil(f, a)
            f, a, r = dev(f), dev(a), dev(rays)
            before = f.clone()
            print(f"[errors] n={n} {spoil.__name__} busy={busy}", flush=True)
            solves.start(busy)
            with pytest.raises(RadError) as e:
                rad.enforce_vf_(f, a, r, max_iter=4)
            assert e.value.code == code
            assert torch.equal(_bits(f), _bits(before))
    f = dev(F)
    rad.enforce_vf_(f, dev(area), dev(rays), max_iter=4)
    assert torch.equal(f, want)


def _device_status(batch):
    """Per model the smallest code of its enforcement and its solve (a NaN is also a singular pivot)."""
    from paper_2511_04277_amd import _lib as L
    out = (L.RadStats * batch.count)()
    L.lib().rad_batch_stats(batch._plan, batch.work.data_ptr(), out, torch.cuda.current_stream().cuda_stream)
    return [s.device_status for s in out]


@pytest.mark.parametrize("spoil,code", SPOILS)
def test_model_of_a_batch(spoil, code):
    """A captured run streams all models, one launch per step."""
    need_gpu()
    import paper_2511_04277_amd as rad
    solves = _Solves()
    models, want = [], []
    for k, n in enumerate((1300, 1200, 300, 130)):
        F, area, rays = _model(n, 10 + k)
        if k == 1:
            spoil(F, area)
        models.append((dev(F), dev(area), dev(rays)))
        want.append(dev(F))
        if k != 1:
            rad.enforce_vf_(want[k], models[k][1], models[k][2], max_iter=5)
    half = [dev(np.full(m[0].shape[0], 0.5)) for m in models]
    batch = rad.Batch([{"F": m[0], "area": m[1], "n_rays": m[2], "eps": [h], "rho": [h]}
                       for m, h in zip(models, half)], precision="fp64")
    print(f"[errors] batch {spoil.__name__}", flush=True)
    solves.start(3)
    batch.run(enforce_iters=5)
    got = _device_status(batch)
    assert got[1] <= code and got[0] == got[2] == got[3] == 0
    for m, w in zip(models, want):
        assert torch.equal(_bits(m[0]), _bits(w))
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        batch.run(enforce_iters=5)
    g.replay()
    assert _device_status(batch) == got


def _overflow(F, area):
    """Finite at first, beyond the range after one iteration."""
    area[0], area[-1] = 1e200, 1e-200
    F[0, F.shape[0] - 1] = 0.5


def _stats(s):
    return [s.iters, s.converged, s.closure_defect, s.recip_err]


@pytest.mark.parametrize("n", [2, 40, 64, 300, 1300, 1984])
@pytest.mark.parametrize("spoil", [f for f, _ in SPOILS] + [_overflow])
def test_statistics_of_a_refused_call(n, spoil):
    """Of the last iteration that was completed, as of the streamed enforcement (a captured run)."""
    need_gpu()
    import paper_2511_04277_amd as rad
    from paper_2511_04277_amd import _lib as L
    if n < 6 and spoil in (_empty_row, _empty_row_and_bad_entry):
        pytest.skip("too few rows")
    lib, stream = L.lib(), torch.cuda.current_stream().cuda_stream
    F, area, rays = _model(n, 3)
    spoil(F, area)
    start, a, r, half = dev(F), dev(area), dev(rays), dev(np.full(n, 0.5))
    f = start.clone()
    batch = rad.Batch([{"F": f, "area": a, "n_rays": r, "eps": [half], "rho": [half]}], precision="fp64",
                      kappa="half")

    def batch_stats():
        out = (L.RadStats * 1)()
        lib.rad_batch_stats(batch._plan, batch.work.data_ptr(), out, stream)
        return _stats(out[0])

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        batch.run(enforce_iters=5)
    g.replay()
    want = batch_stats()
    f.copy_(start)
    batch.run(enforce_iters=5)
    assert batch_stats() == want
    f.copy_(start)
    work = torch.empty(lib.rad_enforce_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    st = L.RadStats()
    code = lib.rad_enforce_vf(f.data_ptr(), n, f.stride(0), a.data_ptr(), r.data_ptr(), L.RAD_KAPPA_HALF, 0.0, 5,
                              work.data_ptr(), work.numel(), st, stream)
    assert code == st.device_status < 0
    assert _stats(st) == want
    assert want[0] == (1 if spoil is _overflow else 0)
