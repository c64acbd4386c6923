"""Memory that calls share or hand over: a job's device memory is kept for the next
job, and host outputs are written by several threads."""
import ctypes as C
import mmap

import numpy as np
import pytest

from paper_1107_3355_amd import gdpm as G
from paper_1107_3355_amd import inputs as I
from tests.gpu_common import balance, physics_events

pytestmark = pytest.mark.gpu
MATS = I.MATERIALS


def _water(side, d, e=2.0):
    ph = I.homogeneous((side,) * 3, (d,) * 3, I.ID_WATER, 1.0)
    return ph, I.Source(I.PHOTON, I.mono(e), [I.parallel_beam_z(ph, 5.0)])


def _hip():
    return C.CDLL("libamdhip64.so")   # the runtime the library uses


def _on_stream(ctx, p, s, **kw):
    """The job on a stream of its own; dose, sigma and run statistics."""
    hip, n = _hip(), p.desc.nvox
    st, bufs = C.c_void_p(), [C.c_void_p(), C.c_void_p()]
    assert hip.hipStreamCreate(C.byref(st)) == 0
    for b in bufs:
        assert hip.hipMalloc(C.byref(b), C.c_size_t(8 * n)) == 0
    try:
        r = ctx.run_async(p, s, bufs[0].value, bufs[1].value, stream=st.value, **kw)
        for k, b in zip(("dose", "sigma"), bufs):
            r[k] = np.empty(n)
            assert hip.hipMemcpy(r[k].ctypes.data_as(C.c_void_p), b, C.c_size_t(8 * n), 2) == 0
    finally:
        for b in bufs:
            hip.hipFree(b)
        hip.hipStreamDestroy(st)
    return r


def test_memory_of_a_refused_batch():
    """A batch is refused at its last job, with the large tallies of the jobs before it
    still being cleared on the context's stream.  The next job, on another stream, takes
    their memory: nothing may write to it any more (same dose as in a fresh context, to
    the order of the FP64 additions)."""
    ph, src = _water(200, 0.2)
    kw = dict(seed=5, n_hist=20_000, n_batches=10)
    c = G.Context(0, materials=MATS)
    try:
        p, s = c.phantom(ph), c.source(src)
        first = _on_stream(c, p, s, **kw)
        for _ in range(3):
            with pytest.raises(G.GdpmError) as e:
                c.run_batch([(p, s, kw)] * 3 + [(p, s, dict(kw, ecut_e=0.3))], want_dose=False)
            assert e.value.status == 1 and "job 3" in str(e.value)
            r = _on_stream(c, p, s, **kw)
            assert physics_events(r) == physics_events(first) and balance(r) < 1e-12
            np.testing.assert_allclose(r["dose"], first["dose"], rtol=1e-12, atol=1e-12 * first["dose"].max())
    finally:
        c.close()


def test_refused_call_does_not_wait():
    """A call that is refused before it launches anything leaves the caller's stream
    alone: work that the stream holds is still running when the call returns."""
    hip, n = _hip(), 1 << 30
    c = G.Context(0, materials=MATS)
    st, buf = C.c_void_p(), C.c_void_p()
    try:
        ph, src = _water(16, 0.5)
        p, s = c.phantom(ph), c.source(src)
        assert hip.hipStreamCreate(C.byref(st)) == 0 and hip.hipMalloc(C.byref(buf), C.c_size_t(n)) == 0
        kw = dict(stream=st.value, n_hist=100, n_batches=2)
        c.run_async(p, s, buf.value, buf.value + n // 2, **kw)
        for call, bad in ((c.run_async, dict(n_hist=0)), (c.run_noalloc, dict(n_batches=1))):
            for _ in range(1000):   # well over 0.1 s
                assert hip.hipMemsetAsync(buf, 0, C.c_size_t(n), st) == 0
            with pytest.raises(G.GdpmError) as e:
                call(p, s, buf.value, buf.value + n // 2, **dict(kw, **bad))
            busy = hip.hipStreamQuery(st)
            assert hip.hipStreamSynchronize(st) == 0
            assert e.value.status == 1 and busy == 600   # hipErrorNotReady
    finally:
        if st:
            hip.hipStreamSynchronize(st)
            hip.hipStreamDestroy(st)
        hip.hipFree(buf)
        c.close()


@pytest.mark.parametrize("n", [1, 12])
def test_outputs_that_share_an_array(n):
    """One array for the dose and the standard error, of all jobs of a batch (a caller that
    has no use for them): the last values stand in it, whole.  An output is one long and
    one short chunk, and the pages are new, so that a copy is slow and the next one has it
    easy."""
    ph = I.homogeneous((52, 51, 50), (0.2,) * 3, I.ID_WATER, 1.0)
    src = I.Source(I.PHOTON, I.mono(6.0), [I.parallel_beam_z(ph, 5.0)])
    kw = dict(n_hist=300, n_batches=2, flags=G.KERMA)   # all jobs end after one photon pass
    c = G.Context(0, materials=MATS)
    try:
        p, s = c.phantom(ph), c.source(src)
        ref = c.run(p, s, seed=n, **kw)["sigma"]
        for _ in range(20):
            shared = np.frombuffer(mmap.mmap(-1, 8 * ph.nvox), dtype=np.float64)
            jobs = (G.JobDesc * n)(*[G.JobDesc(p.handle, s.handle, G._params(dict(kw, seed=k + 1)), G._dp(shared),
                                               G._dp(shared)) for k in range(n)])
            G._check(G.lib().gdpm_run_batch(c.handle, n, jobs, None, None))
            np.testing.assert_allclose(shared, ref, rtol=1e-9, atol=1e-12 * ref.max())
    finally:
        c.close()


def test_kept_memory_is_given_up_for_other_allocations():
    """With the device full but for half a gibibyte, an allocation that needs what the
    context keeps of its last job (its tallies: 1.5 GB) gets it."""
    hip = _hip()
    c, d = G.Context(0, materials=MATS), G.Context(0, materials=MATS)
    blocks = []
    try:
        ph, src = _water(200, 0.2)
        p, s = c.phantom(ph), c.source(src)
        c.run(p, s, n_hist=100, n_batches=24, want_dose=False)
        d.atomic_rate(1 << 20)
        spare = C.c_void_p()
        assert hip.hipMalloc(C.byref(spare), C.c_size_t(256 << 20)) == 0
        size = 32 << 30
        while size >= 256 << 20:   # fill the device up to less than that
            b = C.c_void_p()
            if hip.hipMalloc(C.byref(b), C.c_size_t(size)) == 0:
                blocks.append(b)
            else:
                hip.hipGetLastError()
                size //= 2
        assert hip.hipFree(spare) == 0
        assert d.atomic_rate(1200 << 20) > 0   # (a buffer of its own, of another context)
        r = c.run(p, s, n_hist=100, n_batches=2, want_dose=False)
        assert r["histories"] == 100
    finally:
        for b in blocks:
            hip.hipFree(b)
        d.close()
        c.close()


def test_server_budget_holds_kept_memory():
    """What a context keeps of finished jobs stays within the budget of the server that
    owns it, together with what the running jobs hold, also where their sizes differ."""
    hip = _hip()

    def free():
        a, b = C.c_size_t(), C.c_size_t()
        assert hip.hipMemGetInfo(C.byref(a), C.byref(b)) == 0
        return a.value

    budget, slack = 300 << 20, 24 << 20   # slack: the runtime's own allocations
    c = G.Context(0, materials=MATS)
    try:
        ph, src = _water(128, 0.25)   # 16.8 MB an array
        p, s = c.phantom(ph), c.source(src)
        c.run(p, s, n_hist=1000, n_batches=2)     # queues
        G.Server(c, budget).close()               # gives back what is kept
        base = free()
        c.run(p, s, n_hist=1000, n_batches=50, want_dose=False)   # 872 MB, kept
        assert base - free() > 2 * budget
        with G.Server(c, budget) as srv:
            assert base - free() <= budget + slack
            for nb in (14, 7, 9, 12, 4, 13):
                jobs = [srv.submit(p, s, n_hist=200_000, n_batches=nb, seed=k) for k in range(3)]
                for j in jobs:
                    assert base - free() <= budget + slack, nb
                    assert j.wait()["histories"] == 200_000
                assert base - free() <= budget + slack, nb
            assert srv.info()["high_water_bytes"] <= budget
        assert base - free() <= slack
    finally:
        c.close()
