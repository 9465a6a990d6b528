"""Device inputs that the caller's stream is still writing, and outputs it is
still reading, when a call starts: the library works on its own stream and
waits for the caller's first, for torch's default stream (a null handle) as
for any other.  Every result equals the one from finished inputs bitwise."""
import contextlib

import pytest

import synth
from gpu_common import lattice, log

pytestmark = pytest.mark.gpu

DIMS = (16, 8, 8, 8)


@pytest.mark.parametrize("own_stream", [False, True])
def test_calls_wait_for_the_callers_stream(own_stream):
    import torch
    log(f"test_calls_wait_for_the_callers_stream own_stream={own_stream}")
    n = 2
    U = [torch.from_numpy(synth.gauge_su3(DIMS, 0.3, s)).cuda() for s in (81, 82)]
    x = torch.from_numpy(synth.random_spinor(DIMS, 83, nrhs=n).reshape(n, -1)).cuda()
    m = torch.randn(4096, 4096, device="cuda")
    alpha = synth.alpha_exp(DIMS[0], 0.2)

    def late(dst, src):
        """dst = src on the current stream, behind tens of milliseconds of work."""
        dst.zero_()
        for _ in range(40):
            torch.mm(m, m)
        dst.copy_(src)
        ev = torch.cuda.Event()
        ev.record()
        return ev

    def calls(L, a, y):
        yield "apply", lambda: L.apply_dev(a, y, precond=True)
        yield "schur f32", lambda: L.apply_dev(a, y, precond=True, schur=True, precision="f32")
        yield "slots", lambda: L.apply_dev(a, y, precond=True, masses=[0.3, 0.6])
        yield "noalloc", lambda: L.apply_dev_noalloc(a, y, precond=True)
        yield "solve", lambda: L.solve_dev(a, y, r=1e-9, precision="f32")
        yield "sap", lambda: L.solve_sap_dev(a[0], y[0], block=(4, 4, 4, 4), r=1e-9)

    stream = torch.cuda.Stream() if own_stream else None
    torch.cuda.synchronize()
    with contextlib.ExitStack() as st:
        if stream:
            st.enter_context(torch.cuda.stream(stream))
        # links: the second configuration of a context that has only applied the operator
        y, ref = torch.zeros_like(x), torch.zeros_like(x)
        L, F = st.enter_context(lattice(DIMS)), st.enter_context(lattice(DIMS))
        L.set_gauge(U[0])
        F.set_gauge(U[1])
        for c in (L, F):
            c.set_clover(1.6)
            c.set_mass(0.5)
            c.set_alpha(alpha)
            c.apply_dev(x, ref, precond=True, schur=True)
        buf = torch.zeros_like(U[0])
        torch.cuda.synchronize()
        ev = late(buf, U[1])
        assert not ev.query()  # the links are not there yet
        L.set_gauge(buf)
        assert ev.query()
        L.set_clover(1.6)
        L.apply_dev(x, y, precond=True, schur=True)
        assert torch.equal(y, ref)
        # spinors
        a = torch.zeros_like(x)
        for (name, late_call), (_, ref_call) in zip(calls(L, a, y), calls(F, x, ref)):
            y.zero_()
            ref.zero_()
            torch.cuda.synchronize()
            ref_call()
            ev = late(a, x)
            assert not ev.query(), name
            late_call()
            assert torch.equal(y, ref), name
        # an output whose memory is still being read
        old, kept = torch.randn_like(x), torch.zeros_like(x)
        y.copy_(old)
        torch.cuda.synchronize()
        ev = late(kept, y)
        assert not ev.query()
        L.point_sources((0, 0, 0, 0), 0, n, out=y)
        torch.cuda.synchronize()
        assert torch.equal(kept, old)
