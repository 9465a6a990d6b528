"""Continuous batching on the GPU: right-hand sides with different masses,
profiles and source timeslices enter and leave a running batch; every result
equals the same right-hand side solved alone (bit for bit) and satisfies the
stopping rule when its residual is recomputed by the oracle."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import lattice, log

pytestmark = pytest.mark.gpu

DIMS = (8, 4, 4, 6)


def solo(L, eta, M, alpha, x0, r, precision):
    L.set_mass(M)
    L.set_alpha(alpha)
    S, cpp, info = L.solve(eta, r=r, precision=precision, x0_src=x0)
    return S[0], cpp[0], info[0]


@pytest.mark.parametrize("precision", ["f64", "f32", "f16"])
def test_batch_join_and_leave_matches_solo(precision):
    import torch
    import paper_1006_4028_amd as dp
    from paper_1006_4028_amd.serve import point_columns, profile
    log(f"test_batch_join_and_leave_matches_solo {precision}")
    U = synth.gauge_su3(DIMS, 0.4, 17)
    C = oracle.clover(U, 1.6)
    r = 1e-10
    reqs = [dict(M=0.5, a0=0.4, x0=0, cols=3), dict(M=0.05, a0=0.0, x0=3, cols=2), dict(M=0.2, a0=0.1, x0=6, cols=1)]
    with lattice(DIMS) as L:
        L.set_gauge(U)
        L.set_clover(1.6)
        got = {}
        with dp.Batch(L, 5, precision) as B:
            def admit(k):
                q = reqs[k]
                eta = point_columns(DIMS, q["x0"], q["cols"])
                S_t = torch.zeros(q["cols"], eta[0].size, dtype=torch.complex128, device="cuda")
                slots = B.admit(torch.from_numpy(eta.reshape(q["cols"], -1)).cuda(), S_t, M=q["M"],
                                alpha=profile(DIMS[0], q["a0"], q["x0"]), r=r, x0_src=q["x0"], tag=k)
                q["S_t"] = S_t
                q["slots"] = slots
                return slots
            assert admit(0) is not None and admit(1) is not None
            assert admit(2) is None  # only 5 slots: the third request waits
            B.step(2)
            B.step(2)
            for res in B.harvest():
                got.setdefault(res["tag"], []).append(res)
            while B.status()["free"] < 1:
                B.step(2)
                for res in B.harvest():
                    got.setdefault(res["tag"], []).append(res)
            assert admit(2) is not None  # joins the running batch
            while B.status()["running"] or B.status()["done"]:
                B.step(3)
                for res in B.harvest():
                    got.setdefault(res["tag"], []).append(res)
        for k, q in enumerate(reqs):
            assert len(got[k]) == q["cols"]
            alpha = profile(DIMS[0], q["a0"], q["x0"])
            S_b = q["S_t"].cpu().numpy().reshape((q["cols"],) + DIMS + (4, 3))
            eta = point_columns(DIMS, q["x0"], q["cols"])
            cpp_b = {q["slots"].index(res["slot"]): res["cpp"] for res in got[k]}
            # solo solves of the same columns on a fresh context
            with lattice(DIMS) as L2:
                L2.set_gauge(U)
                L2.set_clover(1.6)
                for c in range(q["cols"]):
                    S1, cpp1, info1 = solo(L2, eta[c], q["M"], alpha, q["x0"], r, precision)
                    assert np.array_equal(S1, S_b[c]), (k, c)
                    assert np.array_equal(cpp1, cpp_b[c]), (k, c)
                    # stopping rule recomputed by the oracle
                    a6 = alpha[:, None, None, None, None, None]
                    res = a6 * eta[c] - oracle.apply(U, C, q["M"], a6 * S_b[c], alpha=alpha)
                    assert np.linalg.norm(res) <= 1.0001 * r * np.linalg.norm(a6 * eta[c])
            log(f"  request {k}: iters {[res['info']['iters'] for res in got[k]]}")


def test_server_poisson_stream_and_memory_gate():
    from paper_1006_4028_amd.serve import Server, poisson_requests, summarize, point_columns, profile
    log("test_server_poisson_stream_and_memory_gate")
    fields = {"a": ((8, 4, 4, 4), synth.gauge_su3((8, 4, 4, 4), 0.3, 1), 1.6),
              "b": ((6, 4, 4, 6), synth.gauge_su3((6, 4, 4, 6), 0.3, 2), 1.6)}
    reqs = poisson_requests(24, rate=400.0, fields=fields, T_of={"a": 8, "b": 6}, seed=3, max_cols=5)
    srv = Server(fields, nslots=8, precision="f32", r=1e-10)
    try:
        out = srv.run(reqs)
        s = summarize(srv, out)
    finally:
        srv.close()
    log("  ", s)
    assert s["done"] == 24 and s["failed"] == 0 and s["rejected"] == 0
    # every request equals the solo solve of its columns
    for q in out[:6]:
        dims, U, csw = fields[q.field]
        with lattice(dims) as L:
            L.set_gauge(U)
            L.set_clover(csw)
            L.set_mass(q.M)
            L.set_alpha(profile(dims[0], q.alpha0, q.x0))
            _, cpp, _ = L.solve(point_columns(dims, q.x0, q.ncols), r=1e-10, precision="f32", x0_src=q.x0,
                                ncols_group=q.ncols)
        assert np.allclose(q.cpp, cpp[0], rtol=1e-12, atol=0), q.rid
    # a budget that holds the fields and workspaces but only one inverse clover
    # per field rejects requests that need a second mass on the same field
    from paper_1006_4028_amd import footprint_bytes
    base = sum(footprint_bytes(d, 8, "f32", 0) for d, _, _ in fields.values())
    one = max(footprint_bytes(d, 0, "f32", 1) - footprint_bytes(d, 0, "f32", 0) for d, _, _ in fields.values())
    srv = Server(fields, nslots=8, precision="f32", r=1e-10, hbm_budget=base + 2 * one)
    try:
        out = srv.run(poisson_requests(16, rate=400.0, fields=fields, T_of={"a": 8, "b": 6}, seed=4, max_cols=3))
        s = summarize(srv, out)
    finally:
        srv.close()
    log("  gated:", s)
    assert s["rejected"] > 0 and s["done"] + s["rejected"] == 16


def test_batch_mass_change_after_shared_inverse():
    """A batch whose slots all hold one mass stages that mass's A_oo^-1 once
    per workgroup (FP32 multi-slot kernels), and its captured iteration graph
    bakes that in; requests of another mass admitted later must get their own
    inverse (the graph is captured again).  Every column equals its solo
    solve bit for bit."""
    import torch
    import paper_1006_4028_amd as dp
    from paper_1006_4028_amd.serve import point_columns, profile
    log("test_batch_mass_change_after_shared_inverse")
    U = synth.gauge_su3(DIMS, 0.4, 23)
    r = 1e-10
    reqs = [dict(M=0.5, a0=0.4, x0=0, cols=4), dict(M=0.05, a0=0.1, x0=2, cols=2),
            dict(M=0.5, a0=0.0, x0=5, cols=2)]
    with lattice(DIMS) as L:
        L.set_gauge(U)
        L.set_clover(1.6)
        got = {}
        with dp.Batch(L, 4, "f32") as B:
            def admit(k):
                q = reqs[k]
                eta = point_columns(DIMS, q["x0"], q["cols"])
                S_t = torch.zeros(q["cols"], eta[0].size, dtype=torch.complex128, device="cuda")
                slots = B.admit(torch.from_numpy(eta.reshape(q["cols"], -1)).cuda(), S_t, M=q["M"],
                                alpha=profile(DIMS[0], q["a0"], q["x0"]), r=r, x0_src=q["x0"], tag=k)
                q["S_t"] = S_t
                return slots

            def drain(until_free):
                while B.status()["free"] < until_free:
                    B.step(2)
                    for res in B.harvest():
                        got.setdefault(res["tag"], []).append(res)

            assert admit(0) is not None  # every slot at M = 0.5: shared inverse
            drain(4)
            assert admit(1) is not None  # M = 0.05 next to stale M = 0.5 slots
            assert admit(2) is not None  # and M = 0.5 again beside it
            drain(4)
        for k, q in enumerate(reqs):
            assert len(got[k]) == q["cols"]
            alpha = profile(DIMS[0], q["a0"], q["x0"])
            S_b = q["S_t"].cpu().numpy().reshape((q["cols"],) + DIMS + (4, 3))
            eta = point_columns(DIMS, q["x0"], q["cols"])
            with lattice(DIMS) as L2:
                L2.set_gauge(U)
                L2.set_clover(1.6)
                for c in range(q["cols"]):
                    S1, _, _ = solo(L2, eta[c], q["M"], alpha, q["x0"], r, "f32")
                    assert np.array_equal(S1, S_b[c]), (k, c)
            log(f"  request {k}: iters {[res['info']['iters'] for res in got[k]]}")


def test_new_configurations_on_one_context():
    """Links, clover and masses replaced on one context (more masses than the
    context keeps buffers for): every Schur application equals a fresh
    context's bitwise, so nothing of an earlier configuration's inverses is
    read again."""
    import torch
    dims = (4, 4, 6, 4)
    log("test_new_configurations_on_one_context")
    alpha = synth.alpha_exp(dims[0], 0.2)
    psi = torch.from_numpy(synth.random_spinor(dims, 17, nrhs=2).reshape(2, -1)).cuda()
    out, ref = torch.empty_like(psi), torch.empty_like(psi)
    torch.cuda.synchronize()
    masses = [0.05, 0.1, 0.2, 0.3, 0.4, 0.5]
    with lattice(dims) as L:
        L.set_alpha(alpha)
        for seed, csw in ((1, 1.6), (2, 1.2), (3, 0.0)):
            U = synth.gauge_su3(dims, 0.4, seed)
            L.set_gauge(U)
            L.set_clover(csw)
            for M in masses[: 7 - 2 * seed]:
                L.set_mass(M)
                L.apply_dev(psi, out, precond=True, schur=True, precision="f16" if M > 0.25 else "f32")
                with lattice(dims) as F:
                    F.set_gauge(U)
                    F.set_clover(csw)
                    F.set_mass(M)
                    F.set_alpha(alpha)
                    F.apply_dev(psi, ref, precond=True, schur=True, precision="f16" if M > 0.25 else "f32")
                assert torch.equal(out, ref), (seed, M)


def test_dropped_inverses_held_memory_is_bounded():
    """What a context holds of dropped inverses: at most 1 GiB, nothing that a
    whole configuration left unused, nothing once it is closed (530 MB an
    inverse here; 64 MB are allowed for what the allocator rounds up)."""
    import torch
    dims = (32, 32, 32, 32)
    log("test_dropped_inverses_held_memory_is_bounded")
    slack = 64 << 20
    one = dims[0] * dims[1] * dims[2] * dims[3] // 2 * 1012

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    x = torch.zeros((1, 12 * 32 ** 4), dtype=torch.complex128, device="cuda")
    y = torch.empty_like(x)
    with lattice((4, 4, 4, 4)):  # the library's static scratch is on the device from here on
        before = free()
    with lattice(dims) as L:
        def configuration(masses):
            L.set_clover(0.0)
            for M in masses:
                L.set_mass(M)
                L.apply_dev(x, y, precision="f32")
            return free()

        work = configuration([0.1]) + one  # free beside the workspace and no inverse
        assert configuration([0.1, 0.2, 0.3, 0.4]) <= work - 4 * one + slack
        L.set_clover(0.0)  # drops the four
        held = work - free()
        log(f"  held after the drop: {held / 2 ** 20:.0f} MiB")
        assert held <= (1 << 30) + slack
        assert configuration([0.5]) >= work - 2 * one - slack  # a kept one taken up, none allocated
        L.set_clover(0.0)  # what the last configuration left over goes back too
        held = work - free()
        log(f"  held after a configuration of one mass: {held / 2 ** 20:.0f} MiB")
        assert held <= one + slack
    assert free() >= before - slack


@pytest.mark.parametrize("precision,nslots", [("f32", 8), ("f64", 13)])
def test_batch_mass_change_shared_tile(precision, nslots):
    """Slots that all hold one mass, then two masses, then one again, at 512
    waves a slot (16^4), where the odd-site kernels read the common A_oo^-1 from
    LDS (FP32 from 2 slots, FP64 from 12) and the captured iterations hold its
    address: every column equals its solo solve bit for bit."""
    import torch
    import paper_1006_4028_amd as dp
    from paper_1006_4028_amd.serve import point_columns, profile
    dims, r = (16, 16, 16, 16), 1e-9
    log(f"test_batch_mass_change_shared_tile {precision} nslots={nslots}")
    U = synth.gauge_su3(dims, 0.3, 24)
    # (mass, columns) of the requests of each wave of admissions
    waves = [[(0.5, nslots)], [(0.2, nslots - 3), (0.5, 3)], [(0.2, nslots)]]
    with lattice(dims) as L, lattice(dims) as L2:
        for c in (L, L2):
            c.set_gauge(U)
            c.set_clover(1.6)
        with dp.Batch(L, nslots, precision) as B:
            for w, reqs in enumerate(waves):
                done = []
                for k, (M, cols) in enumerate(reqs):
                    x0 = (2 * w + 3 * k) % dims[0]
                    eta = torch.from_numpy(np.concatenate([point_columns(dims, (x0 + 12 * j) % dims[0], 12)
                                                           for j in range(2)])[:cols].reshape(cols, -1)).cuda()
                    S = torch.zeros_like(eta)
                    alpha = profile(dims[0], 0.1, x0)
                    assert B.admit(eta, S, M=M, alpha=alpha, r=r, x0_src=x0, tag=10 * w + k) is not None
                    done.append((M, x0, eta, S, alpha))
                while B.status()["free"] < nslots:
                    B.step(3)
                    B.harvest()
                for M, x0, eta, S, alpha in done:
                    L2.set_mass(M)
                    L2.set_alpha(alpha)
                    one = torch.empty_like(eta[0])
                    for c in range(eta.shape[0]):
                        L2.solve_dev(eta[c], one, r=r, precision=precision, x0_src=x0)
                        assert torch.equal(S[c], one), (w, M, c)


@pytest.mark.parametrize("precision,solver,ncols", [("f64", "bicgstab", 3), ("f64", "bicgstab", 13),
                                                    ("f32", "bicgstab", 5), ("f16", "bicgstab", 3), ("f32", "cgnr", 3)])
def test_solve_columns_partial_chunk(precision, solver, ncols):
    """Fused dot products of the kernels that share a tile where a timeslice
    does not fill its last chunk: a solve of several columns at 36x18x20x14
    gives each the solution, C_PP and iteration count of its own solve."""
    import torch
    dims = (36, 18, 20, 14)
    log(f"test_solve_columns_partial_chunk {precision} {solver} ncols={ncols}")
    with lattice(dims) as L:
        L.set_gauge(synth.gauge_su3(dims, 0.3, 25))
        L.set_clover(1.6)
        L.set_mass(0.5)
        L.set_alpha(synth.alpha_exp_sym(dims[0], 0.05, 3))
        eta = torch.cat([L.point_sources((3, 1, 2, 3), 0, 12), L.point_sources((3, 4, 0, 1), 0, 1)])[:ncols].contiguous()
        S, one = torch.zeros_like(eta), torch.zeros_like(eta[0])
        cpp, info = L.solve_dev(eta, S, r=1e-9, solver=solver, precision=precision, x0_src=3)
        for k in range(ncols):
            cpp1, info1 = L.solve_dev(eta[k], one, r=1e-9, solver=solver, precision=precision, x0_src=3)
            assert info[k]["iters"] == info1[0]["iters"], k
            assert torch.equal(S[k], one) and np.array_equal(cpp[k], cpp1[0]), k


@pytest.mark.parametrize("solver", ["bicgstab", "cgnr"])
def test_solve_columns_two_waves_per_simd(solver):
    """Fused dot products where FP64 slots are waves of their own, two a SIMD (13
    columns at 10^4: 1040 waves): each column's solution, C_PP and iteration
    count are those of its own solve."""
    import torch
    dims = (10, 10, 10, 10)
    log(f"test_solve_columns_two_waves_per_simd {solver}")
    with lattice(dims) as L:
        L.set_gauge(synth.gauge_su3(dims, 0.3, 26))
        L.set_clover(1.6)
        L.set_mass(0.5)
        L.set_alpha(synth.alpha_exp_sym(dims[0], 0.05, 3))
        eta = torch.cat([L.point_sources((3, 1, 2, 3), 0, 12), L.point_sources((3, 4, 0, 1), 0, 1)]).contiguous()
        S, one = torch.zeros_like(eta), torch.zeros_like(eta[0])
        cpp, info = L.solve_dev(eta, S, r=1e-9, solver=solver, precision="f64", x0_src=3)
        for k in range(eta.shape[0]):
            cpp1, info1 = L.solve_dev(eta[k], one, r=1e-9, solver=solver, precision="f64", x0_src=3)
            assert info[k]["iters"] == info1[0]["iters"], k
            assert torch.equal(S[k], one) and np.array_equal(cpp[k], cpp1[0]), k
