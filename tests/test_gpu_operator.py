"""GPU parity of the operator kernels against the FP64 oracle, element by element.

The alpha-hop kernel (hop term of D' with the modified time derivatives,
heavy-quark section), its clover epilogues, the Schur operator of the
even-odd reduction, the adjoint, and the FP32 / FP16-storage variants.
Lattices span several 256-site tiles and end in a ragged tail.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import lattice, log, max_rel, oracle_hop, oracle_schur, parity_mask

pytestmark = pytest.mark.gpu

DIMS = [(8, 4, 4, 4), (6, 4, 6, 4), (4, 6, 2, 8)]  # Vh = 256, 288 (ragged), 192


def setup_field(dims, seed, csw=1.6, eps=0.6):
    U = synth.gauge_su3(dims, eps, seed)
    rng = np.random.default_rng(seed)
    alpha = np.exp(rng.uniform(-1.0, 1.0, dims[0]))
    return U, oracle.clover(U, csw), alpha


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("bc_t", [-1, 1, 0])
def test_hop_only(dims, bc_t):
    log(f"test_hop_only dims={dims} bc_t={bc_t}")
    U, _, alpha = setup_field(dims, 100 + dims[1])
    psi = synth.random_spinor(dims, 7)
    with lattice(dims, bc_t) as L:
        L.set_gauge(U)
        L.set_mass(0.3)
        L.set_alpha(alpha)
        for precond in (False, True):
            for dagger in (False, True):
                got = L.apply(psi, precond=precond, dagger=dagger, hop_only=True)
                a = alpha if precond else None
                if dagger:
                    full = oracle.apply(U, None, 0.3, psi, alpha=a, bc_t=bc_t, dagger=True)
                    ref = full - 4.3 * psi
                else:
                    ref = oracle_hop(oracle, U, None, 0.3, psi, a, bc_t)
                assert max_rel(got, ref) < 1e-13, (precond, dagger)


@pytest.mark.parametrize("dims", DIMS)
def test_full_operator_with_clover(dims):
    log(f"test_full_operator_with_clover dims={dims}")
    U, C, alpha = setup_field(dims, 200 + dims[2])
    psi = synth.random_spinor(dims, 8)
    with lattice(dims) as L:
        L.set_gauge(U)
        L.set_clover(1.6)
        L.set_mass(0.5)
        L.set_alpha(alpha)
        for precond in (False, True):
            for dagger in (False, True):
                got = L.apply(psi, precond=precond, dagger=dagger)
                ref = oracle.apply(U, C, 0.5, psi, alpha=alpha if precond else None, dagger=dagger)
                assert max_rel(got, ref) < 1e-13, (precond, dagger)


def test_clover_field_input_and_rejection():
    dims = (4, 4, 4, 4)
    log("test_clover_field_input_and_rejection")
    U, C, alpha = setup_field(dims, 5)
    psi = synth.random_spinor(dims, 9)
    with lattice(dims) as L:
        L.set_gauge(U)
        L.set_clover_field(C)
        L.set_mass(0.2)
        L.set_alpha(alpha)
        got = L.apply(psi, precond=True)
        assert max_rel(got, oracle.apply(U, C, 0.2, psi, alpha=alpha)) < 1e-13
        bad = C.copy()
        bad[..., 0, 7] += 0.5  # mixes the chiralities
        import paper_1006_4028_amd as dp
        with pytest.raises(dp.DPError):
            L.set_clover_field(bad)


@pytest.mark.parametrize("dims", DIMS[:2])
def test_schur_operator(dims):
    log(f"test_schur_operator dims={dims}")
    U, C, alpha = setup_field(dims, 300 + dims[0])
    psi = synth.random_spinor(dims, 10)
    with lattice(dims) as L:
        L.set_gauge(U)
        L.set_clover(1.6)
        L.set_mass(0.05)
        L.set_alpha(alpha)
        got = L.apply(psi, precond=True, schur=True)
        ref = oracle_schur(oracle, U, C, 0.05, psi, alpha)
        assert max_rel(got, ref) < 1e-12
        got_dag = L.apply(psi, precond=True, schur=True, dagger=True)
        assert max_rel(got_dag, oracle_schur(oracle, U, C, 0.05, psi, alpha, dagger=True)) < 1e-12
        # adjoint: <phi, Mhat psi> = <Mhat^+ phi, psi> on the even sites
        phi = synth.random_spinor(dims, 11)
        got_d = L.apply(phi, precond=True, schur=True, dagger=True)
        even = (parity_mask(dims) == 0)[..., None, None]
        lhs = np.vdot(phi * even, ref)
        rhs = np.vdot(got_d, psi * even)
        assert abs(lhs - rhs) < 1e-11 * abs(lhs)


@pytest.mark.parametrize("precision,tol", [("f32", 2e-6), ("f16", 3e-3)])
def test_inner_precision_kernels(precision, tol):
    dims = (8, 4, 6, 4)
    log(f"test_inner_precision_kernels {precision}")
    U, C, _ = setup_field(dims, 400)
    alpha = synth.alpha_exp(dims[0], 0.4)
    psi = synth.random_spinor(dims, 12)
    with lattice(dims) as L:
        L.set_gauge(U)
        L.set_clover(1.6)
        L.set_mass(0.5)
        L.set_alpha(alpha)
        for schur in (False, True):
            for dagger in (False, True):
                got = L.apply(psi, precond=True, schur=schur, dagger=dagger, precision=precision)
                if schur:
                    ref = oracle_schur(oracle, U, C, 0.5, psi, alpha, dagger=dagger)
                else:
                    ref = oracle.apply(U, C, 0.5, psi, alpha=alpha, dagger=dagger)
                e = max_rel(got, ref)
                log(f"  {precision} schur={schur} dagger={dagger} max-element err {e:.2e}")
                assert e < tol


@pytest.mark.parametrize("precision,nrhs", [("f64", 5), ("f32", 5), ("f16", 5), ("f32", 13), ("f32", 2)])
def test_apply_dev_multi_rhs_matches_per_column(precision, nrhs):
    """dp_apply_dev runs the multi-RHS kernels (every right-hand side a slot);
    each column must equal the one-slot dp_apply of that column bitwise (the
    slot arithmetic does not depend on the batch), for the full operator, the
    Schur operator and their adjoints; the per-launch timing samples match
    the launch counts.  13 FP32 columns take two passes of the shared-tile
    workgroup (7 waves, the last one idle in the second pass).  The lattice
    has 1536 sites per timeslice and parity: 24 chunks of 64 sites, three in
    every XCD's slab, so the chunk boundaries, the slab boundaries and the
    neighbours across them are all exercised."""
    import torch
    dims = (4, 16, 12, 16)
    log(f"test_apply_dev_multi_rhs_matches_per_column {precision} nrhs={nrhs}")
    U, _, alpha = setup_field(dims, 31)
    psi = synth.random_spinor(dims, 8, nrhs=nrhs)
    with lattice(dims) as L:
        L.set_gauge(U)
        L.set_clover(1.6)
        L.set_mass(0.2)
        L.set_alpha(alpha)
        in_t = torch.from_numpy(psi.reshape(nrhs, -1)).cuda()
        out_t = torch.empty_like(in_t)
        for schur in (False, True):
            for dagger in (False, True):
                L.set_timing(True)
                L.apply_dev(in_t, out_t, precond=True, dagger=dagger, schur=schur, precision=precision)
                stats = L.timing()
                for name, st in stats.items():
                    assert len(L.timing_samples(name)) == st["launches"]
                L.set_timing(False)
                got = out_t.cpu().numpy().reshape(psi.shape)
                for k in range(nrhs):
                    ref = L.apply(psi[k], precond=True, dagger=dagger, schur=schur, precision=precision)
                    assert np.array_equal(got[k], ref), (schur, dagger, k)
        with pytest.raises(Exception):
            L.apply_dev(in_t, in_t, precond=True)


@pytest.mark.parametrize("dims", DIMS)
def test_light_quark_factorisation_operator(dims):
    """beta(y) = prod_mu a_mu(y_mu) (eqs. redefa, betaa, redefcovs): the full
    operator, the Schur operator and their adjoints against the oracle's
    literal beta (D+M) beta^-1, in FP64, FP32 and FP16 storage; with the
    preconditioning flag off the spatial profiles must not act."""
    log(f"test_light_quark_factorisation_operator dims={dims}")
    U, C, _ = setup_field(dims, 500 + dims[2])
    rng = np.random.default_rng(dims[1])
    beta = tuple(np.exp(rng.uniform(-0.7, 0.7, L)) for L in dims)
    psi = synth.random_spinor(dims, 13)
    with lattice(dims) as L:
        L.set_gauge(U)
        L.set_clover(1.6)
        L.set_mass(0.25)
        L.set_beta(beta)
        for dagger in (False, True):
            ref = oracle.apply_beta(U, C, 0.25, psi, beta, dagger=dagger)
            assert max_rel(L.apply(psi, precond=True, dagger=dagger), ref) < 1e-12
            refs = oracle_schur(oracle, U, C, 0.25, psi, beta, dagger=dagger)
            assert max_rel(L.apply(psi, precond=True, schur=True, dagger=dagger), refs) < 1e-12
            for precision, tol in (("f32", 2e-6), ("f16", 3e-3)):
                e = max_rel(L.apply(psi, precond=True, schur=True, dagger=dagger, precision=precision), refs)
                log(f"  {precision} schur dagger={dagger} max-element err {e:.2e}")
                assert e < tol
        plain = oracle.apply(U, C, 0.25, psi)
        assert max_rel(L.apply(psi, precond=False), plain) < 1e-12


@pytest.mark.parametrize("precision,tol", [("f64", 1e-12), ("f32", 2e-6), ("f16", 3e-3)])
def test_dirichlet_time_boundary_operator(precision, tol):
    """The Dirichlet time boundary (bc_t = 0): full and Schur operators and
    their adjoints against the oracle, every storage precision."""
    dims = (8, 4, 6, 4)
    log(f"test_dirichlet_time_boundary_operator {precision}")
    U, C, alpha = setup_field(dims, 600)
    psi = synth.random_spinor(dims, 14)
    with lattice(dims, bc_t=0) as L:
        L.set_gauge(U)
        L.set_clover(1.6)
        L.set_mass(0.3)
        L.set_alpha(alpha)
        for dagger in (False, True):
            ref = oracle.apply(U, C, 0.3, psi, alpha=alpha, bc_t=0, dagger=dagger)
            assert max_rel(L.apply(psi, precond=True, dagger=dagger, precision=precision), ref) < tol
            refs = oracle_schur(oracle, U, C, 0.3, psi, alpha, bc_t=0, dagger=dagger)
            assert max_rel(L.apply(psi, precond=True, schur=True, dagger=dagger, precision=precision), refs) < tol


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 2, 6, 2), (2, 34, 2, 6), (6, 10, 14, 6)])
@pytest.mark.parametrize("nrhs", [1, 2, 5])
def test_operator_extents(dims, nrhs):
    """The kernels' site arithmetic at the edges of its range: extents of 2
    (half rows of one site, both neighbours the same site), rows that do not
    divide a 64-site chunk, partial chunks; full operator and Schur operator
    in FP64 with one slot and with several, against the oracle."""
    import torch
    log(f"test_operator_extents dims={dims} nrhs={nrhs}")
    U, C, alpha = setup_field(dims, 700 + dims[1])
    psi = synth.random_spinor(dims, 15, nrhs=nrhs)
    with lattice(dims) as L:
        L.set_gauge(U)
        L.set_clover(1.6)
        L.set_mass(0.2)
        L.set_alpha(alpha)
        in_t = torch.from_numpy(psi.reshape(nrhs, -1)).cuda()
        out_t = torch.empty_like(in_t)
        torch.cuda.synchronize()
        for schur, tol in ((False, 1e-13), (True, 1e-12)):
            L.apply_dev(in_t, out_t, precond=True, schur=schur)
            got = out_t.cpu().numpy().reshape(psi.shape)
            for k in range(nrhs):
                ref = (oracle_schur(oracle, U, C, 0.2, psi[k], alpha) if schur
                       else oracle.apply(U, C, 0.2, psi[k], alpha=alpha))
                assert max_rel(got[k], ref) < tol, (schur, k)


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 4, 6, 4)])
def test_schur_inverse_pivots(dims):
    """The per-mass inverse of blocks whose diagonal vanishes (C cancels 4 + M
    there), so that every elimination step needs a row exchange, on fewer and
    on more sites than a wave's 32; FP64 Schur operator against a LAPACK solve
    per site.  Bound: the condition numbers of the random 6x6 blocks stay
    below 1e5, and 1e5 times the FP64 epsilon is 2e-11."""
    log(f"test_schur_inverse_pivots dims={dims}")
    rng = np.random.default_rng(dims[2])
    U = synth.gauge_su3(dims, 0.4, 3)
    A = rng.standard_normal(dims + (12, 12)) + 1j * rng.standard_normal(dims + (12, 12))
    A = A + np.conj(np.swapaxes(A, -1, -2))
    A[..., :6, 6:] = A[..., 6:, :6] = 0.0
    A[..., range(12), range(12)] = 0.0
    assert np.linalg.cond(A).max() < 1e5
    M = 0.25
    C = A - (4.0 + M) * np.eye(12)
    alpha = synth.alpha_exp(dims[0], 0.2)
    psi = synth.random_spinor(dims, 16)
    with lattice(dims) as L:
        L.set_gauge(U)
        L.set_clover_field(C)
        L.set_mass(M)
        L.set_alpha(alpha)
        e = max_rel(L.apply(psi, precond=True, schur=True), oracle_schur(oracle, U, C, M, psi, alpha))
        log(f"  max-element err {e:.2e}")
        assert e < 2e-11


@pytest.mark.parametrize("precision,nrhs", [("f64", 3), ("f64", 9), ("f64", 13), ("f32", 9), ("f16", 9)])
def test_shared_tile_matches_one_wave(precision, nrhs):
    """A batch above the size up to which every slot has a wave of its own (512
    waves a slot) runs the kernels that share a tile's links between the slots,
    in FP64 without the blocks of the epilogue (3), with the clover blocks (9)
    and with both kinds (13): bitwise the one-slot results, full operator (both
    parities in one launch) and Schur operator, with their adjoints."""
    import torch
    dims = (16, 16, 16, 16)
    log(f"test_shared_tile_matches_one_wave {precision} nrhs={nrhs}")
    U = synth.gauge_su3(dims, 0.3, 32)
    psi = synth.random_spinor(dims, 16, nrhs=nrhs)
    with lattice(dims) as L:
        L.set_gauge(U)
        L.set_clover(1.6)
        L.set_mass(0.2)
        L.set_alpha(synth.alpha_exp(dims[0], 0.3))
        in_t = torch.from_numpy(psi.reshape(nrhs, -1)).cuda()
        out_t, one_t = torch.empty_like(in_t), torch.empty_like(in_t[:1])
        torch.cuda.synchronize()
        for schur in (False, True):
            for dagger in (False, True):
                L.apply_dev(in_t, out_t, precond=True, dagger=dagger, schur=schur, precision=precision)
                for k in (0, nrhs // 2, nrhs - 1):
                    L.apply_dev(in_t[k:k + 1], one_t, precond=True, dagger=dagger, schur=schur, precision=precision)
                    assert torch.equal(out_t[k], one_t[0]), (schur, dagger, k)


@pytest.mark.parametrize("nrhs", [1, 10])
def test_f32_hop_error(nrhs):
    """The FP32 hop against the FP64 one, one slot (a wave each) and ten (3360
    waves: the shared tile).  The relative error is the same to 0.2% on every
    lattice, field and source: 8.2e-8 where a link product's pairs are formed
    first and added with one rounding, 8.5e-8 where every product is added by
    itself.  The bound lies between."""
    import torch
    dims = (24, 12, 12, 12)
    log(f"test_f32_hop_error nrhs={nrhs}")
    x = torch.from_numpy(synth.random_spinor(dims, 19, nrhs=nrhs).reshape(nrhs, -1)).cuda()
    y, ref = torch.empty_like(x), torch.empty_like(x)
    with lattice(dims) as L:
        L.set_gauge(synth.gauge_su3(dims, 0.3, 34))
        L.set_mass(0.2)
        for dagger in (False, True):
            L.apply_dev(x, ref, hop_only=True, dagger=dagger)
            L.apply_dev(x, y, hop_only=True, dagger=dagger, precision="f32")
            e = float(((y - ref).norm() / ref.norm()).cpu())
            log(f"  dagger={dagger} relative error {e:.3e}")
            assert e < 8.35e-8, dagger


@pytest.mark.parametrize("nrhs", [1, 5])
def test_full_operator_counts_every_input_once(nrhs):
    """The algorithmic bytes and flops of the full operator's launch: 72 link
    and 72 clover reals a site once, 24 reals of every spinor in and out (FP16:
    a scale of 4 bytes a spinor and a clover site); 1320 flops of the hop, 552
    of the blocks and 48 of the sum."""
    import torch
    dims = (4, 4, 6, 4)
    V = int(np.prod(dims))
    log(f"test_full_operator_counts_every_input_once nrhs={nrhs}")
    x = torch.from_numpy(synth.random_spinor(dims, 20, nrhs=nrhs).reshape(nrhs, -1)).cuda()
    y = torch.empty_like(x)
    with lattice(dims) as L:
        L.set_gauge(synth.gauge_su3(dims, 0.3, 35))
        L.set_clover(1.6)
        L.set_mass(0.2)
        for precision, b, sc in (("f64", 8, 0), ("f32", 4, 0), ("f16", 2, 4)):
            L.set_timing(True)
            L.apply_dev(x, y, precision=precision)
            st = L.timing()[f"hop_{precision}_full"]
            L.set_timing(False)
            assert st["launches"] == 1
            assert st["bytes"] == V * ((72 + 72) * b + sc + nrhs * 2 * (24 * b + sc)), precision
            assert st["flops"] == V * nrhs * (1320 + 552 + 48), precision


@pytest.mark.parametrize("precision,nrhs", [("f64", 3), ("f64", 5), ("f64", 13), ("f32", 3), ("f32", 13),
                                            ("f16", 3), ("f16", 13)])
def test_shared_tile_partial_chunk(precision, nrhs):
    """The kernels that share a tile between the slots on a timeslice that does
    not fill its last chunk (2520 sites of a parity: 24 in the last of 40; 1440
    waves a slot, so three slots are enough), the slots in even and uneven
    rounds of the workgroup's waves (13 over 4 or 5), with a profile in every
    direction: bitwise the one-slot results, full, Schur and hop-only
    operator with their adjoints; nothing is written outside the output."""
    import torch
    dims = (36, 18, 20, 14)
    log(f"test_shared_tile_partial_chunk {precision} nrhs={nrhs}")
    U = synth.gauge_su3(dims, 0.3, 36)
    n, guard = 12 * int(np.prod(dims)), 4096
    x = torch.from_numpy(synth.random_spinor(dims, 21, nrhs=nrhs).reshape(nrhs, -1)).cuda()
    buf = torch.empty(nrhs * n + 2 * guard, dtype=torch.complex128, device="cuda")
    out, one = buf[guard:-guard].view(nrhs, n), torch.empty_like(x[:1])
    with lattice(dims) as L:
        L.set_gauge(U)
        L.set_clover(1.6)
        L.set_mass(0.2)
        L.set_beta(synth.beta_cosh_paper(dims, 0.1))
        for kw in (dict(), dict(schur=True), dict(hop_only=True)):
            for dagger in (False, True):
                buf.fill_(7.0)
                L.apply_dev(x, out, precond=True, dagger=dagger, precision=precision, **kw)
                assert bool((buf[:guard] == 7.0).all()) and bool((buf[-guard:] == 7.0).all()), (kw, dagger)
                for k in range(nrhs):
                    L.apply_dev(x[k:k + 1], one, precond=True, dagger=dagger, precision=precision, **kw)
                    assert torch.equal(out[k], one[0]), (kw, dagger, k)


@pytest.mark.parametrize("dims,nrhs", [((10, 10, 10, 10), 8), ((10, 10, 10, 10), 13), ((10, 10, 10, 10), 26),
                                       ((36, 14, 14, 12), 2), ((60, 14, 14, 12), 2)])
def test_f64_two_waves_per_simd(dims, nrhs):
    """FP64 slots as waves of their own, two a SIMD: launches of more than 1024
    waves with 80 (timeslice, chunk) tiles at any slot count (10^4: 52 sites in
    the last chunk of 8; 13 slots of one parity, 8 of both), and with more tiles
    (684: two slots; 1140: one slot, and two slots that share a tile).  Bitwise
    the one-slot results, full, Schur and hop-only operator with their
    adjoints; nothing is written outside the output."""
    import torch
    log(f"test_f64_two_waves_per_simd {dims} nrhs={nrhs}")
    U = synth.gauge_su3(dims, 0.3, 37)
    n, guard = 12 * int(np.prod(dims)), 4096
    x = torch.from_numpy(synth.random_spinor(dims, 22, nrhs=nrhs).reshape(nrhs, -1)).cuda()
    buf = torch.empty(nrhs * n + 2 * guard, dtype=torch.complex128, device="cuda")
    out, one = buf[guard:-guard].view(nrhs, n), torch.empty_like(x[:1])
    with lattice(dims) as L:
        L.set_gauge(U)
        L.set_clover(1.6)
        L.set_mass(0.2)
        L.set_beta(synth.beta_cosh_paper(dims, 0.1))
        for kw in (dict(), dict(schur=True), dict(hop_only=True)):
            for dagger in (False, True):
                buf.fill_(7.0)
                L.apply_dev(x, out, precond=True, dagger=dagger, **kw)
                assert bool((buf[:guard] == 7.0).all()) and bool((buf[-guard:] == 7.0).all()), (kw, dagger)
                for k in range(nrhs):
                    L.apply_dev(x[k:k + 1], one, precond=True, dagger=dagger, **kw)
                    assert torch.equal(out[k], one[0]), (kw, dagger, k)


@pytest.mark.parametrize("dims,nrhs,dims0,nrhs0", [((2, 16, 16, 16), 24, (2, 16, 16, 16), 16),
                                                   ((10, 10, 10, 10), 16, (10, 10, 10, 10), 12),
                                                   ((18, 16, 16, 16), 2, (16, 16, 16, 16), 2),
                                                   ((36, 16, 16, 16), 1, (32, 16, 16, 16), 1)])
def test_f64_operator_time_follows_the_work(dims, nrhs, dims0, nrhs0):
    """Just beyond the 1024 waves that run at once, one a SIMD, the FP64 Schur
    operator takes no step in time: it grows by at most 10% more than the work
    (13 to 50% here), where one wave a SIMD or a few shared tiles took 17 to 68%
    more."""
    import torch
    log(f"test_f64_operator_time_follows_the_work {dims} x {nrhs} against {dims0} x {nrhs0}")

    def us(d, n):
        x = torch.from_numpy(synth.random_spinor(d, 23).reshape(1, -1)).cuda().repeat(n, 1)
        y = torch.empty_like(x)
        best = np.inf
        with lattice(d) as L:
            L.set_gauge(synth.gauge_su3(d, 0.3, 38))
            L.set_mass(0.5)
            for _ in range(4):
                L.set_timing(True)
                for _ in range(40):
                    L.apply_dev(x, y, precond=True, schur=True)
                best = min(best, sum(np.median(L.timing_samples(f"hop_f64_{q}")) for q in ("inv", "diag")))
                L.set_timing(False)
        return 1e3 * best

    t, t0 = us(dims, nrhs), us(dims0, nrhs0)
    work = np.prod(dims) * nrhs / (np.prod(dims0) * nrhs0)
    log(f"  {t0:.1f} -> {t:.1f} us, work x {work:.3f}, time x {t / t0:.3f}")
    assert t / t0 <= 1.1 * work
