"""Kernels that are chosen by size: GPU GMRES on fields around the size where its Gram-Schmidt step changes
kernels (131072 spectral slots), against the oracle's GMRES.

Sizes: fewer slots than one block of the small-field kernels holds (256), the
largest field they take, and the smallest above it.  A density ratio of 25 makes
the solves run past 24 basis vectors, so every split of the vectors between a
block's wavefronts is used.  Tolerances: both sides stop at a true relative
residual of 1e-10, so the solutions agree to 2e-10 times the condition number
of the preconditioned system, at most the density ratio; CGS with a measured
check and the oracle's MGS differ by rounding, so the iteration counts by at
most one."""
import numpy as np
import pytest

from tests.gpu_util import rel2, smooth_density, to_dev, to_host
from oracle import krylov, operators
from paper_2403_06654_amd import workloads

pytestmark = pytest.mark.gpu
RATIO = 25.0


@pytest.mark.parametrize("shape", [(16, 16), (16, 64), (64, 64, 64), (64, 64, 128)])
@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
def test_gmres_around_the_small_field_limit(shape, precision):
    from paper_2403_06654_amd.api import Grid
    rho = smooth_density(shape, 3, 1.0, RATIO)
    f = workloads.band_limited(shape, min(shape) // 4, seed=2)
    b, _ = operators.project_range(-f, operators.nullspace_basis(shape))
    ref = krylov.gmres(lambda x: operators.apply_pressure(x, rho), b,
                       lambda r: operators.precond_pressure(r, float(rho.mean())), restart=32, rtol=1e-10,
                       max_iter=500)
    g = Grid(shape)
    g.set_density(to_dev(rho))
    p, info = g.solve_pressure(to_dev(f), restart=32, precision=precision)
    p2, _ = g.solve_pressure(to_dev(f), restart=32, precision=precision)
    g.close()
    x = to_host(p)
    assert np.array_equal(x, to_host(p2))
    rr = np.linalg.norm(operators.apply_pressure(x, rho) - b) / np.linalg.norm(b)
    assert info["status"] == 0 and rr <= 1.01e-10
    assert rel2(x, ref["x"]) <= 2e-10 * RATIO
    if precision == "fp64":
        assert ref["iterations"] > 24
        assert abs(info["iterations"] - ref["iterations"]) <= 1


# Gram-Schmidt work inside the operator's passes: the shortest, the longest (512) and
# the first length (1024) that does not carry it, partial tiles, one to several blocks
@pytest.mark.parametrize("shape", [(16, 16), (512, 32), (1024, 32), (16, 16, 16), (128, 16, 32), (256, 64), (32, 64, 64)])
@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
def test_steps_carried_by_the_passes(shape, precision):
    """Restarted solves (the last step of a cycle finishes by itself), a budget
    that ends a cycle early and the first step alone, for the pressure passes
    (dots and check) and the Helmholtz passes (dots).  The oracle's operator
    gives a true residual of 1e-10 (1% for its own rounding); the FP64 counts
    differ from the oracle's by at most one step per cycle."""
    from paper_2403_06654_amd.api import Grid
    rho = smooth_density(shape, 5, 1.0, RATIO)
    f = workloads.band_limited(shape, min(shape) // 4, seed=4)
    b, _ = operators.project_range(-f, operators.nullspace_basis(shape))
    g = Grid(shape)
    g.set_density(to_dev(rho))
    p, info = g.solve_pressure(to_dev(f), restart=20, precision=precision)
    x = to_host(p)
    assert info["status"] == 0
    assert np.linalg.norm(operators.apply_pressure(x, rho) - b) <= 1.01e-10 * np.linalg.norm(b)
    if precision == "fp64":
        ref = krylov.gmres(lambda y: operators.apply_pressure(y, rho), b,
                           lambda r: operators.precond_pressure(r, float(rho.mean())), restart=20, rtol=1e-10,
                           max_iter=500)
        assert abs(info["iterations"] - ref["iterations"]) <= 1 + ref["iterations"] // 20
        for cut in (1, 7):
            q, c = g.solve_pressure(to_dev(f), restart=20, max_iter=cut)
            assert c["status"] == 1 and c["iterations"] == cut
    # a nearly constant density: the step's result almost lies in the basis, so
    # the check asks for second passes, which the first pass of the next step takes
    near = 1.0 + (1e-9 if precision == "fp64" else 2e-4) * smooth_density(shape, 5, 1.0, 2.0)
    g.set_density(to_dev(near))
    p, info = g.solve_pressure(to_dev(f), restart=20, precision=precision)
    assert info["status"] == 0 and info["iterations"] > 1 and info["gs_second_passes"] > 0
    assert np.linalg.norm(operators.apply_pressure(to_host(p), near) - b) <= 1.01e-10 * np.linalg.norm(b)
    g.set_density(to_dev(rho))
    w, wi = g.solve_helmholtz(to_dev(f), 0.05, precision=precision)
    res = operators.apply_helmholtz(to_host(w), rho, 0.05) - f
    g.close()
    assert wi["status"] == 0 and np.linalg.norm(res) <= 1.01e-10 * np.linalg.norm(f)


# CG and RMR work inside the first and last pass, for both operators: each z length
# from the shortest to the longest that carries it (512) and the first that does not,
# on small fields and above their limit, partial tiles, and fields whose last pass
# has more blocks than a reduction takes (its dots then are a launch of their own)
@pytest.mark.parametrize("shape", [(16, 16), (512, 64), (1024, 16), (16, 16, 16), (64, 32, 64), (128, 16, 16),
                                   (256, 16, 32), (16, 128, 256), (32, 128, 128), (128, 64, 64), (64, 1024, 32),
                                   (512, 1024), (16, 512, 512)])
@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
def test_cg_and_rmr_carried_by_the_passes(shape, precision):
    """The oracle's operator gives every returned field a true residual of 1e-10
    (1% for its own rounding); a second solve returns the same bits; a budget
    ends the run after that many steps."""
    from paper_2403_06654_amd.api import Grid
    rho = smooth_density(shape, 6, 1.0, 2.0)
    f = workloads.band_limited(shape, min(shape) // 4, seed=5)
    b, _ = operators.project_range(-f, operators.nullspace_basis(shape))
    g = Grid(shape)
    g.set_density(to_dev(rho))
    fd = to_dev(f)
    for solver in ("cg", "rmr"):
        p, info = g.solve_pressure(fd, solver=solver, precision=precision)
        again, _ = g.solve_pressure(fd, solver=solver, precision=precision)
        x = to_host(p)
        assert info["status"] == 0 and np.array_equal(x, to_host(again))
        assert np.linalg.norm(operators.apply_pressure(x, rho) - b) <= 1.01e-10 * np.linalg.norm(b)
        _, cut = g.solve_pressure(fd, solver=solver, max_iter=3)
        assert cut["status"] == 1 and cut["iterations"] == 3
        w, wi = g.solve_helmholtz(fd, 0.05, solver=solver, precision=precision)
        res = operators.apply_helmholtz(to_host(w), rho, 0.05) - f
        assert wi["status"] == 0 and np.linalg.norm(res) <= 1.01e-10 * np.linalg.norm(f)
    g.close()


# every column length on either side of the limit, the limit itself, and a y
# length (512) that the small configuration is not built for beside z and x
# lengths that it is; tolerances as for the other operator parity tests
@pytest.mark.parametrize("shape", [(16, 256, 16), (16, 64, 32), (32, 16, 512), (16, 512, 16), (64, 64, 64),
                                   (256, 32, 32), (16, 128, 256), (128, 32, 128), (32, 256, 64), (64, 512, 16)])
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32", 2e-5)])
def test_operators_around_the_small_field_limit(shape, prec, tol):
    from paper_2403_06654_amd.api import Grid
    rho = smooth_density(shape, 1)
    x = np.random.default_rng(2).standard_normal(shape)
    g = Grid(shape)
    g.set_density(to_dev(rho))
    y = to_host(g.apply_operator("pressure", to_dev(x), precision=prec))
    yh = to_host(g.apply_operator("helmholtz", to_dev(x), precision=prec, nu=0.013))
    g.close()
    assert rel2(y, operators.apply_pressure(x, rho)) < tol
    assert rel2(yh, operators.apply_helmholtz(x, rho, 0.013)) < tol


# odd and even wall-normal sizes from the smallest to the largest, and fields on
# either side of the size where a contraction computes two column tiles per wave
@pytest.mark.parametrize("nz,nx", [(9, 16), (100, 64), (513, 32), (33, 1024), (257, 512)])
@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
def test_wall_cg_in_the_eigenbasis(nz, nx, precision):
    """CG carried out in the basis of the preconditioner's eigenvectors: the
    oracle's operator gives the returned field a true residual of 1e-10 (1% for
    its own rounding), the field agrees with GMRES's to 2e-10 times the density
    ratio, and a warm start and an iteration budget are honoured."""
    from paper_2403_06654_amd.api import Grid
    fc = operators.FourierChebyshev2D(nx=nx, m=nz - 1, lx=2.0)
    xx, zz = fc.x[None, :], fc.z[:, None]
    rho = np.ascontiguousarray(2.0 + np.tanh((zz - 0.2 * np.sin(np.pi * xx)) / 0.4))
    f = np.ascontiguousarray(np.cos(np.pi * xx) * (1 + zz) + np.sin(2 * np.pi * xx) * zz ** 3)
    b, _ = operators.project_range(fc.rhs(f), fc.nullspace_basis())
    g = Grid((nz, nx), lengths=(2.0, 2.0), cheb=True)
    g.set_density(to_dev(rho))
    p, info = g.solve_pressure(to_dev(f), solver="cg", precision=precision)
    ref, _ = g.solve_pressure(to_dev(f), solver="gmres")
    x = to_host(p)
    assert info["status"] == 0
    assert rel2(fc.apply_pressure(x, rho), b) <= 1.01e-10
    assert rel2(x, to_host(ref)) <= 2e-10 * rho.max() / rho.min()
    warm, winfo = g.solve_pressure(to_dev(f), p=p.clone(), solver="cg", precision=precision, use_x0=True, rtol=1e-9)
    assert winfo["status"] == 0 and winfo["iterations"] == 0
    _, cut = g.solve_pressure(to_dev(f), solver="cg", max_iter=3)
    assert cut["status"] == 1 and cut["iterations"] == 3
    g.close()


@pytest.mark.parametrize("M,N,K,shift", [(257, 513, 100, 0), (514, 514, 514, 0), (520, 530, 33, 0), (600, 512, 64, 1),
                                         (1, 9000, 3, 0), (300, 9000, 1, 0)])
def test_contraction_tiles(M, N, K, shift):
    """Shapes that take the two-column-tile contraction (even N, aligned rows)
    with partial tiles, and the same sizes where it may not be taken: an odd N,
    and a right operand that starts in the middle of an aligned pair."""
    import torch
    from paper_2403_06654_amd.api import dense_matmul
    rng = np.random.default_rng(M + N + K)
    A, B = rng.standard_normal((M, K)), rng.standard_normal((K, N))
    flat = torch.zeros(K * N + 1, dtype=torch.float64, device="cuda")
    Bd = flat[shift:shift + K * N].view(K, N)
    Bd.copy_(torch.from_numpy(B))
    C = dense_matmul(torch.from_numpy(A).cuda(), Bd).cpu().numpy()
    assert rel2(C, A @ B) < 1e-14
    flat32 = torch.zeros(K * N + 1, dtype=torch.float32, device="cuda")
    Bd32 = flat32[shift:shift + K * N].view(K, N)
    Bd32.copy_(torch.from_numpy(B))
    C32 = dense_matmul(torch.from_numpy(A.astype(np.float32)).cuda(), Bd32, precision="fp32").cpu().numpy()
    assert rel2(C32.astype(np.float64), A @ B) < 2e-6


@pytest.mark.parametrize("M,N,K", [(514, 512, 257), (1026, 1024, 513), (600, 520, 1026), (1000, 514, 37),
                                   (384, 512, 40), (385, 512, 40)])
def test_contraction_sums_do_not_depend_on_the_tile(M, N, K):
    """A wide product takes two column tiles per wavefront, a narrow one a single
    tile: an element is the same sum in both, in the same order, so that the
    partial sums (and the FP32 rounding of them) do not grow with the width."""
    import torch
    from paper_2403_06654_amd.api import dense_matmul
    gen = torch.Generator(device="cuda").manual_seed(M + K)
    for precision, dtype in (("fp64", torch.float64), ("fp32", torch.float32)):
        A = torch.randn((M, K), dtype=dtype, device="cuda", generator=gen)
        B = torch.randn((K, N), dtype=dtype, device="cuda", generator=gen)
        C = dense_matmul(A, B, precision=precision)
        for c in range(0, N, 34):  # at most 3 column tiles: 195 tiles of 16 x 16
            part = dense_matmul(A, B[:, c:c + 34].contiguous(), precision=precision)
            assert bool((C[:, c:c + 34] == part).all()), (precision, c)


@pytest.mark.parametrize("cheb", [False, True])
def test_removed_norms_belong_to_their_solve(cheb):
    """rhs_null_norm of solves one after another on one grid, and of two grids
    solved together: each the norm that its own right-hand side lost, none the
    one of the solve before.  (Fourier grid: the mean, c sqrt(N) in Euclidean
    norm; Chebyshev grid: compared with a grid that solves it alone.)"""
    from paper_2403_06654_amd.api import Grid
    shape, kw = ((33, 32), dict(lengths=(2.0, 2.0), cheb=True)) if cheb else ((16, 32), {})
    rho = to_dev(smooth_density(shape, 3))
    f = np.random.default_rng(5).standard_normal(shape) if cheb else workloads.band_limited(shape, 4, seed=5)
    f -= f.mean()
    means = [3.0 * 0.5 ** k for k in range(12)]

    def alone(c):
        g = Grid(shape, **kw)
        g.set_density(rho)
        _, info = g.solve_pressure(to_dev(f + c), rtol=1e-6)
        g.close()
        return info["rhs_null_norm"]

    want = [alone(c) if cheb else c * np.sqrt(f.size) for c in means]
    grids = [Grid(shape, **kw) for _ in range(2)]
    for g in grids:
        g.set_density(rho)
    for c, w in zip(means, want):
        _, info = grids[0].solve_pressure(to_dev(f + c), rtol=1e-6)
        assert info["rhs_null_norm"] == (w if cheb else pytest.approx(w, rel=1e-9))
    for (c, d), (w, v) in zip(zip(means, means[::-1]), zip(want, want[::-1])):
        _, infos = Grid.solve_pressure_batch(grids, [to_dev(f + c), to_dev(f + d)], rtol=1e-6)
        for info, x in zip(infos, (w, v)):
            assert info["rhs_null_norm"] == (x if cheb else pytest.approx(x, rel=1e-9))
    for g in grids:
        g.close()


@pytest.mark.parametrize("shape,kind", [((32, 32, 32), "pressure"), ((64, 32), "pressure"), ((16, 32, 64), "helmholtz"),
                                        ((32, 32, 32), "cg")])
@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
def test_a_profile_changes_no_bit(shape, kind, precision):
    """A timed solve runs the launches of a plain one: the same bits whatever
    classes are timed, with the dots that an operator pass forms counted."""
    from paper_2403_06654_amd.api import Grid
    rho, f = smooth_density(shape, 7, 1.0, 6.0), workloads.band_limited(shape, 4, seed=8)
    g = Grid(shape)
    g.set_density(to_dev(rho))
    fd = to_dev(np.stack([f, np.roll(f, 3, axis=0)])) if kind == "helmholtz" else to_dev(f)

    def solve():
        if kind == "helmholtz":
            return g.solve_helmholtz(fd, 0.02, precision=precision)
        return g.solve_pressure(fd, solver="cg" if kind == "cg" else "gmres", precision=precision)

    want, plain = solve()
    for classes in (True, 1 << 10, 1 << 11, (1 << 4) | (1 << 9)):
        g.profile_read()
        g.profile_enable(classes)
        x, info = solve()
        ms, cnt, _ = g.profile_read()
        g.profile_enable(False)
        assert bool((x == want).all()) and info["iterations"] == plain["iterations"]
        if kind == "pressure" and (classes is True or classes == 1 << 10):
            assert cnt[10] == plain["iterations"] and ms[10] == 0.0
    g.close()


@pytest.mark.parametrize("shape,solver", [((32, 32, 32), "gmres"), ((64, 64), "gmres"), ((32, 32, 32), "cg"),
                                          ((16, 128, 128), "cg"), ((64, 128, 64), "cg"), ((32, 32, 32), "rmr"),
                                          ((64, 128, 64), "rmr")])
def test_a_run_that_halts_leaves_nothing_behind(shape, solver):
    """Solves of growing length on one grid, each ended on the device while the
    next step is queued (by tolerance and by the iteration limit), give the bits
    of a grid that solves each alone: what the blocks of the halting launch left
    of the next step is not read again."""
    from paper_2403_06654_amd.api import Grid
    rho, f = smooth_density(shape, 9, 1.0, 3.0), workloads.band_limited(shape, 4, seed=10)
    rd, fd = to_dev(rho), to_dev(f)
    runs = [dict(rtol=10.0 ** -k) for k in (1, 2, 4, 7, 10)] + [dict(max_iter=m) for m in (1, 2, 5)]
    g = Grid(shape)
    g.set_density(rd)
    for opts in runs:
        h = Grid(shape)
        h.set_density(rd)
        want, iw = h.solve_pressure(fd, solver=solver, **opts)
        h.close()
        for _ in range(3):
            p, info = g.solve_pressure(fd, solver=solver, **opts)
            assert info["iterations"] == iw["iterations"] and bool((p == want).all())
    g.close()
