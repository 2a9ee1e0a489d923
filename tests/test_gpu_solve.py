"""GPU GMRES solves judged by the oracle: the oracle recomputes the residual of the
GPU solution with its own matvec (several solutions are correct; the residual is
what is unique)."""
import numpy as np
import pytest

from oracle import green, matvec as mv, solve
from paper_1803_06237_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1803_06237_amd import vie
    vie.lib()
    return vie


@pytest.fixture(scope="module")
def small_strip():
    """8 x 8 x 32, h = 50 nm, 4 x 4 core, 8-voxel quadratic absorbers, sigma_max = 2."""
    vie = _dev()
    wg = inputs.strip_small(d=2)
    kap = mv.kappa_of(wg.h, wg.k0, wg.eps_b)
    op = mv.Operator(green.green_table(wg.n, kap), mv.contrast(wg.eps(), wg.eps_b))
    plan = vie.Plan(wg.n, wg.h, wg.k0, wg.eps_b, fp32=True)
    plan.set_contrast(torch.from_numpy(wg.eps()).cuda())
    e_inc = inputs.strip_small_dipole_rhs_field(wg)
    b_dip = mv.rhs_from_field(wg.eps(), wg.eps_b, e_inc, wg.h)
    b_gau = inputs.gaussian_rhs(wg.n, 0)
    return wg, op, plan, b_dip, b_gau, e_inc


def _oracle_rel_res(op, b, x):
    return np.linalg.norm(b.ravel() - op(x.ravel())) / np.linalg.norm(b)


@pytest.mark.parametrize("rhs", ["dipole", "gaussian"])
@pytest.mark.parametrize("restart", [50, 400])
def test_fp64_gmres(small_strip, rhs, restart):
    wg, op, plan, b_dip, b_gau, _ = small_strip
    b = b_dip if rhs == "dipole" else b_gau
    x, info = plan.solve(torch.from_numpy(b).cuda(), tol=1e-8, restart=restart)
    rr = _oracle_rel_res(op, b, x.cpu().numpy())
    print(rhs, restart, info, "oracle rel res", rr)
    assert info["status"] == 0
    assert info["rel_res_true"] <= 1e-8
    assert rr <= 1.01e-8


def test_gpu_rhs_builds_the_same_system(small_strip):
    wg, op, plan, b_dip, _, e_inc = small_strip
    b = plan.rhs(torch.from_numpy(e_inc).cuda())
    assert np.max(np.abs(b.cpu().numpy() - b_dip)) <= 4e-16 * np.max(np.abs(b_dip))


def test_mixed_precision_reaches_fp64_tolerance(small_strip):
    wg, op, plan, b_dip, b_gau, _ = small_strip
    for b in (b_dip, b_gau):
        x, info = plan.solve(torch.from_numpy(b).cuda(), tol=1e-8, restart=30, precision=1,
                             inner_restart=20, inner_tol=1e-4)
        rr = _oracle_rel_res(op, b, x.cpu().numpy())
        print("mixed", info, "oracle rel res", rr)
        assert info["status"] == 0 and rr <= 1.01e-8
        assert info["inner_iters"] > 0


def test_solution_matches_dense_lu_within_conditioning():
    vie = _dev()
    wg = inputs.Waveguide(n=(4, 4, 12), h=0.05, core_x=(1, 3), core_y=(1, 3), core_z=(0, 12), n_abs=3,
                          d=1, sigma_max=2.0)
    kap = mv.kappa_of(wg.h, wg.k0, wg.eps_b)
    T = green.green_table(wg.n, kap)
    chi = mv.contrast(wg.eps(), wg.eps_b)
    A = mv.dense_A(T, chi)
    b = inputs.gaussian_rhs(wg.n, 7)
    x_lu = solve.solve_lu(A, b.ravel())
    plan = vie.Plan(wg.n, wg.h, wg.k0, wg.eps_b, fp32=False)
    plan.set_contrast(torch.from_numpy(wg.eps()).cuda())
    x, info = plan.solve(torch.from_numpy(b).cuda(), tol=1e-10, restart=200)
    err = np.linalg.norm(x.cpu().numpy().ravel() - x_lu) / np.linalg.norm(x_lu)
    assert err < 10 * np.linalg.cond(A) * 1e-10


def test_zero_rhs_and_warm_start(small_strip):
    wg, op, plan, b_dip, _, _ = small_strip
    z = torch.zeros((3,) + wg.n, dtype=torch.complex128, device="cuda")
    x, info = plan.solve(z, tol=1e-8)
    assert info["status"] == 0 and torch.count_nonzero(x) == 0
    b = torch.from_numpy(b_dip).cuda()
    x1, i1 = plan.solve(b, tol=1e-8)
    x2, i2 = plan.solve(b, x=x1.clone(), tol=1e-8, use_x0=True)
    assert i2["iters"] == 0 and i2["status"] == 0


def test_maxit_reports_noconv_with_best_iterate(small_strip):
    vie = _dev()
    wg, op, plan, _, b_gau, _ = small_strip
    x, info = plan.solve(torch.from_numpy(b_gau).cuda(), tol=1e-14, restart=5, maxit=5)
    assert info["status"] == vie.VIE_ENOCONV
    rr = _oracle_rel_res(op, b_gau, x.cpu().numpy())
    assert rr < 1.0 and abs(rr - info["rel_res_true"]) < 1e-10


@pytest.mark.parametrize("maxit", [1, 2, 4, 5, 6, 9, 13])
def test_truncated_gmres_matches_oracle_gmres(small_strip, maxit):
    """After every step count the device GMRES(5) iterate is the oracle's GMRES(5)
    iterate: maxit inside a restart cycle (a following step is already queued on the
    device and must be discarded), at its end, and across restarts.  The dipole
    right-hand side lies on the contrast's support, where the device's compressed
    Krylov space equals the full one."""
    vie = _dev()
    wg, op, plan, b_dip, _, _ = small_strip
    x, info = plan.solve(torch.from_numpy(b_dip).cuda(), tol=1e-14, restart=5, maxit=maxit)
    xo, io = solve.gmres(op, b_dip.ravel(), tol=1e-14, restart=5, maxit=maxit)
    assert info["status"] == vie.VIE_ENOCONV and info["iters"] == maxit == io.iters
    xg = x.cpu().numpy().ravel()
    rr = _oracle_rel_res(op, b_dip, xg)
    ro = np.linalg.norm(b_dip.ravel() - op(xo)) / np.linalg.norm(b_dip)
    print(maxit, rr, ro, info["rel_res_est"], io.history[-1])
    assert abs(rr - ro) <= 1e-9 * ro
    assert np.linalg.norm(xg - xo) <= 1e-8 * np.linalg.norm(xo)
    assert abs(info["rel_res_est"] - io.history[-1]) <= 1e-9 * io.history[-1]


def test_stall_rule_stops_below_the_attainable_floor(small_strip):
    """tol = 1e-18 lies below what FP64 GMRES can reach: with stall_restarts the solve
    stops a few restarts after the residual stops falling (VIE_ENOCONV, stalled)
    instead of running to maxit, and the iterate it returns is at the floor."""
    vie = _dev()
    wg, op, plan, b_dip, b_gau, _ = small_strip
    b = torch.from_numpy(b_gau).cuda()
    x, info = plan.solve(b, tol=1e-18, restart=20, maxit=100000, stall_restarts=3)
    rr = _oracle_rel_res(op, b_gau, x.cpu().numpy())
    print(info, "oracle rel res", rr)
    assert info["status"] == vie.VIE_ENOCONV and info["stalled"] == 1 and info["fallback"] == 0
    assert info["iters"] < 5000
    assert info["rel_res_true"] < 1e-13 and rr < 1e-12
    # the same solve to 1e-8 is unchanged by the rule: it progresses every restart
    x1, i1 = plan.solve(b, tol=1e-8, restart=20)
    x2, i2 = plan.solve(b, tol=1e-8, restart=20, stall_restarts=2)
    assert i1["status"] == i2["status"] == 0 and i2["stalled"] == 0
    assert i1["iters"] == i2["iters"] and torch.equal(x1, x2)


@pytest.mark.parametrize("precision", [1, 5])
def test_mixed_tier_hands_a_stall_to_fp64_gmres(small_strip, precision):
    """A mixed-tier outer FGMRES that stalls hands its iterate to FP64 GMRES (fallback)
    for the rest of the budget; below the floor that one stalls too."""
    vie = _dev()
    wg, op, plan, b_dip, b_gau, _ = small_strip
    x, info = plan.solve(torch.from_numpy(b_gau).cuda(), tol=1e-18, restart=20, maxit=100000,
                         precision=precision, inner_restart=10, inner_tol=1e-3, stall_restarts=2)
    rr = _oracle_rel_res(op, b_gau, x.cpu().numpy())
    print(precision, info, "oracle rel res", rr)
    assert info["status"] == vie.VIE_ENOCONV and info["fallback"] == 1 and info["stalled"] == 1
    assert info["iters"] < 5000 and rr < 1e-12


# Arnoldi steps with the two Gram-Schmidt sweeps merged: one cycle of m steps against the
# oracle's GMRES (sweeps apart).  1800 unknowns and 14400 (several blocks per dot, ragged last
# chunks); m past the groups of 4 and 64 vectors.
@pytest.fixture(scope="module", params=[(6, 5, 20), (12, 10, 40)], ids=lambda g: "x".join(map(str, g)))
def slow_system(request):
    vie = _dev()
    n, h, k0, eps_b = request.param, 0.1, inputs.K0, inputs.EPS_B
    rng = np.random.default_rng(sum(n))
    eps = eps_b + 8.0 * rng.random(n) + 0.01j
    op = mv.Operator(green.green_table(n, mv.kappa_of(h, k0, eps_b)), mv.contrast(eps, eps_b))
    plan = vie.Plan(n, h, k0, eps_b, fp32=True)
    plan.set_contrast(torch.from_numpy(eps).cuda())
    b = inputs.gaussian_rhs(n, 3)
    _, info = solve.fgmres(op, b.ravel(), tol=1e-15, restart=140, maxit=140)
    return op, plan, b, info.history


@pytest.mark.parametrize("m", [1, 2, 8, 9, 33, 64, 65, 140])
def test_one_cycle_equals_the_oracle(slow_system, m):
    op, plan, b, history = slow_system
    x, info = plan.solve(torch.from_numpy(b).cuda(), tol=1e-15, restart=m, maxit=m)
    true = _oracle_rel_res(op, b, x.cpu().numpy())
    want = history[min(m, len(history)) - 1]      # the small system ends before 140 steps
    # both residuals in units of ||b||: FP64 rounding of a few hundred products and projections
    assert abs(true - want) <= 1e-12, (m, true, want)
    assert abs(info["rel_res_true"] - true) <= 1e-13


# One voxel of permittivity near zero multiplies its rows of A by |1 - eps_b / eps|: every step
# then cancels to about the reciprocal of that, and the basis stays orthogonal only if what is
# left of w is measured against it again.
def _near_zero_voxel(small):
    n, h, k0, eps_b = (6, 5, 8), 0.05, inputs.K0, inputs.EPS_B
    eps = np.full(n, 12.11 + 0.3j)
    eps[3, 2, 4] = small * (1.0 + 0.5j)
    chi = mv.contrast(eps, eps_b)
    op = mv.Operator(green.green_table(n, mv.kappa_of(h, k0, eps_b)), chi)
    # rounding of the product, 20 steps' worth, in units of ||b||
    return (n, h, k0, eps_b), eps, op, inputs.gaussian_rhs(n, 4), 20 * 2.0 ** -52 * np.abs(chi).max()


@pytest.mark.parametrize("small,m", [(1e-2, 30), (1e-8, 30), (1e-10, 8), (1e-10, 15), (1e-11, 15)])
def test_one_cycle_of_cancelling_steps_equals_the_oracle(small, m):
    vie = _dev()
    args, eps, op, b, bound = _near_zero_voxel(small)
    plan = vie.Plan(*args, fp32=False)
    plan.set_contrast(torch.from_numpy(eps).cuda())
    _, ref = solve.fgmres(op, b.ravel(), tol=1e-15, restart=m, maxit=m)
    x, info = plan.solve(torch.from_numpy(b).cuda(), tol=1e-15, restart=m, maxit=m)
    true = _oracle_rel_res(op, b, x.cpu().numpy())
    assert info["iters"] == m
    assert abs(true - ref.history[m - 1]) <= bound + 1e-12, (true, ref.history[m - 1], bound)
    assert abs(info["rel_res_est"] - true) <= bound + 1e-12


@pytest.mark.parametrize("precision", [1, 3])
@pytest.mark.parametrize("small,m", [(1e-2, 10), (1e-10, 5), (1e-10, 15)])
def test_estimate_of_a_preconditioned_cycle_of_cancelling_steps(precision, small, m):
    """Flexible cycles queue the extra sweep with their first steps and repeat a later one that
    turns out to need it (the 1e-10 cases, on its stored preconditioned vector): the Hessenberg
    estimate stays the true residual."""
    vie = _dev()
    args, eps, op, b, bound = _near_zero_voxel(small)
    plan = vie.Plan(*args, fp32=True)
    plan.set_contrast(torch.from_numpy(eps).cuda())
    plan.build_circulant()
    x, info = plan.solve(torch.from_numpy(b).cuda(), tol=1e-15, restart=m, maxit=m, precision=precision,
                         inner_restart=3, inner_tol=1e-1)
    true = _oracle_rel_res(op, b, x.cpu().numpy())
    assert info["iters"] == m
    assert abs(info["rel_res_est"] - true) <= bound + 1e-12, (info, true, bound)


@pytest.mark.parametrize("cycles", [1, 3])
def test_cycles_of_cancelling_steps_in_a_batch(cycles):
    """The same in a batch, next to a system without the voxel, whose steps do not cancel; the
    second cycle is captured, the third replays it."""
    vie = _dev()
    m, cases, plans = 15, [_near_zero_voxel(s) for s in (1e-10, 12.11, 1e-2, 1e-11)], []
    for args, eps, *_ in cases:
        plans.append(vie.Plan(*args, fp32=False))
        plans[-1].set_contrast(torch.from_numpy(eps).cuda())
    bs = [torch.from_numpy(c[3]).cuda() for c in cases]
    xs, infos, _ = vie.solve_batch(plans, bs, tol=1e-15, restart=m, maxit=cycles * m)
    for (_, _, op, b, bound), x, info in zip(cases, xs, infos):
        _, ref = solve.fgmres(op, b.ravel(), tol=1e-15, restart=m, maxit=cycles * m)
        true = _oracle_rel_res(op, b, x.cpu().numpy())
        assert info["iters"] == cycles * m
        assert abs(true - ref.history[-1]) <= bound + 1e-12, (true, ref.history[-1], bound)


def test_long_cycles_stay_cheap():
    """The Gram matrix's share of a step grows with the square of the cycle.  768 unknowns, so
    that the basis itself stays in cache: an average step of 700 against one of 50 (1.75 times
    it; 3.4 with the projections in one workgroup on uncoalesced reads)."""
    import time
    vie = _dev()
    n = (6, 6, 16)
    eps = np.full(n, inputs.EPS_B, complex)
    eps[1:5, 1:5] += 8.0 * np.random.default_rng(0).random((4, 4, 16)) + 0.01j
    plan = vie.Plan(n, 0.1, inputs.K0, inputs.EPS_B, fp32=False)
    plan.set_contrast(torch.from_numpy(eps).cuda())
    b = torch.from_numpy(inputs.gaussian_rhs(n, 1)).cuda()

    def step(m):
        best = np.inf
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            _, info = plan.solve(b, tol=1e-300, restart=m, maxit=m)
            best = min(best, (time.perf_counter() - t) / info["iters"])
        return best

    assert step(700) <= 2.5 * step(50)


def test_workspace_that_did_not_fit_is_made_again(monkeypatch):
    """A cycle whose Hessenberg matrix is larger than its basis: the first allocations of the
    workspace succeed, that one fails, and the next call makes all of it."""
    vie = _dev()
    args, eps, op, b, _ = _near_zero_voxel(12.11)
    plan = vie.Plan(*args, fp32=False)
    plan.set_contrast(torch.from_numpy(eps).cuda())
    run = lambda m: plan.solve(torch.from_numpy(b).cuda(), tol=1e-9, restart=m, maxit=m)
    run(50)
    monkeypatch.setenv("VIE_DEBUG_MALLOC_ERROR", f"{14 << 20} 2")   # the basis 11.5 MB, the matrix 16
    with pytest.raises(vie.VieError) as err:
        run(1000)
    assert err.value.code in (vie.VIE_ENOMEM, vie.VIE_EDEVICE)
    monkeypatch.delenv("VIE_DEBUG_MALLOC_ERROR")
    x, info = run(1000)
    assert info["status"] == 0 and _oracle_rel_res(op, b, x.cpu().numpy()) <= 1.01e-9
