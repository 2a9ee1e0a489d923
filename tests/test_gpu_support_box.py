"""Solves on the bounding box of the contrast's support: the solution of every tier judged by
the oracle's residual on the plan's whole grid, for supports that fill their box, leave holes
in it, touch the grid's edges or are the whole grid, with the contrast moved and resized on
one plan."""
import numpy as np
import pytest

from oracle import green, matvec as mv
from paper_1803_06237_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N, H, K0, EPSB = (12, 10, 9), 0.05, inputs.K0, inputs.EPS_B


def _dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1803_06237_amd import vie
    vie.lib()
    return vie


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _eps(kind, n=N):
    eps = np.full(n, EPSB, complex)
    core = np.zeros(n, bool)
    if kind == "box":
        core[3:8, 2:5] = True
    elif kind == "moved":                # the same box elsewhere: its spectrum is kept
        core[7:12, 7:10] = True
    elif kind == "holes":                # an L and a stray column: gaps inside the box
        core[1:3, 1:8] = True
        core[1:7, 1:3] = True
        core[6, 6] = True
    elif kind == "column":
        core[11, 0, 2:7] = True
    elif kind == "wide":                 # nearly the whole grid: the plan's own operator
        core[:, 1:] = True
    else:                                # every column: the plan's own operator on the vectors
        core[:] = True
    ramp = np.linspace(0.2, 2.0, n[2])
    eps[core] = (9.0 + 1j * np.broadcast_to(ramp, n))[core]
    return eps


@pytest.fixture(scope="module")
def table():
    return green.green_table(N, mv.kappa_of(H, K0, EPSB))


def _residual(table, eps, b, x):
    op = mv.Operator(table, mv.contrast(eps, EPSB))
    return np.linalg.norm((b - op(x)).ravel()) / np.linalg.norm(b.ravel())


KINDS = ["box", "moved", "holes", "column", "wide", "all", "box"]


@pytest.mark.parametrize("precision", [0, 1, 3, 5])
def test_every_support_on_one_plan(table, precision):
    vie = _dev()
    plan = vie.Plan(N, H, K0, EPSB, fp32=True)
    rng = np.random.default_rng(precision)
    for kind in KINDS:
        eps = _eps(kind)
        plan.set_contrast(_t(eps))
        if precision == 3:
            plan.build_circulant()
        for b in (rng.standard_normal((3,) + N) + 1j * rng.standard_normal((3,) + N),
                  mv.contrast(eps, EPSB) * (1.0 + rng.standard_normal((3,) + N))):   # zero off the support
            x, info = plan.solve(_t(b), tol=1e-9, restart=60, precision=precision)
            assert info["status"] == 0, (kind, info)
            assert _residual(table, eps, b, x.cpu().numpy()) <= 1.01e-9, kind
            if precision in (0, 3):
                y, info = plan.solve_noalloc(_t(b), tol=1e-9, restart=60, precision=precision)
                assert info["status"] == 0
                assert torch.linalg.norm(y - x) <= 1e-10 * torch.linalg.norm(x)


@pytest.mark.parametrize("precision", [0, 1, 3])
@pytest.mark.parametrize("use_graph", [False, True])
def test_supports_of_every_kind_in_one_batch(table, precision, use_graph):
    vie = _dev()
    rng = np.random.default_rng(10 + precision)
    kinds = ["box", "holes", "all", "wide", "column", "box"]
    plans, bs, epss = [], [], []
    for i, kind in enumerate(kinds):
        eps = _eps(kind)
        if i == 5:                       # a second right-hand side of the first system
            plan = plans[0]
        else:
            plan = vie.Plan(N, H, K0, EPSB, fp32=True)
            plan.set_contrast(_t(eps))
            if precision == 3:
                plan.build_circulant()
        plans.append(plan)
        epss.append(eps)
        bs.append(rng.standard_normal((3,) + N) + 1j * rng.standard_normal((3,) + N))
    xs, infos, code = vie.solve_batch(plans, [_t(b) for b in bs], tol=1e-9, restart=40, precision=precision,
                                      use_graph=use_graph)
    assert code == 0, infos
    for kind, eps, b, x in zip(kinds, epss, bs, xs):
        assert _residual(table, eps, b, x.cpu().numpy()) <= 1.01e-9, kind
    again, infos, code = vie.solve_batch(plans, [_t(b) for b in bs], xs=[x.clone() for x in xs], tol=1e-9, restart=40,
                                         precision=precision, use_x0=True, use_graph=use_graph)
    assert code == 0 and all(i["iters"] == 0 for i in infos), infos


def test_first_solve_on_another_box_is_not_much_dearer():
    """Rough guides move the box with every contrast: the first solve of two steps after a change
    against a repeated one (0.05 ms more; 0.35 ms with spectra made for each box)."""
    import os
    import time
    vie = _dev()
    if os.environ.get("VIE_DEBUG_NANFILL") == "1":
        pytest.skip("allocations are filled")
    n = (8, 8, 32)
    plan = vie.Plan(n, H, K0, EPSB, fp32=False)
    rng = np.random.default_rng(0)
    b = _t(rng.standard_normal((3,) + n) + 1j * rng.standard_normal((3,) + n))
    epss = []
    for box in (np.s_[2:6, 2:6], np.s_[1:6, 2:6], np.s_[2:6, 2:7], np.s_[1:7, 2:6]):
        eps = np.full(n, EPSB, complex)
        eps[box] = 12.11 + 0.3j
        epss.append(_t(eps))

    def solve():
        torch.cuda.synchronize()
        t = time.perf_counter()
        plan.solve(b, tol=1e-300, restart=2, maxit=2)
        return time.perf_counter() - t

    first, again = [], []
    for i in range(40):
        plan.set_contrast(epss[i % 4])
        first.append(solve())
        again.append(solve())
    assert np.median(first) - np.median(again) <= 0.15e-3, (np.median(first), np.median(again))


def test_boxes_of_many_circulant_lengths_on_one_plan():
    """More lengths than a plan keeps spectra of, each visited twice, against the oracle."""
    vie = _dev()
    n = (20, 12, 6)
    tab = green.green_table(n, mv.kappa_of(H, K0, EPSB))
    plan = vie.Plan(n, H, K0, EPSB, fp32=True)
    rng = np.random.default_rng(5)
    b = rng.standard_normal((3,) + n) + 1j * rng.standard_normal((3,) + n)
    for w1, w2 in 2 * [(1, 1), (2, 3), (4, 5), (9, 2), (17, 4), (16, 8), (3, 10), (14, 12)]:
        eps = np.full(n, EPSB, complex)
        eps[20 - w1:, 12 - w2:] = 9.0 + 0.5j
        plan.set_contrast(_t(eps))
        for precision in (0, 1):
            x, info = plan.solve(_t(b), tol=1e-9, restart=60, precision=precision)
            assert info["status"] == 0, (w1, w2, info)
            assert _residual(tab, eps, b, x.cpu().numpy()) <= 1.01e-9, (w1, w2)


@pytest.mark.parametrize("precision", [0, 1, 3])
def test_box_is_in_use_unless_there_is_no_memory(table, precision, monkeypatch):
    """Solves run on the box where the rule says so.  Without memory for it they run on the plan's
    own grid until the next contrast; another error of making it is the solve's."""
    vie = _dev()
    boxes = {"box": (3, 8, 2, 5), "moved": (7, 12, 7, 10), "holes": (1, 7, 1, 8), "column": (11, 12, 0, 1)}
    plan = vie.Plan(N, H, K0, EPSB, fp32=True)
    rng = np.random.default_rng(7)
    b = rng.standard_normal((3,) + N) + 1j * rng.standard_normal((3,) + N)

    def contrast(kind, eps=None):
        plan.set_contrast(_t(_eps(kind) if eps is None else eps))
        if precision == 3:
            plan.build_circulant()

    def solve(kind):
        x, info = plan.solve(_t(b), tol=1e-9, restart=60, precision=precision)
        assert info["status"] == 0
        assert _residual(table, _eps(kind), b, x.cpu().numpy()) <= 1.01e-9, kind

    for kind in KINDS:
        contrast(kind)
        assert plan.solve_box() == (0, N[0], 0, N[1])
        solve(kind)
        assert plan.solve_box() == boxes.get(kind, (0, N[0], 0, N[1])), kind
    plan = vie.Plan(N, H, K0, EPSB, fp32=True)
    spread = np.full(N, EPSB, complex)                   # as many columns, all over the grid
    spread.reshape(-1, N[2])[np.linspace(0, N[0] * N[1] - 1, 15).astype(int)] = 9.0 + 0.5j
    contrast("spread", spread)
    plan.solve(_t(b), tol=1e-9, restart=60, precision=precision)
    assert plan.solve_box() == (0, N[0], 0, N[1])        # the workspaces are there, no box is
    contrast("box")
    monkeypatch.setenv("VIE_DEBUG_MALLOC_ERROR", "0 2")  # hipErrorOutOfMemory
    solve("box")
    monkeypatch.delenv("VIE_DEBUG_MALLOC_ERROR")
    solve("box")
    assert plan.solve_box() == (0, N[0], 0, N[1])
    contrast("box")
    monkeypatch.setenv("VIE_DEBUG_MALLOC_ERROR", "0 1")  # hipErrorInvalidValue
    with pytest.raises(vie.VieError) as err:
        plan.solve(_t(b), tol=1e-9, restart=60, precision=precision)
    assert err.value.code == vie.VIE_EDEVICE
    monkeypatch.delenv("VIE_DEBUG_MALLOC_ERROR")
    solve("box")
    assert plan.solve_box() == boxes["box"]
