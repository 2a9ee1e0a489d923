"""GPU block-circulant preconditioner (Section V-D) against the oracle.

* apply parity: z = W^{-1} r from libvie.so vs the oracle's FFT-diagonalised
  inverse, element by element, on grids with radix-2/3/5/43 slice counts, ragged
  supports and the degenerate cases (one slice, no contrast);
* full size (32 x 32 x 512 guide): single-frequency inputs, checked against the
  oracle's block of that frequency solved densely;
* preconditioned solves: FP64 FGMRES with W^{-1} reaches 1e-8 (residual recomputed
  by the oracle) in far fewer iterations than plain GMRES.
"""
import numpy as np
import pytest

from oracle import circulant as circ
from oracle import green, matvec as mv
from paper_1803_06237_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1803_06237_amd import vie
    vie.lib()
    return vie


def _guide(n, core_x, core_y, n_abs, d=2, sigma_max=2.0, h=0.05):
    return inputs.Waveguide(n=n, h=h, core_x=core_x, core_y=core_y, core_z=(0, n[2]), n_abs=n_abs, d=d,
                            sigma_max=sigma_max)


def _ragged_eps(n, seed):
    """Silicon on an irregular set of columns whose extent varies along z (rough sidewalls)."""
    rng = np.random.default_rng(seed)
    eps = np.full(n, inputs.EPS_B, dtype=np.complex128)
    for i3 in range(n[2]):
        w = rng.integers(1, max(2, n[0] - 1))
        lo = rng.integers(0, n[0] - w + 1)
        eps[lo:lo + w, n[1] // 2, i3] = inputs.EPS_SI + 0.3j * (i3 / n[2]) ** 2
        if n[1] > 2:
            eps[lo, n[1] // 2 - 1, i3] = inputs.EPS_SI
    return eps


CASES = [
    ("strip_6x6x32", lambda: _guide((6, 6, 32), (1, 5), (2, 4), 8).eps()),
    ("strip_5x4x24_radix3", lambda: _guide((5, 4, 24), (1, 4), (1, 3), 4).eps()),
    ("strip_4x3x40_radix5", lambda: _guide((4, 3, 40), (1, 3), (1, 2), 6).eps()),
    ("ragged_7x5x129", lambda: _ragged_eps((7, 5, 129), 3)),
    ("ragged_9x4x20", lambda: _ragged_eps((9, 4, 20), 4)),
    ("one_slice_5x5x1", lambda: _guide((5, 5, 1), (1, 4), (2, 3), 0).eps()),
    # core shorter than the grid: slice window (5, 40), and (8, 40) shifted to fit the end
    ("gap_6x6x48", lambda: inputs.Waveguide(n=(6, 6, 48), h=0.05, core_x=(1, 5), core_y=(2, 4), core_z=(5, 43),
                                            n_abs=6, d=2, sigma_max=2.0).eps()),
    ("gap_end_6x5x48", lambda: inputs.Waveguide(n=(6, 5, 48), h=0.05, core_x=(2, 5), core_y=(1, 4),
                                                core_z=(10, 47), n_abs=5, d=1, sigma_max=3.0).eps()),
]


def _oracle_apply(eps, h, r):
    kap = mv.kappa_of(h, inputs.K0, inputs.EPS_B)
    table = green.green_table(eps.shape, kap)
    chi = mv.contrast(eps, inputs.EPS_B)
    S = circ.support_columns(chi)
    Winv = circ.spectrum_inverse(circ.optimal_blocks(table, chi, S))
    return circ.apply(Winv, S, r, circ.support_window(chi))


@pytest.mark.parametrize("fp64", [True, False], ids=["fp64", "fp32"])
@pytest.mark.parametrize("name,make", CASES, ids=[c[0] for c in CASES])
def test_apply_matches_oracle(name, make, fp64):
    vie = _dev()
    eps = make()
    n = eps.shape
    h = 0.05
    plan = vie.Plan(n, h, inputs.K0, inputs.EPS_B)
    plan.set_contrast(torch.from_numpy(eps).cuda())
    info = plan.build_circulant(fp64=fp64)
    rng = np.random.default_rng(11)
    r = rng.standard_normal((3,) + n) + 1j * rng.standard_normal((3,) + n)
    z = plan.apply_circulant(torch.from_numpy(r).cuda()).cpu().numpy()
    zo = _oracle_apply(eps, h, r)
    err = np.max(np.abs(z - zo)) / np.max(np.abs(zo))
    print(name, info, "max rel err", err)
    chi = mv.contrast(eps, inputs.EPS_B)
    z0, P = circ.support_window(chi)
    assert info["block_size"] == 3 * info["support_columns"]
    assert (info["first_slice"], info["blocks"]) == (z0, P)
    assert err <= (1e-11 if fp64 else 2e-5)
    # outside the support columns and outside the slice window the preconditioner is
    # the identity, bit for bit
    outside = ~np.any(chi != 0, axis=2)
    assert np.array_equal(z[:, outside, :], r[:, outside, :])
    assert np.array_equal(z[:, :, :, :z0], r[:, :, :, :z0])
    assert np.array_equal(z[:, :, :, z0 + P:], r[:, :, :, z0 + P:])


def test_no_contrast_is_the_identity():
    vie = _dev()
    n = (4, 4, 8)
    plan = vie.Plan(n, 0.05, inputs.K0, inputs.EPS_B)
    plan.set_contrast(torch.full(n, inputs.EPS_B, dtype=torch.complex128).cuda())
    info = plan.build_circulant()
    assert info["support_columns"] == 0 and info["blocks"] == 0
    r = torch.randn((3,) + n, dtype=torch.complex128).cuda()
    assert torch.equal(plan.apply_circulant(r), r)


def test_state_errors():
    vie = _dev()
    n = (4, 4, 8)
    plan = vie.Plan(n, 0.05, inputs.K0, inputs.EPS_B)
    r = torch.zeros((3,) + n, dtype=torch.complex128).cuda()
    with pytest.raises(vie.VieError) as e:
        plan.build_circulant()
    assert e.value.code == vie.VIE_ESTATE
    eps = _guide(n, (1, 3), (1, 3), 2).eps()
    plan.set_contrast(torch.from_numpy(eps).cuda())
    with pytest.raises(vie.VieError) as e:
        plan.apply_circulant(r)
    assert e.value.code == vie.VIE_ESTATE
    plan.build_circulant()
    plan.apply_circulant(r)
    plan.set_contrast(torch.from_numpy(eps).cuda())        # releases the stale preconditioner
    with pytest.raises(vie.VieError) as e:
        plan.apply_circulant(r)
    assert e.value.code == vie.VIE_ESTATE
    with pytest.raises(vie.VieError) as e:
        plan.solve(r + 1, precision=3)
    assert e.value.code == vie.VIE_ESTATE


def _oracle_support_table(n, S, kappa):
    """Oracle Galerkin entries for the offsets a support S can reach (|m1|, |m2| within S,
    every m3), computed in CPU worker processes; the rest of the table stays zero."""
    import multiprocessing as mp
    import os
    from functools import partial
    d1 = int(S[:, 0].max() - S[:, 0].min()) + 1
    d2 = int(S[:, 1].max() - S[:, 1].min()) + 1
    offs = np.stack(np.meshgrid(np.arange(d1), np.arange(d2), np.arange(n[2]), indexing="ij"), -1).reshape(-1, 3)
    chunks = np.array_split(offs, 64)
    with mp.get_context("spawn").Pool(min(16, os.cpu_count() or 1)) as pool:
        vals = pool.map(partial(green.galerkin_N, kappa=kappa), chunks)
    table = np.zeros((6,) + tuple(n), dtype=np.complex128)
    table[:, :d1, :d2, :] = np.concatenate(vals, axis=1).reshape(6, d1, d2, n[2])
    return table


FREQS = (0, 1, 511)


@pytest.fixture(scope="module")
def long_guide():
    vie = _dev()
    wg = inputs.strip_long(d=2)
    plan = vie.Plan(wg.n, wg.h, wg.k0, wg.eps_b, fp32=True)
    plan.set_contrast(torch.from_numpy(wg.eps()).cuda())
    return wg, plan


@pytest.fixture(scope="module")
def long_guide_blocks(long_guide):
    wg, _ = long_guide
    chi = mv.contrast(wg.eps(), wg.eps_b)
    S = circ.support_columns(chi)
    table = _oracle_support_table(wg.n, S, mv.kappa_of(wg.h, wg.k0, wg.eps_b))
    return S, {f: circ.frequency_block(table, chi, S, f) for f in FREQS}


@pytest.mark.parametrize("fp64", [True, False], ids=["fp64", "fp32"])
def test_full_size_single_frequencies(long_guide, long_guide_blocks, fp64):
    """32 x 32 x 512, 20 x 9 core (m = 540): for r = v e^{2 pi i f i3 / n3} on S the exact
    W^{-1} r is u e^{2 pi i f i3 / n3} with What_f u = v."""
    wg, plan = long_guide
    S, blocks = long_guide_blocks
    info = plan.build_circulant(fp64=fp64)
    print(info)
    s, n3 = len(S), wg.n[2]
    assert info["support_columns"] == s == 180
    assert circ.support_window(mv.contrast(wg.eps(), wg.eps_b)) == (0, n3) == (info["first_slice"], info["blocks"])
    rng = np.random.default_rng(2)
    for f in FREQS:
        v = rng.standard_normal(3 * s) + 1j * rng.standard_normal(3 * s)
        ph = np.exp(2j * np.pi * f * np.arange(n3) / n3)
        r = np.zeros((3,) + wg.n, dtype=np.complex128)
        for a in range(3):
            r[a][S[:, 0], S[:, 1], :] = v[a * s:(a + 1) * s, None] * ph[None]
        z = plan.apply_circulant(torch.from_numpy(r).cuda()).cpu().numpy()
        u = np.linalg.solve(blocks[f], v)
        zo = np.zeros_like(r)
        for a in range(3):
            zo[a][S[:, 0], S[:, 1], :] = u[a * s:(a + 1) * s, None] * ph[None]
        err = np.max(np.abs(z - zo)) / np.max(np.abs(zo))
        print("f", f, "max rel err", err)
        assert err <= (1e-10 if fp64 else 5e-5)


@pytest.fixture(scope="module")
def small_strip():
    vie = _dev()
    wg = inputs.strip_small(d=2)
    kap = mv.kappa_of(wg.h, wg.k0, wg.eps_b)
    op = mv.Operator(green.green_table(wg.n, kap), mv.contrast(wg.eps(), wg.eps_b))
    plan = vie.Plan(wg.n, wg.h, wg.k0, wg.eps_b, fp32=True)
    plan.set_contrast(torch.from_numpy(wg.eps()).cuda())
    b = mv.rhs_from_field(wg.eps(), wg.eps_b, inputs.strip_small_dipole_rhs_field(wg), wg.h)
    return wg, op, plan, b


@pytest.mark.parametrize("fp64", [True, False], ids=["fp64", "fp32"])
def test_preconditioned_solve_small(small_strip, fp64):
    wg, op, plan, b = small_strip
    plan.build_circulant(fp64=fp64)
    bt = torch.from_numpy(b).cuda()
    x0, i0 = plan.solve(bt, tol=1e-8, restart=50, precision=0)
    x3, i3 = plan.solve(bt, tol=1e-8, restart=50, precision=3)
    rr = np.linalg.norm(b.ravel() - op(x3.cpu().numpy().ravel())) / np.linalg.norm(b)
    print("plain", i0["iters"], "circulant", i3["iters"], "oracle rel res", rr)
    assert i3["status"] == 0 and rr <= 1.01e-8
    assert i3["iters"] <= 0.6 * i0["iters"]
    assert i3["inner_iters"] >= i3["iters"]


def test_preconditioned_solve_full_size(long_guide):
    wg, plan = long_guide
    plan.build_circulant(fp64=False)
    b = plan.rhs(torch.from_numpy(inputs.transverse_dipole_field(wg)).cuda())
    x, info = plan.solve(b, tol=1e-8, restart=50, precision=3)
    r = plan.residual(x, b)
    rel = (torch.linalg.norm(r) / torch.linalg.norm(b)).item()
    print(info, rel)
    assert info["status"] == 0 and rel <= 1e-8
    assert info["iters"] <= 150        # plain GMRES(50) needs several hundred here
