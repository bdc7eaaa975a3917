"""The self-energy by the reduced transition matrix with the route chosen and
asserted: GWC_FACTORIZATION=spectral takes the reduction whatever the cost rule
says, and the kernel timers tell which route ran.

Orders: 0 to 20 panels of 32, odd and even in number, with and without padding
rows, panels of one and of several 64-, 128- and 256-row workgroups; one and
several cores; both modes; against the CPU oracle at the suite's 1e-9.  A
matrix whose panels have no 32 independent columns (equal energies: only the
rank-3 coupling tells the transitions apart) runs the reduction, then the Pi
builds, and the results are those of the Pi builds bit for bit."""
import numpy as np
import pytest

import paper_2412_17132_amd as gwc
from oracle import sigma as OS
from extended import dyadic_system, im_sigma_dec
from workloads import CONFIGS, system_from_config
from workloads.configs import small_config

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
TOL = 1e-9


def _run(s, mode, route, monkeypatch, **more):
    """The outputs, and the launches of (reduction, Pi builds)."""
    if route is None:
        monkeypatch.delenv("GWC_FACTORIZATION", raising=False)
    else:
        monkeypatch.setenv("GWC_FACTORIZATION", route)
    d = gwc.to_device(s, torch.device("cuda:0"))
    gwc.timing_enable(True)
    try:
        out = gwc.gwc_sigma_core(d["eps"], d["occ"], d["M_oo"], d["M_ov"], d["core_idx"], d["omega_imag"],
                                 d["w_imag"], d["omega_real"], d["eta"], mode=mode, **more)
        torch.cuda.synchronize()
        ran = gwc.timing_get("spectral_reduce")["launches"], gwc.timing_get("pi_build_f64")["launches"]
    finally:
        gwc.timing_enable(False)
    return out, ran


def _matches_oracle(s, out, mode, tol=TOL):
    ref = OS.sigma_core_system(s, mode)
    for c in range(s.n_core):
        if mode == "full":
            sc, r = out["sigma_c"][c].cpu().numpy(), ref["sigma_c"][c]
            assert np.max(np.abs(sc[:, 0] + 1j * sc[:, 1] - r)) <= tol * np.max(np.abs(r)), c
        im, r = out["im_sigma_dec"][c].cpu().numpy(), ref["im_sigma_dec"][c]
        assert np.max(np.abs(im - r)) <= tol * np.max(np.abs(r)), c
    assert np.allclose(out["e_qp"].cpu().numpy(), ref["e_qp"], rtol=tol, atol=0)


# n_occ, n_virt, n_aux, n_core
ORDERS = [(2, 16, 40, 1), (3, 11, 20, 1), (4, 16, 70, 2), (5, 13, 40, 2), (4, 24, 33, 1), (5, 26, 97, 3),
          (5, 35, 160, 1), (6, 48, 129, 2), (9, 33, 64, 1), (7, 55, 61, 2), (10, 62, 130, 1), (11, 59, 90, 2)]


@pytest.mark.parametrize("case", ORDERS, ids=[f"ov{c[0] * c[1]}" for c in ORDERS])
def test_reduction_matches_oracle(case, monkeypatch):
    n_occ, n_virt, n_aux, n_core = case
    s = system_from_config(small_config(n_occ=n_occ, n_virt=n_virt, n_aux=n_aux, n_core=n_core, n_real=6,
                                        seed=n_occ + n_virt, real_rel_ev=(-30.0, 10.0)))
    print(f"case n_ov {n_occ * n_virt}", flush=True)
    for mode in ("full", "decoupled"):
        out, ran = _run(s, mode, "spectral", monkeypatch)
        assert ran == (1, 0), (mode, ran)
        _matches_oracle(s, out, mode)


def _symmetric(n_irreps, coupling, n_occ=9, n_virt=63, n_aux=288):
    """Coefficients that vanish by the product rule of an Abelian group (up to
    `coupling` of an ordinary one): C falls into n_irreps blocks."""
    s = system_from_config(small_config(n_occ=n_occ, n_virt=n_virt, n_aux=n_aux, n_core=3, n_real=6, seed=n_irreps))
    rng = np.random.default_rng(n_irreps + 5)
    go, gv, gp = (rng.integers(n_irreps, size=n) for n in (n_occ, n_virt, n_aux))
    keep = lambda a, b: np.where((a[:, None] ^ b[None, :])[None] == gp[:, None, None], np.sqrt(n_irreps), coupling)  # noqa: E731
    s.M_oo, s.M_ov = s.M_oo * keep(go, go), s.M_ov * keep(go, gv)
    return s


@pytest.mark.parametrize("coupling", [0.0, 1e-14])
@pytest.mark.parametrize("n_irreps", [2, 4, 8])
def test_symmetric_molecules_are_reduced(n_irreps, coupling, monkeypatch):
    """A band grown from single transitions exhausts one irreducible block before
    the others, and its panels become singular (panel 6 to 14 of 16 here)."""
    print(f"case {n_irreps} blocks, coupling {coupling}", flush=True)
    s = _symmetric(n_irreps, coupling)
    out, ran = _run(s, "decoupled", "spectral", monkeypatch)
    assert ran == (1, 0), ran
    _matches_oracle(s, out, "decoupled")


def test_fewer_coefficients_than_a_panel_has_columns(monkeypatch):
    """The coupling has rank 31: the panels of a band grown from single
    transitions have no 32 independent columns."""
    print("case rank 31", flush=True)
    s = system_from_config(small_config(n_occ=7, n_virt=55, n_aux=31, n_core=2, n_real=6, seed=62, real_rel_ev=(-30.0, 10.0)))
    out, ran = _run(s, "full", "spectral", monkeypatch)
    assert ran == (1, 0), ran
    _matches_oracle(s, out, "full")


def test_dependent_panels_run_the_builds_after_the_reduction(monkeypatch):
    s = system_from_config(small_config(n_occ=3, n_virt=40, n_aux=30, n_core=1, n_real=5, seed=77))
    rng = np.random.default_rng(1)
    s.M_ov = np.einsum("Pk,kia->Pia", rng.standard_normal((30, 3)), rng.standard_normal((3, 3, 40))) * 0.02
    s.eps[:3], s.eps[3:] = -0.5, 0.25
    s.omega_real = np.linspace(-1.4, -0.3, 5)[None]
    print("case rank 3, equal energies", flush=True)
    got, ran = _run(s, "full", "spectral", monkeypatch)
    assert ran[0] == 1 and ran[1] > 0, ran
    want, ran = _run(s, "full", "ldlt", monkeypatch)
    assert ran[0] == 0 and ran[1] > 0, ran
    for k in ("sigma_c", "im_sigma_dec", "sigma_c_eps", "sigma_x", "e_qp"):
        assert torch.equal(got[k], want[k]), k
    _matches_oracle(s, got, "full")


@pytest.mark.parametrize("route", ["spectral", "ldlt"])
@pytest.mark.parametrize("shape", [(5, 35, 48, 60), (9, 63, 80, 24), (3, 21, 30, 30)], ids=["ov175", "ov567", "ov63"])
def test_residues_are_as_exact_as_the_arithmetic_allows(shape, route, monkeypatch):
    """Im Sigma^dec next to the poles against long double, by either route within 8
    eps of the terms of w^T Pi w (extended.py): each takes a few roundings.  The
    reduction rounds the whole matrix by eps max(Delta^2): the band's own W is off
    by 35 to 120 eps of them."""
    n_occ, n_virt, n_aux, n_real = shape
    s = dyadic_system(n_occ, n_virt, n_aux, n_real)
    want, bound = im_sigma_dec(s)
    print(f"case n_ov {n_occ * n_virt} {route}", flush=True)
    out, ran = _run(s, "decoupled", route, monkeypatch)
    assert (ran[0] > 0, ran[1] > 0) == (route == "spectral", route == "ldlt"), ran
    got = out["im_sigma_dec"][0].cpu().numpy()
    assert np.max(np.abs(got - want) / bound) <= 8 * np.finfo(float).eps


@pytest.mark.parametrize("case", [(8, 896), (8, 899), (7, 1033), (10, 725)], ids=lambda c: f"ov{c[0] * c[1]}")
def test_end_of_the_paired_panels(case, monkeypatch):
    """Panels go in pairs while 7168 rows are left: orders with no pair, with one, with
    one and a panel more above the limit, and with two, against the Pi builds."""
    n_occ, n_virt = case
    s = system_from_config(small_config(n_occ=n_occ, n_virt=n_virt, n_aux=50, n_core=1, n_imag=6, n_real=5, seed=n_virt))
    print(f"case n_ov {n_occ * n_virt}", flush=True)
    got, ran = _run(s, "decoupled", "spectral", monkeypatch)
    assert ran == (1, 0), ran
    want, ran = _run(s, "decoupled", "ldlt", monkeypatch)
    assert ran[0] == 0 and ran[1] > 0, ran
    for k in ("im_sigma_dec", "sigma_c_eps", "e_qp"):
        assert torch.max(torch.abs(got[k] - want[k])) <= TOL * torch.max(torch.abs(want[k])), k


def test_residues_in_several_launches(monkeypatch):
    """About 600 residue tasks of 0.11 MB: all at once, and in launches of some 250 and
    150 with a ragged last one, bit for bit; a budget of fewer than 128 goes to the
    Pi builds."""
    s = system_from_config(CONFIGS["c1"])
    print("case c1", flush=True)
    want, ran = _run(s, "full", "spectral", monkeypatch)
    assert ran == (1, 0)
    for budget, reduced in ((32, True), (22, True), (9, False)):
        monkeypatch.setenv("GWC_BATCH_BYTES", str(budget * 10 ** 6))
        got, ran = _run(s, "full", "spectral", monkeypatch)
        assert (ran[0] > 0, ran[1] > 0) == (reduced, not reduced), (budget, ran)
        for k in want:
            if reduced:
                assert torch.equal(got[k], want[k]), (budget, k)


@pytest.mark.parametrize("factor", [30.0, 300.0])
def test_large_coefficients(factor, monkeypatch):
    """V^T V up to 1e7 |Delta^2|: the band's own W is off by 30 to 70 eps of the terms."""
    s = dyadic_system()
    s.M_ov = s.M_ov * factor
    want, bound = im_sigma_dec(s)
    print(f"case coefficients times {factor}", flush=True)
    out, ran = _run(s, "decoupled", "spectral", monkeypatch)
    assert ran == (1, 0), ran
    assert np.max(np.abs(out["im_sigma_dec"][0].cpu().numpy() - want) / bound) <= 8 * np.finfo(float).eps


@pytest.mark.parametrize("case", [(4, 40, 160, 10), (5, 35, 160, 120), (8, 76, 330, 20), (8, 76, 330, 100), (9, 114, 491, 9),
                                  (10, 110, 480, 61)], ids=lambda c: f"ov{c[0] * c[1]}_points{c[3]}")
def test_both_modes_take_one_route(case, monkeypatch):
    """FULL and DECOUPLED share Sigma^c(eps_n) and E_QP, and so their last digits."""
    n_occ, n_virt, n_aux, n_real = case
    s = system_from_config(small_config(n_occ=n_occ, n_virt=n_virt, n_aux=n_aux, n_core=1, n_imag=24, n_real=n_real, seed=n_real))
    print(f"case n_ov {n_occ * n_virt}, {n_real} points", flush=True)
    full, ran_full = _run(s, "full", None, monkeypatch)
    dec, ran_dec = _run(s, "decoupled", None, monkeypatch)
    assert ran_full[0] == ran_dec[0]
    for k in ("im_sigma_dec", "sigma_c_eps", "sigma_x", "e_qp"):
        assert torch.equal(full[k], dec[k]), k


def test_newton_steps_out_of_the_reductions_range(monkeypatch):
    """A v_xc of 1e80 Ha throws Newton's second step to where |z|^4 overflows: the
    elimination's pivots have no reciprocal there, and the call goes by the Pi
    builds (whose chi is 0)."""
    s = system_from_config(small_config(n_occ=5, n_virt=35, n_aux=60, n_core=1, n_real=4, seed=8))
    more = dict(vxc=torch.full((1,), 1e80, dtype=torch.float64, device="cuda:0"), qp=dict(max_iter=4, tol=1e68, step=1e72))
    print("case Newton at -1e80", flush=True)
    want, ran = _run(s, "decoupled", "ldlt", monkeypatch, **more)
    assert ran[0] == 0
    got, ran = _run(s, "decoupled", "spectral", monkeypatch, **more)
    assert ran[0] == 1
    assert torch.isfinite(want["e_qp_newton"]).all()
    for k in ("e_qp_newton", "qp_iterations", "e_qp", "im_sigma_dec"):
        assert torch.equal(got[k], want[k]), k
