"""What a call refuses: bad coefficients, with every output left as it was,
whichever route to W the sizes take and wherever the outputs are; and the orders
and budgets that the Pi builds refuse, also where the reduction would fit."""
import numpy as np
import pytest

import paper_2412_17132_amd as gwc
from workloads import system_from_config
from workloads.configs import small_config

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("outputs", ["device", "host"])
@pytest.mark.parametrize("route", ["builds", "reduction"])
def test_outputs_untouched(outputs, route, monkeypatch):
    if route == "builds":
        monkeypatch.setenv("GWC_FACTORIZATION", "ldlt")
    else:
        monkeypatch.delenv("GWC_FACTORIZATION", raising=False)  # an order of 32 is always reduced
    s = system_from_config(small_config(n_occ=4, n_virt=8, n_aux=30, n_core=2, n_real=40, seed=5))
    d = gwc.to_device(s, torch.device("cuda:0"))
    d["M_ov"][7, 1, 3] = float("nan")
    shapes = {"sigma_c": (2, 40, 2), "im_sigma_dec": (2, 40), "sigma_c_eps": (2, 2), "sigma_x": (2,), "e_qp": (2,)}
    out = {k: torch.full(v, 7.25, dtype=torch.float64, device="cuda:0") if outputs == "device" else np.full(v, 7.25)
           for k, v in shapes.items()}
    with pytest.raises(gwc.GwcError) as e:
        gwc.gwc_sigma_core(d["eps"], d["occ"], d["M_oo"], d["M_ov"], d["core_idx"], d["omega_imag"], d["w_imag"],
                           d["omega_real"], d["eta"], mode="full", out=out)
    assert e.value.status == -4
    for k, v in out.items():
        assert bool((v == 7.25).all()), k


def _status(s):
    d = gwc.to_device(s, torch.device("cuda:0"))
    with pytest.raises(gwc.GwcError) as e:
        gwc.gwc_sigma_core(d["eps"], d["occ"], d["M_oo"], d["M_ov"], d["core_idx"], d["omega_imag"], d["w_imag"],
                           d["omega_real"], d["eta"], mode="decoupled")
    return e.value.status


def test_order_beyond_the_factorisations(monkeypatch):
    monkeypatch.delenv("GWC_FACTORIZATION", raising=False)
    s = system_from_config(small_config(n_occ=2, n_virt=30, n_aux=12270, n_core=1, n_real=4, seed=5))
    print("case order 12302", flush=True)
    assert _status(s) == -8


def test_budget_below_one_matrix(monkeypatch):
    """8 MB: the reduction would take 5 MB, one bordered matrix of order 1018 takes 17 MB."""
    monkeypatch.delenv("GWC_FACTORIZATION", raising=False)
    monkeypatch.setenv("GWC_BATCH_BYTES", "8000000")
    s = system_from_config(small_config(n_occ=2, n_virt=16, n_aux=1000, n_core=1, n_real=4, seed=5))
    print("case 8 MB", flush=True)
    assert _status(s) == -6
