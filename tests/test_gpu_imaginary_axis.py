"""GPU parity of calls whose screening runs by Pi builds and LDL^T, where the
imaginary-axis batch takes the kernels without imaginary parts (Pi in every
precision and the trailing update), at N_aux around the 16, 64 and 256 wide
tiles and one to more than LDLT_GROUP panels.

Tolerances: FP64 the suite's 1e-9 of the oracle; the mixed forms their own bars
(1e-3, 1e-4 and 2^-4 of max |Sigma^c|)."""
import numpy as np
import pytest

import paper_2412_17132_amd as gwc
from oracle import sigma as OS
from workloads import system_from_config
from workloads.configs import small_config

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
BAR = {"fp64": 1e-9, "bf16x3": 1e-3, "fp16x3": 1e-4, "fp8": 2.0 ** -4}


@pytest.mark.parametrize("n_aux", [1, 15, 64, 65, 129, 256, 330])
@pytest.mark.parametrize("precision", list(BAR))
def test_imaginary_axis_batches(precision, n_aux, monkeypatch):
    monkeypatch.setenv("GWC_FACTORIZATION", "ldlt")
    print(f"case {precision} N_aux {n_aux}", flush=True)
    s = system_from_config(small_config(n_occ=4, n_virt=17, n_aux=n_aux, n_core=1, n_real=5, seed=n_aux))
    d = gwc.to_device(s, torch.device("cuda:0"))
    out = gwc.gwc_sigma_core(d["eps"], d["occ"], d["M_oo"], d["M_ov"], d["core_idx"], d["omega_imag"],
                             d["w_imag"], d["omega_real"], d["eta"], mode="full", precision=precision)
    torch.cuda.synchronize()
    ref = OS.sigma_core_system(s)["sigma_c"]
    sc = out["sigma_c"].cpu().numpy()
    assert np.max(np.abs(sc[..., 0] + 1j * sc[..., 1] - ref)) <= BAR[precision] * np.max(np.abs(ref))
