"""GPU parity of gwc_spectral_cumulant at the lengths where its passes and its
phase tables can go wrong: every remainder of log2 n_t by the transform's
radix-16 passes from the smallest length on, n_out up to n_t, and grids of one
to more points than a block of the table.

Tolerance: the suite's 1e-9 of max |A| (the phases' rounding is 1e-13)."""
import numpy as np
import pytest

import paper_2412_17132_amd as gwc
from oracle import cumulant as OC
from workloads import EV_PER_HA

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
TOL = 1e-9

SIZES = [(4, 16, 9), (5, 32, 33), (6, 64, 2), (7, 100, 401), (8, 256, 63), (9, 500, 64), (10, 1024, 65),
         (11, 2048, 129), (12, 1000, 1000), (15, 4000, 257), (17, 5000, 3001)]


@pytest.mark.parametrize("log2_nt,n_out,n_real", SIZES, ids=[f"nt{s[0]}_real{s[2]}" for s in SIZES])
def test_lengths_match_oracle(log2_nt, n_out, n_real):
    rng = np.random.default_rng(log2_nt)
    eps_n, n_t = -10.65, 2 ** log2_nt
    e_qp, eta = eps_n - 0.8, 0.1 / EV_PER_HA
    w = np.linspace(eps_n - 25 / EV_PER_HA, eps_n, n_real)
    im = -0.02 * np.exp(-((w - eps_n + 9 / EV_PER_HA) / 0.05) ** 2) - 0.001 * rng.random(n_real)
    dw = max(60.0 / n_t, 0.01) / EV_PER_HA
    w0 = e_qp - 22 / EV_PER_HA
    print(f"cumulant n_t={n_t} n_out={n_out} n_real={n_real}", flush=True)
    dev = torch.device("cuda:0")
    A, z = gwc.gwc_spectral_cumulant(torch.tensor(w, device=dev), torch.tensor(im, device=dev), eps_n, e_qp, eta,
                                     n_t, dw, n_out, w0)
    torch.cuda.synchronize()
    Ar, Zr, Sr = OC.spectral_cumulant(w, im, eps_n, e_qp, eta, n_t, dw, n_out, w0)
    assert np.max(np.abs(A.cpu().numpy() - Ar)) <= TOL * np.max(np.abs(Ar))
    z = z.cpu().numpy()
    assert abs(z[0] - Zr) <= 1e-12 and abs(z[1] - Sr) <= 1e-12
