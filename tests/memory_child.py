"""Run by test_gpu_memory_limits.py in a process of its own: holds device memory
down to `free_mb`, then runs one self-energy by the asked route and by the Pi
builds, and prints the launches of both and whether the outputs are equal."""
import os
import sys

import numpy as np
import torch

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import paper_2412_17132_amd as gwc  # noqa: E402
from workloads import system_from_config  # noqa: E402
from workloads.configs import small_config  # noqa: E402


def main():
    free_mb, n_occ, n_virt, hold = (int(x) for x in sys.argv[1:5])
    s = system_from_config(small_config(n_occ=n_occ, n_virt=n_virt, n_aux=40, n_core=1, n_imag=4, n_real=4, seed=3))
    dev = torch.device("cuda:0")
    d = gwc.to_device(s, dev)

    def run(route):
        os.environ["GWC_FACTORIZATION"] = route
        gwc.timing_enable(True)
        out = gwc.gwc_sigma_core(d["eps"], d["occ"], d["M_oo"], d["M_ov"], d["core_idx"], d["omega_imag"], d["w_imag"],
                                 d["omega_real"], d["eta"], mode="decoupled")
        torch.cuda.synchronize()
        ran = [gwc.timing_get(k)["launches"] for k in ("spectral_reduce", "pi_build_f64")]
        gwc.timing_enable(False)
        return {k: v.cpu().numpy() for k, v in out.items() if v is not None}, ran

    held = []
    while hold and torch.cuda.mem_get_info()[0] > (free_mb + 64) * 2 ** 20:  # the first takes other memory back, too
        held.append(torch.empty(torch.cuda.mem_get_info()[0] - free_mb * 2 ** 20, dtype=torch.uint8, device=dev))
    left = torch.cuda.mem_get_info()[0]
    got, ran = run("spectral")
    want, _ = run("ldlt")
    same = all(np.array_equal(got[k], want[k]) for k in want)
    close = all(np.allclose(got[k], want[k], rtol=1e-9, atol=1e-9 * np.max(np.abs(want[k]))) for k in want)
    print("ran", *ran, "same", int(same), "close", int(close), "left", left >> 20, flush=True)


if __name__ == "__main__":
    main()
