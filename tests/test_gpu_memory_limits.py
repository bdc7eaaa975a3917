"""The reduction beside other holders of the device's memory (each case in a
process of its own, which keeps all memory but the stated rest)."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
pytest.importorskip("torch")
CHILD = os.path.join(os.path.dirname(os.path.abspath(__file__)), "memory_child.py")


def _run(free_mb, n_occ, n_virt, hold):
    env = {k: v for k, v in os.environ.items() if k not in ("GWC_BATCH_BYTES", "GWC_MAX_BATCH")}
    print(f"case {n_occ} x {n_virt}, {free_mb if hold else 'all'} MB free", flush=True)
    p = subprocess.run([sys.executable, CHILD, str(free_mb), str(n_occ), str(n_virt), str(int(hold))], env=env,
                       capture_output=True, text=True, timeout=100)
    assert p.returncode == 0, p.stdout + p.stderr
    w = p.stdout.split("ran", 1)[1].split()
    return dict(reduced=int(w[0]), built=int(w[1]), same=int(w[3]), close=int(w[5]))


def test_route_does_not_depend_on_free_memory():
    """1.3 GB of reduction (order 12000) with 2 GB free, and with all of it."""
    for hold in (False, True):
        assert _run(2000, 24, 500, hold) == dict(reduced=1, built=0, same=0, close=1), hold


def test_no_room_for_the_reduction():
    """3.2 GB of matrix (order 20000) with 2 GB free: the call goes by the Pi builds."""
    assert _run(2000, 20, 1000, True) == dict(reduced=0, built=2, same=1, close=1)
