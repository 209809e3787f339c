"""The launches that the library plans for a push (rad_debug_plan: host only, no GPU needed)."""
import ctypes

import numpy as np
import pytest

from paper_1802_03972_amd import _lib
from workloads import block_log_omegas

DP = ctypes.POINTER(ctypes.c_double)
CUS = 256
FIXED, FLEXIBLE, MATRIX = 0, 1, 2


def plan(n_dir, n_omega, n, kind="uniform", shape="cic", tile=None, omega_max=1e19, shape_len=1e-7, cus=CUS):
    th = np.linspace(-0.02, 0.02, n_dir)
    dirs = np.ascontiguousarray(np.stack([th, np.zeros(n_dir), np.sqrt(1.0 - th ** 2)], axis=1))
    om = {"uniform": None, "log": np.geomspace(1e15, omega_max, n_omega),
          "blocks": block_log_omegas(1e15, omega_max, n_omega)}[kind]
    d = _lib.GridDesc(n_dir, dirs.ctypes.data_as(DP), 0.0, omega_max / max(1, n_omega - 1), n_omega, _lib.SHAPES[shape],
                      shape_len, 5e-17, 0, 0, None if om is None else om.ctypes.data_as(DP))
    out = (_lib.DebugLaunch * 64)()
    count = ctypes.c_int32()
    t = None if tile is None else ctypes.byref(_lib.Tile(*tile))
    _lib.check(_lib.lib().rad_debug_plan(ctypes.byref(d), t, cus, n, out, len(out), ctypes.byref(count)))
    assert count.value <= len(out)
    return out[:count.value]


@pytest.mark.parametrize("kind", ["uniform", "log", "blocks"])
@pytest.mark.parametrize("n_dir", [1, 2, 3, 5, 7, 8, 9, 11, 13, 15])
def test_flexible_lds(n_dir, kind):
    """The flexible build's LDS: its table of weights is read 16 bytes at a time, so it starts on
    16 bytes for odd chunks of an odd number of directions too; a chunk fits the staging arrays, and two
    workgroups fit a CU's 160 KB."""
    odd = 0
    for n_omega in [16, 100, 241, 300, 529, 540, 600, 700, 800, 1000, 1024]:
        for n in [1, 37, 333, 1000, 5003, 27 * 512, 50001, 200003]:
            for l in plan(n_dir, n_omega, n, kind):
                if l.kernel != FLEXIBLE:
                    continue
                odd += l.chunk * n_dir % 2
                assert l.weights_at % 16 == 0, (n_omega, n, l.chunk)
                assert l.chunk <= 128 and 2 * l.lds_bytes <= 160 * 1024
    if n_dir in (7, 9, 11, 13, 15):      # the odd chunks that this is about
        assert odd > 0
