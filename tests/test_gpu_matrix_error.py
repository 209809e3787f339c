"""The matrix-core kernel's error of the complex sum S, against plain FP64.

A term's error: two phases rounded to 24 bits (0.82e-7 rad each, root mean square) and two hardware
sines (0.35e-7 each), 1.26e-7 of the term; its amplitude F A in FP32 (weight, reciprocal, products) about
1e-7; so at most 2.2e-7, with a margin of a third.  Terms' errors are independent, so S is off by
that much of sqrt(sum of the terms' squares).  On top a split of P particles rounds its FP32 sum once for
each 16 of them, at the size that it has by then: 2^-25 sqrt(P / 32) of the same.

What this is to catch: a part that grows with the sum, or one of constant sign, in the matrix
instructions' sums.  Versions that had them were off by up to 2 times (sign, short splits) and 8 times (growth,
long ones) this."""
import numpy as np
import pytest

import paper_1802_03972_amd as rad_pkg
from tests.test_launch_plan import MATRIX, plan
from workloads import SINGLE
from tests.helpers import to_device

pytestmark = pytest.mark.gpu

C_LIGHT = 299792458.0
FIRST = 16          # frequencies from here on: below, the terms may be coherent


@pytest.fixture(scope="module")
def rad():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1802_03972_amd.build import ensure_built
    ensure_built()    # a built library is used as is
    rad_pkg._lib.lib()
    return rad_pkg


def reference(dev, times, dirs, om, shape, L):
    """S[dir][omega][3] and the sum of the terms' squares, in torch FP64."""
    import torch
    f = {k: v.double() for k, v in dev.items()}
    n = f["x"].numel() // len(times)
    t = torch.as_tensor(np.asarray(times, np.float64), device="cuda").repeat_interleave(n)
    r = torch.stack([f["x"], f["y"], f["z"]])
    beta = torch.stack([f["bx"], f["by"], f["bz"]])
    rate = torch.stack([f["dbx"], f["dby"], f["dbz"]])
    om = torch.as_tensor(om, device="cuda")
    g = torch.ones_like(om) if shape == "point" else torch.exp(-(om * L / C_LIGHT) ** 2)
    S = torch.zeros((len(dirs), 3, len(om)), dtype=torch.complex128, device="cuda")
    squares = torch.zeros((len(dirs), len(om)), dtype=torch.float64, device="cuda")
    for d in range(len(dirs)):
        nn = torch.as_tensor(dirs[d], device="cuda")
        D = 1.0 - nn @ beta
        A = ((nn[:, None] - beta) * (nn @ rate) - rate * D) / D ** 2
        turns = (t - (nn @ r) / C_LIGHT) / (2.0 * np.pi)
        for i in range(0, t.numel(), 1 << 15):
            N = f["w"][i:i + (1 << 15), None]
            F = torch.sqrt(N * N * g + N * (1.0 - g))
            ph = turns[i:i + (1 << 15), None] * om
            ph = (ph - torch.floor(ph)) * (2.0 * np.pi)
            a = A[:, i:i + (1 << 15)]
            S[d] += torch.complex(a @ (F * torch.cos(ph)), a @ (F * torch.sin(ph)))
            squares[d] += (a * a).sum(dim=0) @ (F * F)
    return S.permute(0, 2, 1).cpu().numpy(), squares.cpu().numpy()


@pytest.mark.parametrize("n,steps,nx,ny,n_omega,shape,dtype,omega_max", [
    # long splits (8192 particles) of terms that cancel
    (16384, 64, 4, 4, 1024, "point", "f64", 1e20),
    (16384, 32, 8, 4, 512, "gauss", "f32", 1e19),
    # short splits: 32, 48 and 64 particles, one to four times the 16 of a matrix instruction
    (3000, 1, 5, 1, 250, "point", "f32", 1e19),
    (31460, 1, 3, 2, 229, "point", "f64", 1e19),
    (31460, 1, 3, 2, 229, "gauss", "f32", 1e19),
    (43000, 1, 3, 2, 229, "point", "f64", 1e19),
    (24624, 1, 8, 1, 236, "gauss", "f32", 1e19),
    (20000, 1, 4, 2, 700, "point", "f32", 1e19)])
def test_error_of_the_sum(rad, n, steps, nx, ny, n_omega, shape, dtype, omega_max):
    w = SINGLE.scaled(n_particles=n, n_steps=steps, nx_dir=nx, ny_dir=ny, n_omega=n_omega, seed=106, in_dtype=dtype,
                      omega_max=omega_max)
    dev = to_device(w.steps(), dtype)
    g = rad.Grid(w.directions(), 0.0, w.domega, n_omega, shape=shape, shape_len=w.shape_len, dt=w.dt)
    g.push_steps(0.0, steps, dev)
    S, squares = reference(dev, w.times(), w.directions(), np.arange(n_omega) * w.domega, shape, w.shape_len)
    l, = plan(nx * ny, n_omega, n * steps, shape=shape, omega_max=omega_max)
    assert l.kernel == MATRIX
    err = np.sum(np.abs(g.spectrum_complex() - S) ** 2, axis=2)[:, FIRST:] / squares[:, FIRST:]
    tol = np.hypot(2.2e-7, 2.0 ** -25 * np.sqrt(l.per_split / 32.0))
    rms = np.sqrt(err.mean())
    print(f"{n} x {steps}, {nx * ny} x {n_omega} {shape} {dtype}: splits of {l.per_split}, rms {rms:.2e} of {tol:.2e}")
    assert rms <= tol
