"""Steps of 3D grids on the line kernels: every pass of a run of several steps, and both
orders of the linear substep's passes, against the FP64 oracle.

Tolerances: a TS2 step is 6 transforms of some 9 levels and a pointwise stage; roundings of
6e-8 (complex64) add up as their square root, to 2e-7 a step, those of complex128 are
allowed to add up linearly, 6e-15 a step.  For three steps: 2e-6 and 2e-14."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import rel_l2, to_gpu

pytestmark = pytest.mark.gpu

L = (8.0, 9.0, 7.0)
PARAMS = (60.0, -2.0, 3.0, 0.7, 0.9, 1.0, 1.1, 1.3)
TAU = 2e-3
TOL = {"complex128": 2e-14, "complex64": 2e-6}


def state(shape, seed):
    rng = np.random.default_rng(seed)
    ax = [np.exp(-np.linspace(-3.0, 3.0, n, endpoint=False) ** 2) for n in shape]
    g = ax[0][:, None, None] * ax[1][:, None] * ax[2]
    w = rng.standard_normal(5) + 1j * rng.standard_normal(5)
    noise = rng.standard_normal((5,) + shape) + 1j * rng.standard_normal((5,) + shape)
    psi = (w[:, None, None, None] + 0.01 * noise) * g
    return psi / np.sqrt((np.abs(psi) ** 2).sum() * np.prod([2.0 * l / n for l, n in zip(L, shape[::-1])]))


# (nz, ny, nx): three steps at every length of the x-lines; y-lines of 64 to 256 complex64
# points from the number of points that takes their line kernel; one step at the z-lines
# that take it beyond the Infinity Cache only
@pytest.mark.parametrize("dtype,shape,steps", [
    ("complex64", (64, 256, 64), 3), ("complex64", (16, 512, 128), 3), ("complex64", (32, 192, 192), 3),
    ("complex64", (64, 64, 256), 3), ("complex64", (16, 192, 384), 3), ("complex64", (16, 128, 512), 3),
    ("complex64", (16, 128, 768), 3), ("complex64", (384, 16, 192), 3),
    ("complex64", (128, 64, 256), 3), ("complex64", (64, 128, 256), 3), ("complex64", (32, 256, 256), 3),
    ("complex64", (512, 128, 128), 1), ("complex64", (192, 192, 256), 1),
    ("complex128", (64, 128, 64), 3), ("complex128", (16, 256, 128), 3), ("complex128", (16, 128, 256), 3),
    ("complex128", (16, 64, 512), 3), ("complex128", (256, 32, 64), 3),
])
def test_steps_on_line_kernels_in_both_orders(dtype, shape, steps):
    import torch
    from paper_2603_25282_amd.sgp import Solver
    psi0 = state(shape, sum(shape))
    print(f"case {steps} steps on line kernels {shape} {dtype}", flush=True)
    ref = oracle.evolve(psi0, L, PARAMS, 2, TAU, steps, t0=0.1)
    s = Solver(shape, L, PARAMS, dtype=dtype)
    s.build_propagator(TAU, 2)
    for order in (0, 1):
        s.set_plan([0, 0, 0, order])
        psi = to_gpu(s, psi0)
        s.time = 0.1
        s.step(psi, steps)
        torch.cuda.synchronize()
        err = rel_l2(Solver.from_device_layout(psi.cpu().numpy()), ref)
        print(f"  order {order}: rel l2 {err:.2e}", flush=True)
        assert err <= TOL[dtype]


@pytest.mark.parametrize("dtype,shape,slabs", [
    ("complex64", (128, 64, 256), 2), ("complex64", (16, 512, 128), 16), ("complex128", (64, 128, 64), 4),
])
def test_slabs_on_line_kernels_change_nothing(dtype, shape, slabs):
    """z-slabs launch the x- and y-line kernels on parts of the grid that start at plane z0
    (one plane each at 16 slabs): the bits of whole passes."""
    import torch
    from paper_2603_25282_amd.sgp import Solver
    psi0 = state(shape, 3)
    print(f"case {slabs} slabs on line kernels {shape} {dtype}", flush=True)
    out = []
    for n in (0, slabs):
        s = Solver(shape, L, PARAMS, dtype=dtype)
        s.build_propagator(TAU, 4)
        s.set_slabs(n)
        psi = to_gpu(s, psi0)
        s.time = 0.1
        for steps in (4, 6):  # bodies of 3 and 5 steps
            s.step(psi, steps)
        torch.cuda.synchronize()
        out.append(psi)
    assert torch.equal(out[0], out[1])
