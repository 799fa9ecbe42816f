"""Parameter gradients over the block shapes of the adjoint passes: lines of 16 to 768
points at every plan width, one line per block (few lines) or many, blocks wider than the
grid's columns (16-point lines), blocks of whole wavefronts or not.

One TS2 step in complex128 against the oracle.  A gradient is a sum of at most 2^17 terms of
either sign, each with a few roundings of 1.1e-16: relative errors up to 1e-11 are possible
by cancellation, and 1e-9 is asserted; a lost or doubled partial is 1e-5 or more."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import rel_l2
from tests.test_gpu_adjoint import PIDX

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    (16, 16), (512, 16, 16), (32, 64), (128, 32, 32), (64, 128), (32, 64, 64), (16, 128, 64),
    (192, 16), (16, 64, 192), (384, 64), (16, 768), (512, 256), (16, 512, 16),
])
def test_parameter_gradients_over_block_shapes(shape):
    import torch
    from paper_2603_25282_amd.autograd import evolve
    from paper_2603_25282_amd.sgp import Solver, plan_widths
    params = (60.0, -2.0, 3.0, 0.7, 0.9, 1.0, 1.2, 1.4)
    L, tau = 6.0, 4e-3
    rng = np.random.default_rng(sum(shape))
    co = np.meshgrid(*[np.linspace(-3.0, 3.0, n, endpoint=False) for n in shape], indexing="ij")
    g = np.exp(-sum(c * c for c in co))

    def noise():
        return rng.standard_normal((5,) + shape) + 1j * rng.standard_normal((5,) + shape)

    w5 = rng.standard_normal(5) + 1j * rng.standard_normal(5)
    psi0 = w5.reshape((5,) + (1,) * len(shape)) * g + 0.1 * g * noise()
    psi0 /= np.linalg.norm(psi0) * np.sqrt(np.prod([2.0 * L / n for n in shape]))
    w = noise()
    g_ref, d_ref = oracle.adjoint(psi0, w, L, params, 2, tau, 1, t0=0.3, K=1)
    widths = [plan_widths(n, "complex128") for n in shape[::-1]]
    for k in range(max(len(v) for v in widths)):
        plan = [v[k % len(v)] for v in widths]
        print(f"case parameter gradients {shape} plan {plan}", flush=True)
        p0 = torch.from_numpy(Solver.to_device_layout(psi0)).cuda().requires_grad_(True)
        par = torch.tensor([params[i] for i in PIDX], dtype=torch.float64, requires_grad=True)
        out = evolve(p0, par, shape, L, params[5:8], tau, 1, order=2, K=1, t0=0.3, plan=plan)
        torch.sum((torch.conj(torch.from_numpy(Solver.to_device_layout(w)).cuda()) * out).real).backward()
        eg = rel_l2(Solver.from_device_layout(p0.grad.cpu().numpy()), g_ref)
        ed = np.abs(par.grad.numpy() - d_ref) / np.abs(d_ref)
        print(f"  state grad {eg:.1e}, params {ed}", flush=True)
        assert eg <= 1e-13
        assert np.all(ed <= 1e-9)
