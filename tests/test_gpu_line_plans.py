"""Plan widths on 3D grids whose passes run on the line kernels."""
import numpy as np
import pytest

from tests.gpu_util import to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,shape,kept", [
    ("complex64", (16, 512, 128), (0, 1)), ("complex64", (384, 16, 192), (0, 2)),
    ("complex128", (64, 128, 64), (0, 1)), ("complex128", (256, 32, 64), (0, 2)),
])
def test_autotune_keeps_widths_that_the_step_does_not_use(dtype, shape, kept):
    """The tuner times steps, so an axis whose pass has a width of its own keeps the width
    that was set (for the adjoint and the observables), whatever it was."""
    import torch
    from paper_2603_25282_amd.sgp import Solver, plan_widths
    rng = np.random.default_rng(2)
    psi0 = rng.standard_normal((5,) + shape) + 1j * rng.standard_normal((5,) + shape)
    s = Solver(shape, 8.0, (10.0, -1.0, 2.0, 0.5, 1.0, 1.0, 1.1, 1.2), dtype=dtype)
    s.build_propagator(1e-3, 2)
    psi = to_gpu(s, psi0 / np.linalg.norm(psi0))
    allowed = [plan_widths(n, dtype) for n in shape[::-1]]
    for pick in (0, -1):
        want = [w[pick] for w in allowed]
        print(f"case autotune {shape} {dtype} from {want}", flush=True)
        s.set_plan(want)
        widths, ms = s.autotune(psi, 2, steps=2, cache=False)
        assert ms > 0 and widths == s.get_plan()
        for ax in range(3):
            assert widths[ax] == want[ax] if ax in kept else widths[ax] in allowed[ax]
    torch.cuda.synchronize()
