"""Repeated calls of an ensemble of more instances than one launch of its argument kernel
covers: new state buffers, a new clock and another number of steps reach every instance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [64, 65, 130])
@pytest.mark.parametrize("dtype", ["complex128", "complex64"])
def test_second_call_on_new_buffers_equals_unbatched(dtype, n):
    import torch
    from paper_2603_25282_amd.sgp import SGP_OPT_BATCHED, Ensemble
    print(f"case second ensemble call {n} x 64^2 {dtype}", flush=True)
    rng = np.random.default_rng(n)
    p0 = rng.standard_normal((n, 64, 64, 5)) + 1j * rng.standard_normal((n, 64, 64, 5))
    p0 /= np.linalg.norm(p0[0])
    pars = [(100.0 + i, -3.0, 5.0, 0.3 + 0.004 * i, 1.0, 1.0, 1.2, 1.0) for i in range(n)]
    outs = []
    for batched in (1, 0):
        ens = Ensemble([(64, 64)] * n, [8.0] * n, pars, dtype=dtype)
        ens.build_propagator(1e-3, 2)
        ens.set_option(SGP_OPT_BATCHED, batched)
        first = [torch.from_numpy(p).to(ens.torch_dtype).cuda() for p in p0]
        ens.step(first, 3)
        held = [p.clone() for p in first]
        second = [p.clone() for p in first]
        assert abs(ens.time - 3e-3) < 1e-15
        ens.step(second, 4)
        ens.time = 0.4
        ens.step(second, 20)  # replays the step graph
        torch.cuda.synchronize()
        for i in range(n):
            assert torch.equal(first[i], held[i]), f"instance {i}: the first call's buffer was written"
        outs.append(second)
    for i in range(n):
        assert torch.equal(outs[0][i], outs[1][i]), f"instance {i} batched != unbatched"
