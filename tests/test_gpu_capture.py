"""Steps captured into a caller's graph: the first call with a buffer and later ones give the
same launches, and every replay the bits of the eager call from the captured clock."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(64, 64), (16, 32, 32)])
@pytest.mark.parametrize("nsteps", [1, 5, 200])
def test_captured_steps_replay_like_eager_ones(shape, nsteps):
    import torch
    from paper_2603_25282_amd.sgp import Solver
    print(f"case captured steps {shape} x {nsteps}", flush=True)
    rng = np.random.default_rng(5)
    p0 = rng.standard_normal((5,) + shape) + 1j * rng.standard_normal((5,) + shape)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        s = Solver(shape, 8.0, (10.0, -1.0, 2.0, 0.5, 0.8, 1.0, 1.1, 1.2), dtype="complex128", stream=stream)
        s.build_propagator(1e-3, 4)
        start = torch.from_numpy(Solver.to_device_layout(p0 / np.linalg.norm(p0))).cuda()
        want, psi = start.clone(), start.clone()
        s.time = 0.25
        s.step(want, nsteps)
        stream.synchronize()
        graphs = []
        for _ in range(2):  # the first call with the buffer, and one more
            g = torch.cuda.CUDAGraph()
            s.time = 0.25
            with torch.cuda.graph(g, stream=stream):
                s.step(psi, nsteps)
            assert abs(s.time - (0.25 + nsteps * 1e-3)) < 1e-12
            graphs.append(g)
        other = start.clone()
        for rep in range(3):
            for k, g in enumerate(graphs):
                psi.copy_(start)
                g.replay()
                s.step(other, 3)  # the program's own work between replays
                stream.synchronize()
                assert torch.equal(psi, want), f"capture {k}, replay {rep}"


def test_batched_ensemble_steps_refuse_capture():
    import torch
    from paper_2603_25282_amd.sgp import Ensemble, SgpError
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ens = Ensemble([(64, 64)] * 2, [8.0] * 2, [(10.0, -1.0, 2.0, 0.5, 0.8, 1.0, 1.1, 1.2)] * 2,
                       dtype="complex64", stream=stream)
        ens.build_propagator(1e-3, 2)
        psis = [torch.zeros((64, 64, 5), dtype=torch.complex64, device="cuda") for _ in range(2)]
        probe = torch.zeros(4, device="cuda")
        for _ in range(2):  # before and after a step
            stream.synchronize()
            t = ens.time
            with torch.cuda.graph(torch.cuda.CUDAGraph(), stream=stream):
                probe.add_(1.0)
                with pytest.raises(SgpError, match="captured"):
                    ens.step(psis, 3)
            assert ens.time == t
            ens.step(psis, 3)
        stream.synchronize()
