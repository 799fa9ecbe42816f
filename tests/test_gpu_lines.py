"""Line kernels (a point's five components in one thread), the passes of an ensemble
partition large enough for them, and step graphs over several state buffers.

Tolerances: against the FP64 oracle those of the parity tests (relative l2 1e-11 for
complex128, 5e-5 for complex64, the targets for 1000 steps); batched against unbatched
and graph against direct launches bitwise, since every path does the same operations
in the same order."""
import numpy as np
import pytest

import oracle
from paper_2603_25282_amd import inputs as I
from tests.gpu_util import rel_l2, run_gpu, to_gpu

pytestmark = pytest.mark.gpu

TOL = {"complex128": 1e-11, "complex64": 5e-5}


# (nz, ny, nx), chosen so that every length with a line kernel is run along every axis,
# at the smallest number of points that takes them (2^19 complex128, 2^20 complex64) or
# just above, and 256-point z-lines also where their plan changes (2^23 points).
@pytest.mark.parametrize("dtype,shape", [
    ("complex128", (64, 64, 128)), ("complex128", (16, 512, 64)), ("complex128", (512, 16, 64)),
    ("complex128", (256, 128, 16)), ("complex128", (64, 16, 512)), ("complex128", (128, 16, 256)),
    ("complex128", (128, 256, 16)), ("complex128", (32, 64, 256)),
    ("complex64", (128, 64, 128)), ("complex64", (64, 128, 192)), ("complex64", (256, 16, 256)),
    ("complex64", (32, 512, 64)), ("complex64", (512, 32, 64)), ("complex64", (384, 192, 16)),
    ("complex64", (16, 384, 192)), ("complex64", (16, 192, 384)), ("complex64", (768, 16, 128)),
    ("complex64", (16, 768, 128)), ("complex64", (16, 128, 768)), ("complex64", (32, 64, 512)),
    ("complex64", (32, 256, 128)), ("complex64", (256, 256, 128)),
])
def test_line_kernels_against_the_oracle(dtype, shape):
    L = (8.0, 9.0, 7.0)
    params = (500.0, -5.0, 10.0, 0.9, 1.0, 1.0, 1.1, 1.3)
    rng = np.random.default_rng(sum(shape))
    co = np.meshgrid(*[np.linspace(-3.0, 3.0, n, endpoint=False) for n in shape], indexing="ij")
    g = np.exp(-sum(c * c for c in co))
    w = rng.standard_normal(5) + 1j * rng.standard_normal(5)
    psi0 = w[:, None, None, None] * g + 0.01 * g * (rng.standard_normal((5,) + shape)
                                                   + 1j * rng.standard_normal((5,) + shape))
    psi0 /= np.sqrt((np.abs(psi0) ** 2).sum() * np.prod([2.0 * l / n for l, n in zip(L, shape[::-1])]))
    print(f"case line kernels {shape} {dtype}", flush=True)
    ref = oracle.evolve(psi0, L, params, 2, 1e-3, 1)
    got, _ = run_gpu(shape, L, params, psi0, 2, 1e-3, 1, dtype=dtype)
    err = rel_l2(got, ref)
    print("rel l2", err)
    assert err <= TOL[dtype]


# Partitions just above the number of points that takes line kernels, of one or two
# lengths (the second one's last block is the smallest).
@pytest.mark.parametrize("dtype,plan,sizes", [
    ("complex64", 4, [256] * 16 + [128]), ("complex64", 4, [256] * 15 + [128] * 5),
    ("complex64", 12, [384] * 8 + [192]), ("complex64", 12, [768] * 2 + [384]),
    ("complex128", 4, [256] * 8 + [128]), ("complex128", 4, [128] * 33),
])
def test_ensemble_on_line_kernels_equals_unbatched(dtype, plan, sizes):
    import torch
    from paper_2603_25282_amd.sgp import SGP_OPT_BATCHED, Ensemble, Solver
    sizes = sizes + [64]  # beside the partition, an instance of another width
    psis, outs = [], []
    for i, n in enumerate(sizes):
        c = I.with_(I.C1, shape=(n, n), seed=40 + i, name=f"line-{i}")
        psis.append(Solver.to_device_layout(I.initial_state(c)))
    print(f"case ensemble {dtype} E={plan} {sizes}", flush=True)
    for batched in (1, 0):
        ens = Ensemble([(n, n) for n in sizes], [8.0] * len(sizes),
                       [(100.0 + i, -3.0, 5.0, 0.5, 1.0, 1.0, 1.0, 1.0) for i in range(len(sizes))], dtype=dtype)
        for n in sorted(set(sizes)):
            for ax in (0, 1):
                ens.set_plan(n, ax, 8 if n == 64 else plan)
        ens.build_propagator(1e-3, 2)
        ens.set_option(SGP_OPT_BATCHED, batched)
        st = [torch.from_numpy(p).to(ens.torch_dtype).cuda().contiguous() for p in psis]
        ens.step(st, 3)
        torch.cuda.synchronize()
        outs.append([p.cpu().numpy() for p in st])
    for i, n in enumerate(sizes):
        assert np.array_equal(outs[0][i], outs[1][i]), f"instance {i} ({n}^2) batched != unbatched"


@pytest.mark.parametrize("dtype", ["complex128", "complex64"])
@pytest.mark.parametrize("shape", [(16, 16), (128, 64), (16, 32, 32)])
def test_step_graphs_over_new_and_alternating_buffers(dtype, shape):
    """The first call on a buffer, a repeated one and calls alternating between buffers
    (with other lengths between) give the bits of the same calls launched directly."""
    import torch
    from paper_2603_25282_amd.sgp import Solver
    rng = np.random.default_rng(3)
    p0 = [rng.standard_normal((5,) + shape) + 1j * rng.standard_normal((5,) + shape) for _ in range(3)]
    s = Solver(shape, 8.0, (10.0, -1.0, 2.0, 0.5, 1.0, 1.0, 1.1, 1.2), dtype=dtype)
    s.build_propagator(1e-3, 4)

    def run(order, lens):
        bufs = [to_gpu(s, p / np.linalg.norm(p)) for p in p0]
        for b, n in zip(order, lens):
            s.time = 0.25
            s.step(bufs[b], n)
        torch.cuda.synchronize()
        return [b.cpu().numpy() for b in bufs]

    order, lens = [0, 0, 1, 2, 1, 0, 2, 2, 1], [17, 17, 17, 5, 5, 1, 40, 17, 130]
    s.set_graph(False)
    want = run(order, lens)
    s.set_graph(True)
    for rep in range(2):
        got = run(order, lens)
        for b in range(3):
            assert np.array_equal(got[b], want[b]), f"buffer {b}, repetition {rep}"
