"""The flat shapes (256 consecutive sites per block, csrc/flat.h) at the
extents where their division and wraps can go wrong, against the 64 x 4 tile:
extents of one, blocks that end inside a row, rows shorter and longer than a
block; single steps, pairs and leftovers; and batches of such boxes."""

import numpy as np
import pytest
import torch

import flb_workloads as W
from helpers import gpu_params

pytestmark = pytest.mark.gpu

KW = dict(rho0=1.0, kT=1e-4, rate_bulk=1.2, rate_shear=1.6, rate_ghost=0.9, seed=5)
BOXES = [("D3Q19", n) for n in [(1, 1, 1), (1, 1, 300), (1, 7, 40), (9, 1, 31), (300, 1, 1), (17, 16, 1),
                                (255, 2, 3), (256, 3, 2), (257, 5, 3), (33, 20, 7), (64, 4, 4)]]
BOXES += [("D2Q9", n) for n in [(1, 700, 1), (1000, 600, 1), (999, 601, 1)]]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("lattice,n", BOXES)
def test_flat_shapes_same_bits(lattice, n, precision):
    from paper_1012_3632_amd import Simulation
    p = gpu_params(lattice=lattice, precision=precision, nx=n[0], ny=n[1], nz=n[2], **KW)
    drho = W.initial_drho((n[2], n[1], n[0]), 9, 0.01)
    ref = Simulation(p, drho_init=drho)
    ref.set_launch(0)
    flat = [c for c in range(ref.launch_configs()[0]) if ref.launch_shape(c)[7] == 3]
    assert len(flat) == 2
    tol = 1e-12 if precision == "fp64" else 5e-6   # of FP32 sums over other rows, as for every shape
    counts = ((1, 1), (4, 1), (3, 2), (2, 0))
    for k, stride in counts:
        ref.step(k, stats_stride=stride)
    s0, q0, n0 = ref.moments()
    for cfg in flat:
        sim = Simulation(p, drho_init=drho)
        sim.set_launch(cfg)
        for k, stride in counts:
            sim.step(k, stats_stride=stride)
        assert torch.equal(sim.state(), ref.state()), cfg
        s1, q1, n1 = sim.moments()
        assert n1 == n0
        np.testing.assert_allclose(q1, q0, rtol=tol, atol=0)
        assert np.all(np.abs(s1 - s0) <= tol * np.sqrt(n0 * np.prod(n) * q0) + 1e-300)


def test_batch_of_thin_boxes():
    """Replicas with an extent of one advance as single runs do."""
    from paper_1012_3632_amd import Batch, Simulation
    dims = [(1, 9, 5), (9, 1, 5), (1, 1, 17), (5, 9, 1), (12, 1, 1)]
    kw = {k: v for k, v in KW.items() if k != "seed"}
    b = Batch(gpu_params(lattice="D3Q19", precision="fp32", **kw), dims, seeds=range(5))
    b.step(5)
    for r, n in enumerate(dims):
        one = Simulation(gpu_params(lattice="D3Q19", precision="fp32", nx=n[0], ny=n[1], nz=n[2],
                                    seed=r, replica=r, **kw))
        one.set_launch(0)
        one.step(5)
        assert torch.equal(b.replica_state(r), one.state()), n


FORCE_BOXES = [(1, 1, 1), (1, 1, 300), (1, 7, 40), (9, 1, 31), (300, 1, 1), (17, 16, 1), (255, 2, 3),
               (256, 3, 2), (257, 5, 3), (2, 2, 2), (33, 20, 7), (64, 4, 4),
               (64, 64, 32), (64, 64, 33)]   # the last box of one launch for both fields, the first of two


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n", FORCE_BOXES)
def test_flat_force_shape(n, precision):
    """The flat D3Q19 force shape (density, chemical potential and step as
    three launches) against the 32 x 4 x 2 tile, with eta zero and one."""
    from paper_1012_3632_amd import Simulation
    tol = 1e-12 if precision == "fp64" else 5e-6   # as for every force shape against another
    for eta in (0, 1):
        p = gpu_params(lattice="D3Q19", precision=precision, nx=n[0], ny=n[1], nz=n[2], eta=eta,
                       force_model=1, a=-0.01, b=0.1, rho_c=1.0, kappa=0.05, **dict(KW, kT=1e-6))
        drho = W.initial_drho((n[2], n[1], n[0]), 9, 0.01)
        sims = {}
        for cfg in (0, 12):
            sim = sims[cfg] = Simulation(p, drho_init=drho)
            sim.set_launch(cfg)
            for k, stride in ((1, 1), (4, 1), (3, 2), (2, 0)):
                sim.step(k, stats_stride=stride)
        assert sims[12].launch_shape(12)[7] == 3
        a, b = sims[12].state().double(), sims[0].state().double()
        assert float((a - b).abs().max()) <= tol * float(b.abs().max())
        s0, q0, n0 = sims[0].moments()
        s1, q1, n1 = sims[12].moments()
        assert n1 == n0
        # modes that a thin box leaves at rounding level have no scale of their own
        assert np.all(np.abs(q1 - q0) <= 20 * tol * q0.max())
        assert np.all(np.abs(s1 - s0) <= 20 * tol * np.sqrt(n0 * np.prod(n) * q0.max()))


@pytest.mark.parametrize("n", [(24, 30, 20), (101, 77, 53)])   # one launch for both fields, two
def test_flat_force_graph_replays(n):
    """Captured flat force steps replayed three times = eager calls, bit for bit."""
    from paper_1012_3632_amd import Simulation
    p = gpu_params(lattice="D3Q19", precision="fp32", nx=n[0], ny=n[1], nz=n[2], eta=1, force_model=1,
                   a=-0.01, b=0.1, rho_c=1.0, kappa=0.05, **dict(KW, kT=1e-6))
    drho = W.initial_drho((n[2], n[1], n[0]), 9, 0.01)
    eager, graph = (Simulation(p, drho_init=drho) for _ in range(2))
    assert eager.launch_shape(eager.launch_configs()[1][1])[7] == 3   # the untuned shape
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        graph.graph_capture(4, stats_stride=1, stream=stream)
    for _ in range(3):
        eager.step(4, stats_stride=1)
        with torch.cuda.stream(stream):
            graph.graph_launch(stream)
        torch.cuda.synchronize()
        assert torch.equal(eager.state(), graph.state())
    for a, b in zip(eager.moments(), graph.moments()):
        assert np.array_equal(a, b)


# the largest boxes of the flat shapes: populations (record count and plane
# offsets) just below 2^32 bytes, (V - 1) nx or (V / nx - 1) ny (the division by
# a reciprocal) just below 2^32, and one box past each limit, which runs the
# row tile
LARGEST = [("D3Q19", "fp32", (76, 743, 1000), True), ("D3Q19", "fp64", (152, 304, 611), True),
           ("D3Q19", "fp32", (256, 256, 256), True), ("D3Q19", "fp32", (16384, 16, 1), True),
           ("D3Q19", "fp64", (1, 256, 65536), True), ("D2Q9", "fp64", (256, 65535, 1), True),
           ("D3Q19", "fp32", (76, 744, 1000), False), ("D3Q19", "fp64", (16385, 16, 1), False)]


def _fits(lattice, precision, n):
    V, Q, rb = n[0] * n[1] * n[2], 19 if lattice == "D3Q19" else 9, 4 if precision == "fp32" else 8
    return Q * V * rb < 2 ** 32 and (V - 1) * n[0] < 2 ** 32 and (V // n[0] - 1) * n[1] < 2 ** 32


@pytest.mark.parametrize("lattice,precision,n,fits", LARGEST)
def test_flat_shapes_at_their_limits(lattice, precision, n, fits):
    """A pair and a lone step of both flat shapes against the 32 x 8 tile."""
    from paper_1012_3632_amd import Simulation
    assert _fits(lattice, precision, n) == fits
    p = gpu_params(lattice=lattice, precision=precision, nx=n[0], ny=n[1], nz=n[2], **KW)
    ref, sim = Simulation(p), Simulation(p)
    ref.set_launch(3)
    for cfg in (15, 16):
        sim.set_launch(cfg)
        for s in (ref, sim):
            s.step(3, stats_stride=1)
        for a, b in zip(sim.state(), ref.state()):   # plane by plane
            assert torch.equal(a, b), cfg
    (s0, q0, n0), (s1, q1, n1) = ref.moments(), sim.moments()
    assert n0 == n1 == 6
    tol = 1e-12 if precision == "fp64" else 5e-6   # of FP32 sums over other rows, as for every shape
    np.testing.assert_allclose(q1, q0, rtol=tol, atol=0)
    assert np.all(np.abs(s1 - s0) <= tol * np.sqrt(n0 * np.prod(n) * q0) + 1e-300)


@pytest.mark.parametrize("precision,n,fits", [c[1:] for c in LARGEST if c[0] == "D3Q19"])
def test_flat_force_at_its_limits(precision, n, fits):
    """The same for the force step (against the 32 x 4 x 2 tile)."""
    from paper_1012_3632_amd import Simulation
    tol = 1e-12 if precision == "fp64" else 5e-6   # as for every force shape against another
    p = gpu_params(lattice="D3Q19", precision=precision, nx=n[0], ny=n[1], nz=n[2], eta=1,
                   force_model=1, a=-0.01, b=0.1, rho_c=1.0, kappa=0.05, **KW)
    ref, sim = Simulation(p), Simulation(p)   # the noise makes the density
    ref.set_launch(0)
    sim.set_launch(12)
    for s in (ref, sim):
        s.step(3)
    for a, b in zip(sim.state(), ref.state()):
        assert float((a - b).abs().max()) <= tol * float(b.abs().max())


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_forward_steps_beside_a_recompute(precision):
    """Forward steps of the default (flat) force shape on one stream while a
    reverse pass of the same handle recomputes its segments on others: both
    give what they give alone, bit for bit."""
    from paper_1012_3632_amd import Simulation
    n, every, nsteps = (48, 40, 36), 4, 16
    p = gpu_params(lattice="D3Q19", precision=precision, nx=n[0], ny=n[1], nz=n[2], eta=1,
                   force_model=1, a=-0.01, b=0.1, rho_c=1.0, kappa=0.05, **dict(KW, kT=1e-6))
    sim = Simulation(p, drho_init=W.initial_drho(n[::-1], 9, 0.01))
    assert sim.launch_shape(sim.launch_configs()[1][0])[7] == 3
    ckpts = []
    for _ in range(0, nsteps, every):
        ckpts.append(sim.state().clone())
        sim.step(every)
    start = sim.state().clone()
    g = torch.Generator(device="cuda").manual_seed(3)
    seed = torch.randn(start.shape, generator=g, device="cuda", dtype=torch.float64).to(start.dtype)
    want = seed.clone()
    work = sim.adjoint_run(ckpts, want, every, nsteps)
    sim.step(40)
    end = sim.state().clone()
    torch.cuda.synchronize()
    fwd, rev = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(3):
        got = seed.clone()
        sim.load_state(start)
        sim.seek(nsteps)
        torch.cuda.synchronize()
        sim.step(20, stream=fwd)
        sim.adjoint_run(ckpts, got, every, nsteps, work=work, stream=rev)
        sim.step(20, stream=fwd)
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        assert torch.equal(sim.state(), end)
