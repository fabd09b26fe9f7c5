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
