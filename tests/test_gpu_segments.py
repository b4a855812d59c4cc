"""The adjoint with one checkpoint segment's trajectory rows at a time
(segment_rows): its steps run again from the checkpoint, and the gradient is
bitwise that of the rows kept by the forward run, for every kind of solve, both
adjoint kernels, events inside a segment, horizons that are no multiple of the
segment, and components that leave the LDS no room."""
import dataclasses
import math
import sys

import numpy as np
import pytest

from paper_1903_01081_amd import netgen
from paper_1903_01081_amd.netgen import CAP, RL, SRC

pytestmark = pytest.mark.gpu

W60 = 2 * math.pi * 60


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return torch


def feeder(n, rec_nodes):
    rng = np.random.default_rng(2)
    br = [dict(k=0, m=-1, kind=SRC, R=0.5, L=10e-3, E=1.0, omega=W60, phase=0.3)]
    for j in range(n - 1):
        br.append(dict(k=j, m=j + 1, kind=RL, R=rng.uniform(0.1, 0.5), L=rng.uniform(1e-4, 2e-4), line=j))
        if j % 3 == 0:
            br.append(dict(k=j + 1, m=-1, kind=CAP, C=0.5 * rng.uniform(8e-9, 12e-9), line=j))
    return netgen.circuit(n, br, rec_nodes=rec_nodes)


def same_gradient(torch, nets, dt, T, K, oracle=None, **kw):
    from paper_1903_01081_amd.sim import Simulator
    out, size = [], []
    for segment_rows in (False, True):
        sim = Simulator(nets, dt, T, checkpoint_every=K, segment_rows=segment_rows, **kw)
        size.append(sim.info()["device_bytes"])
        sim.factor()
        rec = sim.step(T)
        cot = np.random.default_rng(5).standard_normal((sim.S, T, sim.R))
        grads = [sim.adjoint(torch.tensor(cot, device=sim.device)).cpu().numpy() for _ in range(2)]
        sim.sync()
        assert np.array_equal(grads[0], grads[1])  # the second finds the first one's rows
        out.append((rec.cpu().numpy(), grads[0]))
        sim.close()
    assert size[1] < size[0] or 2 * K >= T
    assert np.max(np.abs(out[0][1])) > 0 and np.all(np.isfinite(out[0][1]))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    if oracle is not None:
        for s, net in enumerate(nets):
            th, ref = net.theta0(), oracle.adjoint(net, dt, T, cot[s][:, :net.n_rec])
            a, b = th * out[1][1][s][:len(th)], th * ref
            assert np.max(np.abs(a - b) / np.maximum(np.abs(b), 1e-12 * np.max(np.abs(b)))) < 1e-6


@pytest.mark.parametrize("serial", [False, True])
@pytest.mark.parametrize("n_bus,T,K,kw", [
    (9, 45, 10, {}), (9, 45, 1, {}), (9, 45, 45, {}), (9, 45, 100, {}), (9, 45, 10, dict(solver="sparse")),
    (40, 45, 10, dict(solver="sparse")), (40, 45, 7, dict(block_size=256)), (20, 45, 10, dict(dense_tail=12)),
    (20, 45, 10, dict(solver="dense")), (150, 45, 10, dict(block_size=512)),
    (40, 45, 10, dict(sweep_from_global=True)), (40, 45, 10, dict(sweep_from_global=True, solver="sparse")),
])
def test_segment_rows(torch_cuda, oracle_mod, n_bus, T, K, kw, serial):
    say(f"segment rows: {n_bus} buses, {T} steps, segments of {K}, {kw}, serial {serial}")
    net = netgen.small_grid(n_bus, n_bus, fault_step=23, n_mon=min(30, 3 * n_bus))
    same_gradient(torch_cuda, [net], 50e-6, T, K, oracle_mod, serial_adjoint=serial, **kw)


@pytest.mark.parametrize("kw", [{}, dict(pack_nodes=256), dict(solver="sparse")])
def test_segment_rows_of_an_uneven_batch(torch_cuda, oracle_mod, kw):
    say(f"segment rows: uneven batch, {kw}")
    nets = [netgen.small_grid(s, n, fault_step=11 + s, n_mon=20) for s, n in enumerate((9, 30, 12, 45))]
    same_gradient(torch_cuda, nets, 50e-6, 40, 9, oracle_mod, **kw)


def test_segment_rows_of_more_items_than_compute_units(torch_cuda):
    base = netgen.small_grid(7, 100, fault_step=12, n_mon=20)
    nets = [dataclasses.replace(base, E=base.E * (1.0 + 0.01 * s)) for s in range(100)]
    say("segment rows: 300 items of 100 nodes")
    same_gradient(torch_cuda, nets, 20e-6, 25, 6)


@pytest.mark.parametrize("n", [4500, 6000])
def test_segment_rows_of_components_that_fill_the_lds(torch_cuda, n):
    # no room for the trajectory row; none for cotangents and EMFs either
    say(f"segment rows: feeder of {n} nodes, all recorded")
    same_gradient(torch_cuda, [feeder(n, list(range(n)))], 20e-6, 9, 4)


def test_segment_rows_of_a_node_in_many_columns(torch_cuda):
    say("segment rows: 16400 columns of one node")
    same_gradient(torch_cuda, [feeder(8, [5] * 16400)], 20e-6, 9, 4)
