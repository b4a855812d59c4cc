"""Closed-form solve of one-workgroup components and the kernels around it
(csrc/closed.h, csrc/step.h) at the sizes where a lane, a tail capacity or
the LDS runs out: forced and chosen cuts at every workgroup size, batches of
more items than compute units, more lines, groups and switches than a
workgroup holds in registers, switches next to components that need the
general kernel, and components at the LDS limit. Against the CPU oracle
(forward 1e-9 of the largest voltage, gradient 1e-6 per parameter)."""
import dataclasses
import math
import sys

import numpy as np
import pytest

from paper_1903_01081_amd import netgen
from paper_1903_01081_amd.netgen import CAP, CSWITCH, LINE, RES, RL, SRC, SWITCH

pytestmark = pytest.mark.gpu

TOL, GTOL = 1e-9, 1e-6
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


def rel(a, b):
    s = np.max(np.abs(b))
    return float(np.max(np.abs(a - b)) / (s if s > 0 else 1.0))


def grad_err(g, ref, theta):
    a, b = theta * g, theta * ref
    return float(np.max(np.abs(a - b) / np.maximum(np.abs(b), 1e-12 * np.max(np.abs(b)))))


@pytest.mark.parametrize("n_bus,block,tail,kw", [
    (2, 64, -1, {}), (9, 64, -1, {}), (20, 64, 0, {}), (20, 64, 31, {}), (40, 64, 32, {}), (60, 64, -1, {}),
    (9, 256, -1, {}), (33, 256, 33, {}), (65, 256, 64, {}), (100, 256, -1, {}), (20, 256, -1, dict(pack_nodes=256)),
    (9, 512, -1, {}), (129, 512, 128, {}), (150, 512, -1, {}), (60, 512, 63, dict(sweep_from_global=True)),
    (60, 256, -1, dict(serial_adjoint=True)),
])
def test_cuts_and_workgroup_sizes(torch_cuda, oracle_mod, n_bus, block, tail, kw):
    from paper_1903_01081_amd.sim import Simulator
    dt, T, K = 50e-6, 45, 10
    net = netgen.small_grid(n_bus, n_bus, fault_step=23, n_mon=min(30, 3 * n_bus))
    say(f"closed form: {n_bus} buses, block {block}, tail {tail}, {kw}")
    sim = Simulator([net], dt, T, checkpoint_every=K, block_size=block, dense_tail=tail, **kw)
    sim.factor()
    rec = sim.step(T)
    assert rel(rec.cpu().numpy()[0], oracle_mod.run(net, dt, T)) < TOL
    cot = np.random.default_rng(n_bus).standard_normal((1, T, net.n_rec))
    g = sim.adjoint(torch_cuda.tensor(cot, device=sim.device)).cpu().numpy()[0]
    assert grad_err(g, oracle_mod.adjoint(net, dt, T, cot[0]), net.theta0()) < GTOL


def test_more_items_than_compute_units(torch_cuda, oracle_mod):
    # each item may then stage half of a compute unit's LDS only
    from paper_1903_01081_amd.sim import Simulator
    dt, T, K, S = 20e-6, 30, 10, 90
    base = netgen.small_grid(7, 160, fault_step=12, n_mon=20)
    sw = np.where(base.kind == SWITCH)[0]
    nets = []
    for s in range(S):
        k = base.k.copy()
        k[sw] = 3 * s + np.arange(3)
        nets.append(dataclasses.replace(base, k=k))
    say("closed form: 270 items of 160 nodes")
    sim = Simulator(nets, dt, T, checkpoint_every=K)
    sim.factor()
    rec = sim.step(T).cpu().numpy()
    cot = np.random.default_rng(1).standard_normal((S, T, base.n_rec))
    g = sim.adjoint(torch_cuda.tensor(cot, device=sim.device)).cpu().numpy()
    for s in (0, S - 1):
        assert rel(rec[s], oracle_mod.run(nets[s], dt, T)) < TOL
        assert grad_err(g[s], oracle_mod.adjoint(nets[s], dt, T, cot[s]), base.theta0()) < GTOL


@pytest.mark.parametrize("kind", ["lines", "groups"])
def test_more_lines_or_groups_than_registers(torch_cuda, oracle_mod, kind):
    # 64 lanes hold 3 lines and 2 groups each
    from paper_1903_01081_amd.sim import Simulator
    dt, T = 20e-6, 90
    if kind == "lines":
        net = netgen.small_grid(11, 150, fault_step=40, travelling_wave_dt=dt)
        assert np.sum(net.kind == LINE) / 3 > 3 * 64
    else:
        net = netgen.small_grid(11, 50, fault_step=40, coupled=True)
        assert len(np.unique(net.group[net.group >= 0])) > 2 * 64
    say(f"{kind} at 64 lanes")
    sim = Simulator([net], dt, T, block_size=64)
    sim.factor()
    got = np.concatenate([sim.step(n).cpu().numpy()[0] for n in (31, T - 31)])
    assert rel(got, oracle_mod.run(net, dt, T)) < TOL


def bank(n_sw, n_leg, fault_step):
    """n_sw open-loop switches of their own phases (references of 50 Hz
    alone) from a source to n_leg R-C legs, and a switch to ground."""
    br = [dict(k=0, m=-1, kind=SRC, R=1.0, L=1e-4, E=10.0, omega=W60, phase=0.0),
          dict(k=0, m=-1, kind=SWITCH, R=1e-2, ins=0)]
    for j in range(n_leg):
        br += [dict(k=1 + j, m=-1, kind=CAP, C=1e-4), dict(k=1 + j, m=-1, kind=RES, R=20.0)]
    for q in range(n_sw):
        br.append(dict(k=0, m=1 + q % n_leg, kind=CSWITCH, R=0.5 + 0.01 * q, E=1.0, omega=2 * math.pi * 50 * 20,
                       phase=0.37 * q, C=0.1, L=0.3, meas=(-1, -1)))
    return netgen.circuit(1 + n_leg, br, events=[(fault_step, 1, 1)])


@pytest.mark.parametrize("n_sw,n_leg,block", [(70, 7, 64), (1, 1, 64), (130, 63, 64), (70, 33, 256), (140, 127, 512)])
def test_switch_banks(torch_cuda, oracle_mod, n_sw, n_leg, block):
    from paper_1903_01081_amd.sim import Simulator
    dt, T = 20e-6, 150
    net = bank(n_sw, n_leg, 80)
    cs = np.where(net.kind == CSWITCH)[0]
    t = dt * np.arange(1, T + 1)[:, None]
    r = net.E[cs] * np.cos(net.omega[cs] * t + net.phase[cs]) + net.C[cs]
    assert np.min(np.abs(np.abs(r) - net.L[cs])) > 1e-9
    say(f"{n_sw} switches, {n_leg} legs, block {block}")
    sim = Simulator([net], dt, T, block_size=block)
    sim.factor()
    ref = oracle_mod.run(net, dt, T)
    got = np.concatenate([sim.step(n).cpu().numpy()[0] for n in (79, 1, T - 80)])
    sim.sync()
    assert rel(got, ref) < TOL
    sim.reset()
    assert np.array_equal(sim.step(T).cpu().numpy()[0], got)


@pytest.mark.parametrize("other", ["lines", "groups", "levels"])
def test_switches_beside_the_general_kernel(torch_cuda, oracle_mod, other):
    # the components with switches are factorised by levels, in the order that
    # suits levels
    from paper_1903_01081_amd.sim import Simulator
    dt, T = 20e-6, 100
    net = bank(9, 5, 60)
    if other == "lines":
        mate = netgen.small_grid(3, 30, fault_step=40, travelling_wave_dt=dt)
    elif other == "groups":
        mate = netgen.small_grid(3, 12, fault_step=40, coupled=True)
    else:
        mate = bank(140, 140, 60)  # more terminals than the tail takes
    say(f"switches beside {other}")
    sim = Simulator([net, mate], dt, T)
    sim.factor()
    rec = sim.step(T).cpu().numpy()
    sim.sync()
    for s, n in enumerate((net, mate)):
        assert rel(rec[s][:, :n.n_rec], oracle_mod.run(n, dt, T)) < TOL


def test_hub_at_the_lds_limit(torch_cuda, oracle_mod):
    # 7000 one-node clusters around one hub: the closed form's two vectors and
    # the injections exceed the LDS, level passes do not. All leaves with a
    # capacitor move together, the others follow the hub
    from paper_1903_01081_amd.sim import Simulator
    n_leaf, n_cap, dt, T = 7000, 1000, 20e-6, 12
    br = [dict(k=0, m=-1, kind=SRC, R=1.0, L=1e-3, E=10.0, omega=W60, phase=0.0)]
    br += [dict(k=0, m=1 + j, kind=RES, R=50.0) for j in range(n_leaf)]
    br += [dict(k=1 + j, m=-1, kind=CAP, C=1e-7) for j in range(n_cap)]
    net = netgen.circuit(1 + n_leaf, br, rec_nodes=[0, 1, n_cap, n_leaf])
    small = netgen.circuit(2, [br[0], dict(k=0, m=1, kind=RES, R=50.0 / n_cap),
                               dict(k=1, m=-1, kind=CAP, C=1e-7 * n_cap)])
    say("hub of 7001 nodes")
    sim = Simulator([net], dt, T)
    sim.factor()
    got = sim.step(T).cpu().numpy()[0]
    ref = oracle_mod.run(small, dt, T)
    assert rel(got, ref[:, [0, 1, 1, 0]]) < TOL


def test_adjoint_row_beyond_the_lds(torch_cuda):
    # a feeder of 4500 nodes, all recorded: no room in the LDS for the
    # trajectory row. With 30 recorded nodes there is, and the same cotangent
    # gives the same gradient
    from paper_1903_01081_amd.sim import Simulator
    n, dt, T, K = 4500, 20e-6, 9, 4
    rng = np.random.default_rng(2)
    br = [dict(k=0, m=-1, kind=SRC, R=0.5, L=10e-3, E=1.0, omega=W60, phase=0.3)]
    for j in range(n - 1):
        br.append(dict(k=j, m=j + 1, kind=RL, R=rng.uniform(0.1, 0.5), L=rng.uniform(1e-4, 2e-4), line=j))
        if j % 2 == 0:
            br.append(dict(k=j + 1, m=-1, kind=CAP, C=0.5 * rng.uniform(8e-9, 12e-9), line=j))
    few = np.sort(rng.choice(n, 30, replace=False))
    grads = []
    w = rng.standard_normal((T, 30))
    for nodes in (np.arange(n), few):
        net = netgen.circuit(n, br, rec_nodes=nodes.tolist())
        say(f"feeder of {n} nodes, {len(nodes)} recorded")
        sim = Simulator([net], dt, T, checkpoint_every=K)
        sim.factor()
        sim.step(T, record=False)
        cot = np.zeros((1, T, len(nodes)))
        cot[0][:, np.searchsorted(nodes, few)] = w
        grads.append(sim.adjoint(torch_cuda.tensor(cot, device=sim.device)).cpu().numpy()[0])
        sim.close()
    assert np.all(np.isfinite(grads[0])) and np.max(np.abs(grads[0])) > 0
    assert np.max(np.abs(grads[0] - grads[1])) <= 1e-12 * np.max(np.abs(grads[1]))
