"""Networks at the limits of the step kernels' formats and of the LDS. Against
the CPU oracle, a smaller network with the same solution, or the same network
recorded differently."""
import math
import sys

import numpy as np
import pytest

from paper_1903_01081_amd import netgen
from paper_1903_01081_amd.netgen import CAP, DIODE, RES, RL, SRC

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


def rel(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


def feeder(n, seed, rec_nodes, cap_every=2):
    """A radial feeder of n nodes whose sections are pi lines, every
    cap_every-th with its capacitor."""
    rng = np.random.default_rng(seed)
    br = [dict(k=0, m=-1, kind=SRC, R=0.5, L=10e-3, E=1.0, omega=W60, phase=0.3)]
    for j in range(n - 1):
        br.append(dict(k=j, m=j + 1, kind=RL, R=rng.uniform(0.1, 0.5), L=rng.uniform(1e-4, 2e-4), line=j))
        if j % cap_every == 0:
            br.append(dict(k=j + 1, m=-1, kind=CAP, C=0.5 * rng.uniform(8e-9, 12e-9), line=j))
    return netgen.circuit(n, br, rec_nodes=rec_nodes)


def gradient(torch, net, T, K, cot, **kw):
    from paper_1903_01081_amd.sim import Simulator
    sim = Simulator([net], 20e-6, T, checkpoint_every=K, **kw)
    sim.factor()
    sim.step(T, record=False)
    g = sim.adjoint(torch.tensor(cot[None], device=sim.device)).cpu().numpy()[0]
    sim.sync()
    sim.close()
    return g


@pytest.mark.parametrize("n_col,kw", [(16000, {}), (16321, {}), (16400, dict(serial_adjoint=True)), (40000, {})])
def test_one_node_recorded_in_many_columns(torch_cuda, n_col, kw):
    # the node's cotangent is the sum over its columns; the sums' rounding
    # (40000 terms of order one, in two orders) is below 1e-11 of it
    T, K = 9, 4
    cot = 1.0 + np.random.default_rng(1).random((T, n_col))
    say(f"one node in {n_col} columns")
    got = gradient(torch_cuda, feeder(8, 3, [5] * n_col), T, K, cot, **kw)
    ref = gradient(torch_cuda, feeder(8, 3, [5]), T, K, cot.sum(1, keepdims=True))
    assert np.max(np.abs(ref)) > 0 and rel(got, ref) < 1e-10


@pytest.mark.parametrize("n,kw", [(4500, {}), (5800, {}), (6000, {}), (6000, dict(serial_adjoint=True))])
def test_adjoint_of_large_components_with_every_node_recorded(torch_cuda, n, kw):
    # the LDS has no room for the trajectory row and, from about 5820 nodes on,
    # none for the cotangents and EMFs either; with 30 recorded nodes it has,
    # and the same cotangent gives the same gradient (its terms meet in another
    # order: 9 steps of sums of order one, 1e-11 of the largest)
    T, K = 9, 4
    rng = np.random.default_rng(2)
    few = np.sort(rng.choice(n, 30, replace=False))
    w = rng.standard_normal((T, 30))
    cot = np.zeros((T, n))
    cot[:, few] = w
    say(f"feeder of {n} nodes, all recorded, {kw}")
    got = gradient(torch_cuda, feeder(n, 2, list(range(n)), 3), T, K, cot, **kw)
    ref = gradient(torch_cuda, feeder(n, 2, few.tolist(), 3), T, K, w, **kw)
    assert np.all(np.isfinite(ref)) and np.max(np.abs(ref)) > 0 and rel(got, ref) < 1e-11


def hub(n_leaf, n_chain, caps=0):
    """A hub with a source, n_leaf leaves on resistors of 50 ohm and a chain of
    n_chain nodes; the first `caps` leaves have a capacitor."""
    br = [dict(k=0, m=-1, kind=SRC, R=1.0, L=1e-3, E=10.0, omega=W60, phase=0.0)]
    br += [dict(k=j if j else 0, m=j + 1, kind=RES, R=5.0) for j in range(n_chain)]
    br.append(dict(k=n_chain, m=-1, kind=CAP, C=1e-6))
    a = 1 + n_chain
    br += [dict(k=0, m=a + j, kind=RES, R=50.0) for j in range(n_leaf)]
    br += [dict(k=a + j, m=-1, kind=CAP, C=1e-7) for j in range(caps)]
    return a, br


@pytest.mark.parametrize("n_leaf", [5500, 5869, 6100])
def test_hub_with_a_chain_at_the_lds_limit(torch_cuda, oracle_mod, n_leaf):
    # the chain makes level passes dear, so that the closed form is chosen; its
    # vectors fit the LDS with 12 branch slots a lane, and from about 5870
    # nodes on not with the 16 of the kernels without staged factors. Leaves
    # without a capacitor follow the hub
    from paper_1903_01081_amd.sim import Simulator
    n_chain, dt, T = 30, 20e-6, 12
    a, br = hub(n_leaf, n_chain)
    net = netgen.circuit(a + n_leaf, br, rec_nodes=[0, n_chain, a, a + n_leaf - 1])
    small = netgen.circuit(a, hub(0, n_chain)[1], rec_nodes=[0, n_chain])
    say(f"hub with {n_leaf} leaves and a chain")
    sim = Simulator([net], dt, T)
    say(sim.info())
    assert (sim.info()["sweep_levels"] <= 3) == (n_leaf < 5800)
    sim.factor()
    got = sim.step(T).cpu().numpy()[0]
    ref = oracle_mod.run(small, dt, T)
    assert rel(got, ref[:, [0, 1, 0, 0]]) < 1e-9


def rectifier():
    """A half-wave rectifier: a source, a diode, an R-C load."""
    return [dict(k=0, m=-1, kind=SRC, R=0.5, L=1e-3, E=10.0, omega=W60, phase=-1.2),
            dict(k=0, m=1, kind=DIODE, R=1e-2, ins=0), dict(k=1, m=-1, kind=CAP, C=1e-4),
            dict(k=1, m=-1, kind=RES, R=20.0), dict(k=0, m=-1, kind=RES, R=1e3)]


@pytest.mark.parametrize("what", ["plain", "diode"])
def test_staged_batch_that_fills_the_lds(torch_cuda, what):
    # as many recorded columns as the LDS of a compute unit takes beside the
    # rest of a batch that goes by level passes
    from paper_1903_01081_amd.sim import Simulator
    T = 300

    def build(n_col):
        net = feeder(8, 3, [5] * n_col) if what == "plain" else netgen.circuit(2, rectifier(), rec_nodes=[1] * n_col)
        return Simulator([net], 20e-6, T, solver="sparse")

    sim = build(30000)
    info = sim.info()
    assert info["lds_staged"]
    sim.close()
    for n_col in range(30000 + (info["lds_limit"] - info["lds_bytes"]) // 4, 30000, -4):
        sim = build(n_col)
        if sim.info()["lds_staged"]:
            break
        sim.close()
    assert sim.info()["lds_bytes"] > info["lds_limit"] - 64
    say(f"{what}: {n_col} columns, {sim.info()['lds_bytes']} bytes of LDS")
    sim.factor()
    got = sim.step(T).cpu().numpy()[0]
    sim.sync()
    sim.close()
    one = build(1)
    one.factor()
    ref = one.step(T).cpu().numpy()[0]
    assert np.max(np.abs(ref)) > 0 and np.array_equal(got, np.repeat(ref, n_col, axis=1))


def test_diode_grid_stays_staged(torch_cuda, oracle_mod):
    # 640 nodes with 20 diode bridges, refactorised by levels inside the loop:
    # the factor and its structure stay in the LDS, where only the node CSR has
    # no room beside them
    from paper_1903_01081_amd.sim import Simulator
    T = 60
    nets, cfg = netgen.config1(seed=3, n_bus=200, n_steps=T, fault_step=30, rectifiers=20)
    say("20 diode bridges, sparse solver")
    sim = Simulator(nets, cfg["dt"], T, solver="sparse")
    assert sim.info()["lds_staged"]
    sim.factor()
    got = sim.step(T).cpu().numpy()[0]
    sim.sync()
    assert rel(got, oracle_mod.run(nets[0], cfg["dt"], T)) < 1e-9


def floating(n, r_ground):
    """A ring of n nodes, driven by a source between two of them, tied to the
    ground and to a grounded source through r_ground alone."""
    rng = np.random.default_rng(0)
    br = [dict(k=0, m=-1, kind=SRC, R=1.0, L=1e-3, E=1.0, omega=W60, phase=0.2), dict(k=1, m=0, kind=RL, R=1.0, L=1e-3)]
    for j in range(n):
        br.append(dict(k=2 + j, m=2 + (j + 1) % n, kind=RL, R=float(rng.uniform(0.1, 1)), L=1e-3))
        if j % 3 == 0:
            br.append(dict(k=2 + j, m=2 + (j + 7) % n, kind=RES, R=float(rng.uniform(5, 20))))
    br.append(dict(k=2, m=2 + n // 2, kind=SRC, R=0.5, L=1e-3, E=2.0, omega=W60, phase=0.5))
    br += [dict(k=5, m=-1, kind=RES, R=r_ground), dict(k=1, m=7, kind=RES, R=r_ground)]
    return netgen.circuit(2 + n, br)


@pytest.mark.parametrize("n", [12, 40, 150])
def test_no_tail_keeps_differences_of_a_floating_part(torch_cuda, oracle_mod, n):
    # triangular sweeps lose digits of the part's common voltage (1e9 ohm over
    # 1 ohm) but not of the differences inside it
    from paper_1903_01081_amd.sim import Simulator
    T, net = 200, floating(n, 1e9)
    say(f"floating ring of {n} nodes, no dense tail")
    sim = Simulator([net], 20e-6, T, dense_tail=0)
    sim.factor()
    got = sim.step(T).cpu().numpy()[0]
    ref = oracle_mod.run(net, 20e-6, T)
    assert rel(got[:, 2:] - got[:, 2:3], ref[:, 2:] - ref[:, 2:3]) < 1e-10


@pytest.mark.parametrize("n_bus,device", [(40, dict(rectifiers=2)), (30, dict(rectifiers=1)), (60, dict(rectifiers=4))])
def test_cut_of_components_with_diode_bridges(torch_cuda, oracle_mod, n_bus, device):
    # the tail is factorised anew in most steps: it is not the whole component
    from paper_1903_01081_amd.sim import Simulator
    T = 400
    nets, cfg = netgen.config1(seed=3, n_bus=n_bus, n_steps=T, fault_step=200, **device)
    say(f"{n_bus} buses, {device}")
    sim = Simulator(nets, cfg["dt"], T)
    assert sim.info()["sweep_levels"] <= 3 and 0 < sim.info()["max_tail"] <= 64
    sim.factor()
    got = sim.step(T).cpu().numpy()[0]
    sim.sync()
    assert rel(got, oracle_mod.run(nets[0], cfg["dt"], T)) < 1e-9


def test_forward_only_batch_is_staged_by_its_own_size(torch_cuda, oracle_mod):
    # 1000-node components, every node recorded, by level passes: the forward
    # kernel's arrays fit the LDS, an adjoint's would not, and without
    # checkpoints there is none
    from paper_1903_01081_amd.sim import Simulator
    T = 40
    net = netgen.small_grid(1, 1000, fault_step=20)
    say("1000 buses, all recorded, level passes around a 128-node tail")
    sim = Simulator([net], 20e-6, T, block_size=512, dense_tail=128)
    assert sim.info()["lds_staged"]
    sim.factor()
    assert rel(sim.step(T).cpu().numpy()[0], oracle_mod.run(net, 20e-6, T)) < 1e-9


@pytest.mark.parametrize("what,closed", [
    ("9 buses", True), ("100 buses", True), ("400 buses", True), ("sparse", False), ("no tail", False),
    ("coupled", True), ("lines", True), ("choppers", True), ("bridges", True), ("1200 buses", False),
])
def test_routes(torch_cuda, what, closed):
    # at most three solve phases in closed form, one per level otherwise
    from paper_1903_01081_amd.sim import Simulator
    kw = dict(sparse=dict(solver="sparse")).get(what, dict(dense_tail=0) if what == "no tail" else {})
    if what in ("choppers", "bridges"):
        net = netgen.config1(seed=3, n_bus=100, n_steps=10, fault_step=5,
                             **{dict(choppers="choppers", bridges="rectifiers")[what]: 4})[0][0]
    elif what == "coupled":
        net = netgen.small_grid(1, 100, coupled=True)
    elif what == "lines":
        net = netgen.small_grid(1, 300, travelling_wave_dt=20e-6)
    else:
        net = netgen.small_grid(1, int(what.split()[0]) if what[0].isdigit() else 60)
    say(f"route of {what}")
    sim = Simulator([net], 20e-6, 10, **kw)
    assert (sim.info()["sweep_levels"] <= 3) == closed
