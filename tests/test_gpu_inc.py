"""OP2-style edge-to-cell increment on the GPU against the oracle's loop.

The plan path adds every cell's increments in the loop's own order, so it
must equal the oracle bit for bit. The atomic path adds them in whatever
order the atomics land: each cell with k increments is within
2 k 2^-53 (|cell| + sum |edge|) of the loop's result."""
import numpy as np
import pytest

import oracle
import paper_1302_5586_amd as pf
import synth
from gpu_util import device

pytestmark = pytest.mark.gpu


def _t(a, dev):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to(dev)


def _random_mesh(seed, ncells, nedges):
    rng = np.random.default_rng(seed)
    e2c = rng.integers(0, ncells, (nedges, 2)).astype(np.int32)
    if nedges > 4:
        e2c[1, 1] = e2c[1, 0]          # a self-loop: its cell is incremented twice
        e2c[3] = e2c[2]                # a repeated edge
    return e2c, rng.standard_normal(nedges), rng.standard_normal(ncells)


@pytest.mark.parametrize("ncells,nedges", [(1, 0), (1, 5), (7, 3), (100, 1000), (5000, 12345), (70000, 300000)])
def test_plan_bitwise(ncells, nedges):
    dev = device()
    e2c, edge, cell = _random_mesh(ncells + nedges, ncells, nedges)
    plan = pf.IncPlan(ncells, e2c)
    got = plan.run(_t(edge, dev), _t(cell, dev)).cpu().numpy()
    ref = oracle.edge_inc_f64(ncells, e2c, edge, cell)
    assert np.array_equal(got, ref)
    plan.close()


@pytest.mark.parametrize("ncells,nedges", [(300, 299), (300, 300), (1025, 2500), (64, 5000)])
def test_plan_degrees_bitwise(ncells, nedges):
    """Meshes on both sides of the line between lists and fours, with a cell
    of every number of edges from 0 to 12 among the others, so that the first
    four, the fourth place and the rest behind it all occur."""
    dev = device()
    e2c, edge, cell = _random_mesh(ncells + nedges, ncells, nedges)
    e2c = np.where(e2c < 13, 13 + e2c, e2c)      # cells 0..12 only as set here
    e2c[np.arange(78), 1] = np.repeat(np.arange(13), np.arange(13))
    edge[[2, 3]] = [np.inf, -0.0]
    ref = oracle.edge_inc_f64(ncells, e2c, edge, cell)
    plan = pf.IncPlan(ncells, e2c)
    for _ in range(2):
        got = plan.run(_t(edge, dev), _t(cell, dev)).cpu().numpy()
        assert np.array_equal(got, ref, equal_nan=True)
    plan.close()


@pytest.mark.parametrize("kind,ncells,nedges", [
    ("random", 700001, 1400000), ("random", 4300000, 2700000), ("hub", 700001, 1400000), ("sparse", 700001, 5000000),
    ("few", 1000, 1400000), ("ordered", 900000, 1400000), ("local", 900000, 1400000)])
def test_large_plans_bitwise(kind, ncells, nedges):
    """Meshes above and around the sizes where a plan keeps its visits in
    rounds: a remainder of cells in the last bin, more cells than one sweep
    holds, a cell in very many edges, a bin visited a few times far apart,
    few cells, edges numbered along the cells, and edges shuffled among some
    thousands of neighbours."""
    dev = device()
    e2c, edge, cell = _random_mesh(nedges, ncells, nedges)
    if kind == "hub":
        e2c[::50, 0] = 12345
    elif kind == "sparse":
        e2c = np.maximum(e2c, 256)            # cells below 256 only as set here
        e2c[[7, 2500000, 4999999], 0] = 3
        e2c[4999998] = [255, 3]
    elif kind == "local":
        e2c[:, 0] = np.minimum(np.arange(nedges) * ncells // nedges + e2c[:, 0] % 20000, ncells - 1)
        e2c[:, 1] = np.minimum(np.arange(nedges) * ncells // nedges + e2c[:, 1] % 20000, ncells - 1)
    elif kind == "ordered":
        e2c[:, 0] = np.arange(nedges) * ncells // nedges
        e2c[:, 1] = (e2c[:, 0] + 1) % ncells
    edge[[5, 6]] = [np.inf, -0.0]
    cell[-1] = -0.0
    ref = oracle.edge_inc_f64(ncells, e2c, edge, cell)
    plan = pf.IncPlan(ncells, e2c)
    for _ in range(2):
        got = plan.run(_t(edge, dev), _t(cell, dev)).cpu().numpy()
        assert np.array_equal(got, ref, equal_nan=True)
    plan.close()


def test_plan_mesh_bitwise_and_repeatable():
    dev = device()
    m = synth.config_mesh()
    plan = pf.IncPlan(m.ncells, m.edge_to_cells)
    ed, c0 = _t(m.edge, dev), _t(m.cell, dev)
    c = c0.clone()
    plan.run(ed, c)
    ref = oracle.edge_inc_f64(m.ncells, m.edge_to_cells, m.edge, m.cell)
    assert np.array_equal(c.cpu().numpy(), ref)
    c2 = c0.clone()
    plan.run(ed, c2)
    assert np.array_equal(c2.cpu().numpy(), ref)
    plan.close()


def test_atomic_within_rounding():
    dev = device()
    m = synth.quad_mesh(300, 200, 9)
    got = pf.edge_inc_atomic(_t(m.edge_to_cells.reshape(-1), dev), _t(m.edge, dev), _t(m.cell, dev)).cpu().numpy()
    ref = oracle.edge_inc_f64(m.ncells, m.edge_to_cells, m.edge, m.cell)
    k = np.bincount(m.edge_to_cells.reshape(-1), minlength=m.ncells)
    mag = np.abs(m.cell).copy()
    np.add.at(mag, m.edge_to_cells[:, 0], np.abs(m.edge))
    np.add.at(mag, m.edge_to_cells[:, 1], np.abs(m.edge))
    assert np.all(np.abs(got - ref) <= 2 * np.maximum(k, 1) * 2.0 ** -53 * mag)


def test_atomic_skips_out_of_range_entries():
    dev = device()
    e2c = np.array([[0, 1], [1, 7], [-3, 2]], np.int32)   # 7 and -3 are outside 0..2
    edge = np.array([1.0, 2.0, 4.0])
    cell = np.zeros(3)
    got = pf.edge_inc_atomic(_t(e2c.reshape(-1), dev), _t(edge, dev), _t(cell, dev)).cpu().numpy()
    assert np.array_equal(got, [1.0, 3.0, 4.0])


def test_plan_rejects():
    dev = device()
    with pytest.raises(pf.PFInvalid):
        pf.IncPlan(3, np.array([[0, 3]], np.int32))
    plan = pf.IncPlan(3, np.array([[0, 1]], np.int32))
    import torch
    with pytest.raises(ValueError):
        plan.run(torch.zeros(2, dtype=torch.float64, device=dev), torch.zeros(3, dtype=torch.float64, device=dev))
    x = torch.zeros(8, dtype=torch.float64, device=dev)
    with pytest.raises(pf.PFAlias):
        pf._check(pf.load().pf_inc_plan_run(plan._h, 3, 1, x.data_ptr(), x.data_ptr(), None))
    plan.close()


def test_large_plans_made_at_once():
    """Plans of large random meshes, each made by several threads, made from
    four threads at the same time: every one gives the sequential loop's bits."""
    from concurrent.futures import ThreadPoolExecutor
    dev = device()
    meshes = [_random_mesh(seed, 500000 + 70001 * seed, 1400000) for seed in range(4)]
    ncells = [500000 + 70001 * seed for seed in range(4)]
    with ThreadPoolExecutor(4) as pool:
        plans = list(pool.map(lambda k: pf.IncPlan(ncells[k], meshes[k][0]), range(4)))
    for n, (e2c, edge, cell), plan in zip(ncells, meshes, plans):
        assert np.array_equal(plan.run(_t(edge, dev), _t(cell, dev)).cpu().numpy(), oracle.edge_inc_f64(n, e2c, edge, cell))
        plan.close()


@pytest.mark.parametrize("ncells", [257, 40000])
@pytest.mark.parametrize("fifth", [False, True])
def test_plan_of_four_edges_to_a_cell(ncells, fifth):
    """Every cell in at most four edges, some in fewer and some in none, with
    self-loops and repeated edges, and the same mesh with one cell in a fifth."""
    dev = device()
    rng = np.random.default_rng(ncells)
    ends = rng.permutation(np.repeat(np.arange(1, ncells), 4))[:2 * ncells + 2]
    e2c = ends.reshape(-1, 2).astype(np.int32)
    free = np.flatnonzero(np.bincount(ends, minlength=ncells) == 0)
    e2c[5] = free[1]                # a self-loop
    e2c[7] = e2c[9] = [free[2], free[3]]
    if fifth:
        full = np.flatnonzero(np.bincount(e2c.ravel(), minlength=ncells) == 4)[-1]
        e2c = np.concatenate([e2c, [[full, free[4]]]]).astype(np.int32)
    assert np.bincount(e2c.ravel(), minlength=ncells).max() == (5 if fifth else 4) and len(e2c) >= ncells
    edge, cell = rng.standard_normal(len(e2c)), rng.standard_normal(ncells)
    edge[[2, 3]] = [np.inf, -0.0]
    ref = oracle.edge_inc_f64(ncells, e2c, edge, cell)
    plan = pf.IncPlan(ncells, e2c)
    for _ in range(2):
        assert np.array_equal(plan.run(_t(edge, dev), _t(cell, dev)).cpu().numpy(), ref, equal_nan=True)
    plan.close()
