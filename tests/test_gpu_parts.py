"""Leaves done in parts by several workgroups (small launches, and the last
round of large ones) against whole leaves, bit for bit: the same columns are
walked by the same code and summed in the same order, whoever does them.
Sizes at the edges of the rule's ranges on 256 compute units; each launch
runs twice, so that its counters are seen to be left at zero."""
import numpy as np
import pytest

from paper_2107_10987_amd.workloads import PERIODIC, LeafSet, uniform_tree

pytestmark = pytest.mark.gpu

GAMMA = 5.0 / 3.0
OMEGA = 0.005   # at most 1.3 at the end of a row of 513 leaves, with the time step well inside the CFL limit


def rough(n, edge=8, seed=5):
    r = np.random.default_rng(seed)
    shape = (n, edge, edge, edge)
    rho = r.uniform(1.0, 3.0, shape)
    v = [r.uniform(-0.5, 0.5, shape) for _ in range(3)]
    e = r.uniform(1.0, 2.0, shape)
    return np.ascontiguousarray(np.stack([rho, rho * v[0], rho * v[1], rho * v[2],
                                          e + 0.5 * rho * sum(x * x for x in v), e ** (1 / GAMMA),
                                          rho * r.uniform(0.0, 1.0, shape)], axis=1))


def two_steps(tree, U, schedule, **opts):
    import torch
    from paper_2107_10987_amd.hydro import Hydro
    hy = Hydro(max_leaves=tree.n, schedule=schedule, leaf_edge=tree.leaf_edge, **opts)
    try:
        g = hy.grid(tree, torch.tensor(U, device="cuda"), OMEGA, GAMMA)
        a = [hy.step(g, 2e-3) for _ in range(2)]
        return g.U.cpu().numpy(), np.stack(a)
    finally:
        hy.close()


@pytest.mark.parametrize("n", [1, 2, 32, 33, 64, 65, 85, 86, 128, 129, 257, 288, 384, 385, 513])
def test_parts_equal_whole_leaves(n):
    print("case: parts,", n, "leaves", flush=True)
    t = uniform_tree((n, 1, 1), (PERIODIC,) * 3, (0.0, 0.0, 0.0), 1.0 / 16)
    U = rough(n)
    whole = two_steps(t, U, "persistent")
    for schedule in ("auto", "tiled"):
        got = two_steps(t, U, schedule)
        assert np.array_equal(whole[0], got[0]) and np.array_equal(whole[1], got[1]), schedule


@pytest.mark.parametrize("edge,opts", [(16, dict()), (8, dict(rk_order=3)), (8, dict(centre_only=True)),
                                       (8, dict(reflux=True))])
def test_parts_with_options(edge, opts):
    print("case: parts,", edge, opts, flush=True)
    t = uniform_tree((3, 2, 1), (PERIODIC,) * 3, (0.0, 0.0, 0.0), 1.0 / 32, leaf_edge=edge)
    U = rough(t.n, edge)
    whole = two_steps(t, U, "persistent", **opts)
    got = two_steps(t, U, "auto", **opts)
    assert np.array_equal(whole[0], got[0]) and np.array_equal(whole[1], got[1])


def test_parts_in_a_graph():
    """Replays of captured steps, with eager work between them."""
    import torch
    from paper_2107_10987_amd.hydro import Hydro
    print("case: parts in a graph, 45 leaves", flush=True)
    t = uniform_tree((45, 1, 1), (PERIODIC,) * 3, (0.0, 0.0, 0.0), 1.0 / 16)
    U0 = torch.tensor(rough(45), device="cuda")
    s = torch.cuda.Stream()
    eager, graph = Hydro(max_leaves=45, schedule="persistent"), Hydro(max_leaves=45)
    try:
        ge = eager.grid(t, U0.clone(), OMEGA, GAMMA, stream=s)
        gg = graph.grid(t, U0.clone(), OMEGA, GAMMA, stream=s)
        de, dg = (torch.full((1,), 1e-3, dtype=torch.float64, device="cuda") for _ in range(2))
        torch.cuda.synchronize()
        graph.graph_capture(gg, 0.3, dg, 2)
        for _ in range(3):
            graph.graph_launch(s)
            for _ in range(2):
                eager.step_dev(ge, 0.3, de)
            torch.cuda.synchronize()
            assert torch.equal(ge.U, gg.U) and torch.equal(de, dg)
    finally:
        eager.close()
        graph.close()


@pytest.mark.parametrize("n,per", [(96, 48), (128, 32), (60, 3), (300, 38)])
def test_parts_in_launches_side_by_side(n, per):
    """Launches that share the chip are split by what runs beside them."""
    import torch
    from paper_2107_10987_amd.hydro import Hydro
    print("case: parts in launches,", n, "in", per, flush=True)
    t = uniform_tree((n, 1, 1), (PERIODIC,) * 3, (0.0, 0.0, 0.0), 1.0 / 16)
    U = rough(n)
    whole = two_steps(t, U, "persistent")
    hy = Hydro(max_leaves=n)
    try:
        g = hy.grid(t, torch.tensor(U, device="cuda"), OMEGA, GAMMA, launch_off=list(range(0, n, per)) + [n])
        a = np.stack([hy.step(g, 2e-3) for _ in range(2)])
        assert np.array_equal(whole[0], g.U.cpu().numpy()) and np.array_equal(whole[1], a)
    finally:
        hy.close()


def refined(nb, corners):
    ls = LeafSet((nb,) * 3, (PERIODIC,) * 3, (0.0, 0.0, 0.0), 1.0 / (8 * nb),
                 [(0, i, j, k) for i in range(nb) for j in range(nb) for k in range(nb)])
    for c in corners:
        ls.refine(0, c)
    return ls.tree()


def wavy(tree):
    x, y, z = np.moveaxis(2 * np.pi * tree.cell_centres(), 1, 0)
    # (a jump of 12 in density: the learned path's cells there fall back)
    rho = (1.0 + 0.4 * np.sin(x + 0.3) * np.cos(2 * y)) * np.where(x + y < 4.0, 12.0, 1.0)
    v = [0.4 * np.sin(y + z), 0.3 * np.cos(x + 0.1) * np.sin(z), 0.3 * np.sin(2 * x + y)]
    e = 1.5 + 0.4 * np.cos(z + x)
    return np.ascontiguousarray(np.stack([rho, rho * v[0], rho * v[1], rho * v[2],
                                          e + 0.5 * rho * sum(q * q for q in v), e ** (1 / GAMMA),
                                          rho * (0.5 + 0.3 * np.sin(x + y + z))], axis=1))


# 22 leaves in 8 parts, 120 in 2, 258 as a whole round and two leaves in 8
REFINED = [(2, [(0, 0, 0), (1, 1, 1)]), (4, [(i, j, k) for i in (0, 2) for j in (0, 2) for k in (0, 2)]),
           (6, [(0, 0, 0), (2, 2, 0), (4, 4, 0), (0, 2, 3), (2, 4, 3), (4, 0, 3)])]


@pytest.mark.parametrize("opts", [dict(reflux=True), dict(prolong=True), dict(learned=True),
                                  dict(reflux=True, prolong=True, learned=True)],
                         ids=lambda o: "+".join(o))
@pytest.mark.parametrize("nb,corners", REFINED, ids=["22", "120", "258"])
def test_parts_on_refined_meshes(nb, corners, opts):
    """Coarse/fine faces corrected, prolonged ghosts and learned values."""
    import torch
    from paper_2107_10987_amd.hydro import Hydro
    t = refined(nb, corners)
    print("case: parts,", t.n, "leaves", opts, flush=True)
    U = torch.tensor(wavy(t), device="cuda")
    out = []
    for schedule in ("persistent", "auto"):
        hy = Hydro(max_leaves=t.n, schedule=schedule, **opts)
        try:
            if hy.learned:
                hy.mlp_load(np.random.default_rng(3).normal(0.0, 0.15, 8090))
            g = hy.grid(t, U.clone(), OMEGA, GAMMA)
            assert not hy.reflux or g.n_reflux > 0
            assert not hy.prolong or g.ptable is not None
            a = [hy.step(g, 1e-3) for _ in range(2)]
            if hy.learned:
                cells, fallback = hy.mlp_stats()
                assert 0 < fallback < cells
            out.append((g.U.cpu().numpy(), np.stack(a)))
        finally:
            hy.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
