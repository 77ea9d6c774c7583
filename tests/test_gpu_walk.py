"""The column walk's reconstruction and flux where their case distinctions
sit: rough states (the constraint's every case, extrema on every line),
plateaus and exact ties, and a NaN next to a cell, which must reach the flux.

Tolerance: the parity bounds of tests/parity.py (1e-12 per field and per
element): each value is formed from at most a few hundred operations on
operands of the local scale."""
import numpy as np
import pytest

from parity import check
from paper_2107_10987_amd.workloads import PERIODIC, uniform_tree

pytestmark = pytest.mark.gpu

GAMMA = 5.0 / 3.0


def state(kind, n, seed):
    r = np.random.default_rng(seed)
    shape = (n, 8, 8, 8)
    if kind in ("rough", "pressureless"):   # every cell its own value
        draw = lambda lo, hi: r.uniform(lo, hi, shape)  # noqa: E731
    elif kind == "ties":         # few distinct values: equal neighbours, equal differences
        draw = lambda lo, hi: lo + (hi - lo) * r.integers(0, 3, shape) / 2.0  # noqa: E731
    else:                        # steps between plateaus
        draw = lambda lo, hi: np.where(r.integers(0, 2, (n, 2, 2, 2)).repeat(4, 1).repeat(4, 2).repeat(4, 3) > 0, lo, hi)  # noqa: E731
    rho = draw(1.0, 3.0)
    v = [draw(-0.5, 0.5) for _ in range(3)]
    e = draw(1.0, 2.0)
    U = np.stack([rho, rho * v[0], rho * v[1], rho * v[2], e + 0.5 * rho * sum(x * x for x in v), e ** (1 / GAMMA),
                  rho * draw(0.0, 1.0)], axis=1)
    if kind == "pressureless":   # e = 0 and tau = 0: the sound speed is the root of zero
        U[:, 4] -= e
        U[:, 5] = 0.0
    return np.ascontiguousarray(U)


@pytest.mark.parametrize("kind", ["rough", "ties", "plateaus", "pressureless"])
def test_walk_against_oracle(kind):
    import torch
    import oracle
    from paper_2107_10987_amd.hydro import Hydro
    t = uniform_tree((3, 2, 2), (PERIODIC,) * 3, (-0.2, 0.1, 0.0), 1.0 / 16)
    U = state(kind, t.n, 11)
    print("case:", kind, flush=True)
    o = oracle.Oracle(t, GAMMA, 0.3)
    hy = Hydro(max_leaves=t.n, schedule="column")
    try:
        g = hy.grid(t, torch.tensor(U, device="cuda"), 0.3, GAMMA)
        dt = 0.2 * o.dt(U)
        want, a = o.stage(1, dt, U)
        out = torch.empty_like(g.U)
        am = torch.zeros(t.n, dtype=torch.float64, device="cuda")
        hy.stage(g, 1, dt, g.U, None, out, am)
        assert np.abs(am.cpu().numpy() - a).max() <= 1e-12 * a.max()
        check(out.cpu().numpy(), want, o, U, label=kind)
    finally:
        hy.close()


@pytest.mark.parametrize("cell", [(-1, 3, 3), (8, 0, 7), (2, -1, 5), (4, 4, 8), (-1, -1, 3), (8, 2, -1), (8, 8, 8),
                                  (-1, 8, -1)])
def test_nan_beside_a_cell_is_reported(cell):
    """A ghost cell without a value (a prolongation row that does not exist)
    is NaN; it touches an interior cell by a face, an edge or a corner."""
    import torch
    from paper_2107_10987_amd import hydro
    t = uniform_tree((1, 1, 1), (PERIODIC,) * 3, (0.0, 0.0, 0.0), 1.0 / 8)
    U = state("rough", 1, 3)
    print("case: NaN at", cell, flush=True)
    gm = hydro.ghost_map(t).copy()
    slot = 0
    for k in range(-3, 11):
        for j in range(-3, 11):
            for i in range(-3, 11):
                if 0 <= i < 8 and 0 <= j < 8 and 0 <= k < 8:
                    continue
                if (i, j, k) == cell:
                    gm[0, slot] = -(1 << 30) - 1
                slot += 1
    hy = hydro.Hydro(max_leaves=1, schedule="column")
    try:
        g = hy.grid(t, torch.tensor(U, device="cuda"), 0.0, GAMMA, gmap=gm)
        with pytest.raises(hydro.HydroError) as e:
            hy.step(g, 1e-4)
        assert e.value.code == hydro.ENONPHYS
    finally:
        hy.close()


def test_nan_spreads_as_in_the_oracle():
    """One stage on a state with two NaN cells: the same cells and fields go
    bad (a slope that has a NaN two cells off is finite, with a sign that the
    NaN's own sign bit gives, so the values beside them are nobody's)."""
    import torch
    import oracle
    from paper_2107_10987_amd.hydro import Hydro
    print("case: two NaN cells", flush=True)
    t = uniform_tree((2, 2, 2), (PERIODIC,) * 3, (0.0, 0.0, 0.0), 1.0 / 16)
    U = state("rough", t.n, 17)
    U[1, 0, 3, 4, 5] = np.nan
    U[6, 5, 0, 7, 0] = np.nan
    o = oracle.Oracle(t, GAMMA, 0.0)
    want, _ = o.stage(1, 1e-3, U)
    hy = Hydro(max_leaves=t.n, schedule="column")
    try:
        g = hy.grid(t, torch.tensor(U, device="cuda"), 0.0, GAMMA)
        out = torch.empty_like(g.U)
        hy.stage(g, 1, 1e-3, g.U, None, out, None)
        got = out.cpu().numpy()
        bad = np.isnan(want)
        assert bad.any() and not bad.all()
        assert np.array_equal(bad, np.isnan(got))
        with pytest.raises(Exception):
            hy.check()
    finally:
        hy.close()


@pytest.mark.parametrize("kind", ["rough", "ties", "plateaus"])
def test_face_centre_scheme_against_oracle(kind):
    """One point per face with weight one: the face-normal line alone."""
    import torch
    import oracle
    from paper_2107_10987_amd.hydro import Hydro
    t = uniform_tree((3, 2, 2), (PERIODIC,) * 3, (-0.2, 0.1, 0.0), 1.0 / 16)
    U = state(kind, t.n, 13)
    print("case: face centres,", kind, flush=True)
    o = oracle.Oracle(t, GAMMA, 0.3, centre_only=True)
    hy = Hydro(max_leaves=t.n, schedule="column", centre_only=True)
    try:
        g = hy.grid(t, torch.tensor(U, device="cuda"), 0.3, GAMMA)
        dt = 0.2 * o.dt(U)
        want, a = o.stage(1, dt, U)
        out = torch.empty_like(g.U)
        am = torch.zeros(t.n, dtype=torch.float64, device="cuda")
        hy.stage(g, 1, dt, g.U, None, out, am)
        assert np.abs(am.cpu().numpy() - a).max() <= 1e-12 * a.max()
        check(out.cpu().numpy(), want, o, U, label=kind)
    finally:
        hy.close()


@pytest.mark.parametrize("scale", [2.0 ** 100, 2.0 ** -100])
def test_huge_and_tiny_values_against_oracle(scale):
    """The scheme is homogeneous in the conserved fields (the entropy tracer by
    its own exponent), so a state times 2^100 or 2^-100, its tracer to match,
    gives that times the result and the same speeds: checked against the
    oracle at unit scale."""
    import torch
    import oracle
    from paper_2107_10987_amd.hydro import Hydro
    t = uniform_tree((2, 2, 1), (PERIODIC,) * 3, (0.0, 0.0, 0.0), 1.0 / 16)
    U = state("rough", t.n, 19)
    print("case: scale", scale, flush=True)
    factor = np.full(7, scale)
    factor[5] = scale ** (1 / GAMMA)
    o = oracle.Oracle(t, GAMMA, 0.3)
    dt = 0.2 * o.dt(U)
    want, a = o.stage(1, dt, U)
    f = factor[None, :, None, None, None]
    hy = Hydro(max_leaves=t.n, schedule="column")
    try:
        g = hy.grid(t, torch.tensor(U * f, device="cuda"), 0.3, GAMMA)
        out = torch.empty_like(g.U)
        am = torch.zeros(t.n, dtype=torch.float64, device="cuda")
        hy.stage(g, 1, dt, g.U, None, out, am)
        assert np.abs(am.cpu().numpy() - a).max() <= 1e-12 * a.max()
        check(out.cpu().numpy() / f, want, o, U, label="scale")
    finally:
        hy.close()
