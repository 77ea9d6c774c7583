"""The rounding of the column walk: the two sides of an interface agree to the
bit where no limiter acts, and L(U) is no further from its 80-bit value than a
plain FP64 evaluation."""
import numpy as np
import pytest

from paper_2107_10987_amd.workloads import OUTFLOW, PERIODIC, uniform_tree

pytestmark = pytest.mark.gpu

GAMMA = 5.0 / 3.0


def conserved(rho, v, e, X):
    return np.ascontiguousarray(np.stack([rho, rho * v[0], rho * v[1], rho * v[2],
                                          e + 0.5 * rho * sum(x * x for x in v), e ** (1 / GAMMA), X], axis=1))


@pytest.mark.parametrize("schedule", ["column", "tiled"])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_contact_at_rest_stays_to_the_bit(axis, schedule):
    """Smooth monotone density and species at rest under one pressure: where
    the constraint does not act, both sides of a face reconstruct the same
    value, the jump is exactly zero, and so is every flux but the pressure's.
    The time step is so long that an ulp's jump would show."""
    import torch
    from paper_2107_10987_amd.hydro import Hydro
    print("case: contact along", axis, schedule, flush=True)
    t = uniform_tree((2, 2, 2), (OUTFLOW,) * 3, (0.0, 0.0, 0.0), 1.0 / 16)
    x = t.cell_centres()[:, axis]
    rho = np.exp(1.7 * x)
    one = np.ones_like(rho)
    U = conserved(rho, [0.0 * one] * 3, 0.37 * one, rho * (0.3 + 0.11 * x))
    hy = Hydro(max_leaves=t.n, schedule=schedule)
    try:
        g = hy.grid(t, torch.tensor(U, device="cuda"), 0.0, GAMMA)
        out = torch.empty_like(g.U)
        hy.stage(g, 1, 2.0 ** 30, g.U, None, out, None)
        got = out.cpu().numpy()
    finally:
        hy.close()
    inner = (x > 3.0 / 16) & (x < 13.0 / 16)   # the outflow boundary's kink does not reach these
    for f in range(7):
        assert np.array_equal(got[:, f][inner], U[:, f][inner]), f


def flow(kind, t):
    x, y, z = np.moveaxis(t.cell_centres(), 1, 0)
    if kind == "transonic":
        rho = 1.0 + 0.3 * np.sin(6.3 * x + 0.4) * np.cos(6.3 * y)
        v = [np.sin(6.3 * y + 1.0), np.sin(6.3 * z + 2.0), np.cos(6.3 * x + 0.2)]
        return conserved(rho, v, 0.9 * (1.0 + 0.3 * np.sin(6.3 * z + x)), rho * (0.5 + 0.2 * np.sin(6.3 * x + y)))
    s = (0.7 * x + 0.5 * y + 0.3 * z) if kind == "star" else x
    rho = np.exp(-1.9 * s * s - 0.8 * s)
    if kind == "star":     # slow against its sound speed
        v = [1e-3 * np.sin(3.0 * y), 1e-3 * np.sin(2.0 * z + 1.0), 1e-3 * np.cos(2.5 * x)]
    else:
        v = [1e-3 + 0.0 * x, 5e-4 + 0.0 * x, 2e-4 + 0.0 * x]
    return conserved(rho, v, 0.45 * rho ** GAMMA, rho * (0.5 + 0.1 * s))


@pytest.mark.parametrize("kind,nb,limit", [("planar", (32, 1, 1), 2.0), ("star", (2, 2, 2), 1.4),
                                           ("transonic", (2, 2, 2), 1.4)])
def test_rounding_error_of_the_rhs(kind, nb, limit):
    """Mean error of L(U) per field against 80 bits, by a stage with a time
    step so long that the state it starts from is lost in the result, over the
    cells that no boundary reaches.  The oracle rounds every operation to
    nearest; the walk fuses some and takes 1 / rho and the root, which enter
    through the velocities and the speed, within an ulp instead of half of one:
    its error may be a third larger where those are most of it (1.4), and along
    a plane wave of 250 different cells, whose sums largely vanish, the two
    means scatter (2)."""
    import torch
    import oracle
    from oracle import wide
    from paper_2107_10987_amd.hydro import Hydro
    print("case:", kind, flush=True)
    across = PERIODIC if kind == "planar" else OUTFLOW
    t = uniform_tree(nb, (OUTFLOW, across, across), (0.0, 0.0, 0.0), 1.0 / (8 * nb[0]))
    U = flow(kind, t)
    dt = 2.0 ** 30
    o = oracle.Oracle(t, GAMMA, 0.0)
    exact = U + np.longdouble(dt) * wide.rhs(o.padded(U), t.dx, t.origin, GAMMA)
    plain, _ = o.stage(1, dt, U)
    hy = Hydro(max_leaves=t.n, schedule="column")
    try:
        g = hy.grid(t, torch.tensor(U, device="cuda"), 0.0, GAMMA)
        out = torch.empty_like(g.U)
        hy.stage(g, 1, dt, g.U, None, out, None)
        got = out.cpu().numpy()
    finally:
        hy.close()
    c = t.cell_centres() / t.dx[0]
    inner = np.all([(c[:, a] > 3) & (c[:, a] < 8 * nb[a] - 3) for a in range(3) if nb[a] > 1], axis=0)
    err = [np.array([np.abs((a - exact) / dt)[:, f][inner].mean() for f in range(7)], np.float64) for a in (got, plain)]
    print("mean error against the oracle's:", np.array2string(err[0] / err[1], precision=2), flush=True)
    assert np.all(err[0] <= limit * err[1]), err
