"""The rounding of the column walk: the two sides of an interface agree to the
bit where no limiter acts."""
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
