"""The rounding of the column walk: the two sides of an interface agree to the
bit where no limiter acts, L(U) is no further from its 80-bit value than a
plain FP64 evaluation, the dual-energy switch decides as it is written, and the
ends of a steep line are the face kernel's."""
from fractions import Fraction

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


def switch_states():
    """Uniform states whose internal energy falls on the other side of
    eta1 E when the kinetic energy is formed with fused multiply-adds: four
    that take tau's pressure as the switch is written, four that do not."""
    def fma(a, b, c):
        return float(Fraction(a) * Fraction(b) + Fraction(c))
    r = np.random.default_rng(4)
    out = {True: [], False: []}
    while min(map(len, out.values())) < 4:
        rho = 2.0 ** int(r.integers(-1, 2))   # 1 / rho exact on both sides
        s = r.uniform(0.5, 2.0, 3)
        rinv = 1.0 / rho
        ek = 0.5 * (s[0] * s[0] + s[1] * s[1] + s[2] * s[2]) * rinv
        E = ek / (1.0 - 1e-3) * (1.0 + 2.0 ** -52 * int(r.integers(-4, 5)))
        fused = fma(-0.5 * rinv, fma(s[2], s[2], fma(s[1], s[1], s[0] * s[0])), E) < 1e-3 * E
        written = E - ek < 1e-3 * E
        if fused != written and len(out[bool(written)]) < 4:
            out[bool(written)].append((rho, *s, E, 1.0, 0.5))
    return out[True] + out[False]


@pytest.mark.parametrize("schedule", ["face", "column", "tiled"])
def test_dual_energy_switch_as_written(schedule):
    """At the threshold the pressure jumps (tau = 1 here, e = 1e-3 E): signal
    speeds as the oracle's, to the sound speed's rounding."""
    import torch
    import oracle
    from paper_2107_10987_amd.hydro import Hydro
    t = uniform_tree((1, 1, 1), (PERIODIC,) * 3, (0.0, 0.0, 0.0), 1.0 / 8)
    o = oracle.Oracle(t, GAMMA, 0.0)
    hy = Hydro(max_leaves=1, schedule=schedule)
    try:
        for k, q in enumerate(switch_states()):
            print("case: state", k, schedule, flush=True)
            U = np.ascontiguousarray(np.broadcast_to(np.array(q)[None, :, None, None, None], (1, 7, 8, 8, 8)))
            a = hy.signal_speed(hy.grid(t, torch.tensor(U, device="cuda"), 0.0, GAMMA)).cpu().numpy()
            assert abs(a[0] - o.signal_speed(U)[0]) <= 1e-12 * a[0], (k, a, o.signal_speed(U))
    finally:
        hy.close()


def test_steep_ends_as_the_face_kernel_forms_them():
    """Energy rising by random factors along x, at rest, density one: a leaf's
    signal speed is the root of the largest end on its upper face, from lines
    that both kernels walk the same way, so it is the same to the bit."""
    import torch
    from paper_2107_10987_amd.hydro import Hydro
    print("case: steep ends", flush=True)
    n = 4096
    t = uniform_tree((n, 1, 1), (PERIODIC,) * 3, (0.0, 0.0, 0.0), 1.0 / 16)
    rise = np.random.default_rng(21).uniform(0.0, 3.0, (8 * n // 32, 32)).cumsum(axis=1) - 20.0   # four leaves each
    cell = np.rint(t.cell_centres()[:, 0] * 16 - 0.5).astype(int)
    e = np.exp(rise.reshape(-1)[cell])
    U = conserved(np.ones_like(e), [0.0 * e] * 3, e, 0.5 * np.ones_like(e))
    speed = []
    for schedule in ("face", "column"):
        hy = Hydro(max_leaves=n, schedule=schedule, centre_only=True)
        try:
            speed.append(hy.signal_speed(hy.grid(t, torch.tensor(U, device="cuda"), 0.0, GAMMA)).cpu().numpy())
        finally:
            hy.close()
    assert np.array_equal(speed[0], speed[1]), np.count_nonzero(speed[0] != speed[1])
