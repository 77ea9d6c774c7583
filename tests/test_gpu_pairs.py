"""Training pairs of leaves whose ghosts are means of finer cells, injected or
linearly prolonged coarser ones, and outflow copies, bit for bit as the oracle
forms them (the targets' FP64 values differ by an ulp at most, which float32
rounding does not show), and the mark of flat rows."""
import numpy as np
import pytest

from paper_2107_10987_amd.workloads import OUTFLOW, PERIODIC, LeafSet

pytestmark = pytest.mark.gpu

GAMMA = 5.0 / 3.0


def two_levels(bc):
    ls = LeafSet((2, 2, 2), (bc,) * 3, (0.0, 0.0, 0.0), 1.0 / 16,
                 [(0, i, j, k) for i in range(2) for j in range(2) for k in range(2)])
    ls.refine(0, (0, 0, 0))
    ls.refine(0, (1, 1, 1))
    return ls.tree()


@pytest.mark.parametrize("bc,prolong", [(PERIODIC, False), (OUTFLOW, False), (OUTFLOW, True)])
def test_pairs_match_oracle(bc, prolong):
    import torch
    import oracle
    from paper_2107_10987_amd.hydro import Hydro
    print("case: pairs, bc", bc, "prolong", prolong, flush=True)
    t = two_levels(bc)
    r = np.random.default_rng(9)
    U = r.uniform(0.5, 2.0, (t.n, 7, 8, 8, 8))
    U[:, 6] = 0.25                     # one flat field
    o = oracle.Oracle(t, GAMMA, 0.0, prolong=prolong)
    P = o.padded(U)
    hy = Hydro(max_leaves=t.n, prolong=prolong)
    try:
        g = hy.grid(t, torch.tensor(U, device="cuda"), 0.0, GAMMA)
        X, T, valid = (v.cpu().numpy() for v in hy.mlp_pairs(g))
    finally:
        hy.close()
    assert valid.reshape(t.n, 512, 7)[:, :, 6].max() == 0 and valid.reshape(t.n, 512, 7)[:, :, :6].min() == 1
    for leaf in r.permutation(t.n)[:8]:
        V = oracle.reconstruct_values(P[leaf])
        for c in np.concatenate([r.permutation(512)[:24], [0, 7, 56, 63, 448, 511]]):
            i, j, k = c & 7, (c >> 3) & 7, c >> 6
            for f in range(7):
                row = (leaf * 512 + c) * 7 + f
                nb, s, x = oracle.mlp_features(P[leaf], i, j, k, f)
                if x is None:
                    assert not X[row, :27].any() and not T[row].any() and X[row, 27 + f] == 1
                    continue
                assert np.array_equal(X[row], x.astype(np.float32))
                cell = (k + 1) * 100 + (j + 1) * 10 + (i + 1)
                assert np.array_equal(T[row], ((V[cell, :, f] - nb[13]) * (1.0 / s)).astype(np.float32))


@pytest.mark.parametrize("x_off,t_off", [(1, 0), (0, 1), (2, 3), (4, 4)])
def test_buffers_of_any_alignment(x_off, t_off):
    import torch
    from paper_2107_10987_amd.hydro import Hydro, _ptr, C
    print("case: pairs, offsets", x_off, t_off, flush=True)
    t = two_levels(PERIODIC)
    n = t.n * 512 * 7
    U = torch.tensor(np.random.default_rng(3).uniform(0.5, 2.0, (t.n, 7, 8, 8, 8)), device="cuda")
    hy = Hydro(max_leaves=t.n)
    try:
        g = hy.grid(t, U, 0.0, GAMMA)
        X, T, valid = hy.mlp_pairs(g)
        mx, mt = (torch.full((n * c + 8,), 7.0, device="cuda") for c in (34, 26))
        v = torch.empty(n, dtype=torch.uint8, device="cuda")
        hy._check(hy.L.hydro_mlp_pairs(hy.h, C.byref(g.c), _ptr(mx[x_off:]), _ptr(mt[t_off:]), _ptr(v)))
    finally:
        hy.close()
    for m, off, whole in ((mx, x_off, X), (mt, t_off, T)):
        k = whole.numel()
        assert torch.equal(m[off:off + k], whole.reshape(-1))
        assert bool((m[:off] == 7.0).all()) and bool((m[off + k:] == 7.0).all())   # nothing beside the rows
    assert torch.equal(v, valid)
