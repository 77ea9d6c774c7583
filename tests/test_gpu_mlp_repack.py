"""An Adam step writes the bf16 weight copies and the inference image of the new
parameters itself: after some steps, every use of the network is bit for bit
that of a handle which loads the stepped parameters."""
import numpy as np
import pytest

from paper_2107_10987_amd.workloads import PERIODIC, LeafSet

pytestmark = pytest.mark.gpu

GAMMA = 5.0 / 3.0


@pytest.mark.parametrize("B,steps", [(1, 1), (65, 2), (4096, 3)])
def test_step_leaves_what_a_load_would(B, steps):
    import torch
    from paper_2107_10987_amd.hydro import Hydro
    print("case: repack", B, steps, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(B)
    X = torch.randn((B, 34), generator=gen, device="cuda")
    T = torch.randn((B, 26), generator=gen, device="cuda")
    p = np.random.default_rng(B).normal(0, 0.15, 8090).astype(np.float32)
    t = LeafSet((2, 1, 1), (PERIODIC,) * 3, (0.0, 0.0, 0.0), 1.0 / 16, [(0, 0, 0, 0), (0, 1, 0, 0)]).tree()
    U = torch.tensor(np.random.default_rng(4).uniform(0.5, 2.0, (t.n, 7, 8, 8, 8)), device="cuda")
    stepped, loaded = (Hydro(max_leaves=t.n, learned=True) for _ in range(2))
    try:
        stepped.mlp_load(p)
        for _ in range(steps):
            stepped.mlp_train_step(X, T, 1e-2)
        q = stepped.mlp_save()
        assert not np.array_equal(q, p)
        loaded.mlp_load(q)
        out = []
        for hy in (stepped, loaded):
            grad, loss = hy.mlp_grad(X, T)
            out.append([hy.mlp_forward(X), grad, loss, *hy.mlp_values(hy.grid(t, U, 0.0, GAMMA), want_y=True)])
        for a, b in zip(*out):
            assert torch.equal(a, b)
    finally:
        stepped.close()
        loaded.close()
