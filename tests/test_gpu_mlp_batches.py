"""The network's forward pass and gradients at the edges of their tiles: 16
rows in four waves, 32 a workgroup, 128 workgroups before a workgroup takes a
second group of rows.

Tolerances: a row's outputs do not depend on the batch (bit for bit); loss
and gradients against the bf16-emulating oracle as in test_gpu_mlp.py (1e-4
and 1e-3 of the largest entry per parameter block), where an entry's rounding
differs by the order of at most a few thousand float32 sums."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def params(seed):
    r = np.random.default_rng(seed)
    return np.concatenate([r.normal(0, 0.2, 64 * 34), r.normal(0, 0.1, 64), r.normal(0, 0.15, 64 * 64),
                           r.normal(0, 0.1, 64), r.normal(0, 0.15, 26 * 64), r.normal(0, 0.1, 26)]).astype(np.float32)


@pytest.mark.parametrize("B", [1, 15, 16, 17, 63, 64, 65, 1003])
def test_forward_rows_are_the_batch_of_4096s(B):
    import torch
    from paper_2107_10987_amd.hydro import Hydro, _ptr
    print("case: forward", B, flush=True)
    X = torch.randn((4096, 34), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    hy = Hydro(max_leaves=1)
    try:
        hy.mlp_load(params(2))
        whole = hy.mlp_forward(X)
        out = torch.full((B + 3, 26), 7.0, device="cuda")
        hy._check(hy.L.hydro_mlp_forward(hy.h, _ptr(X), B, _ptr(out), None))
        assert torch.equal(out[:B], whole[:B])
        assert bool((out[B:] == 7.0).all())      # nothing past the batch
        mem = torch.empty(B * 34 + 5, device="cuda")   # outputs over the inputs
        x = mem[:B * 34].view(B, 34).copy_(X[:B])
        y = mem[5:5 + B * 26].view(B, 26)
        hy._check(hy.L.hydro_mlp_forward(hy.h, _ptr(x), B, _ptr(y), None))
        assert torch.equal(y, whole[:B])
    finally:
        hy.close()


@pytest.mark.parametrize("B", [1, 16, 17, 63, 64, 65, 129, 4095, 4097, 8200])
def test_gradients_at_tile_edges(B):
    import torch
    import oracle
    from paper_2107_10987_amd.hydro import Hydro
    print("case: gradient", B, flush=True)
    p = params(3)
    r = np.random.default_rng(B)
    X = r.normal(size=(B, 34)).astype(np.float32)
    T = r.normal(size=(B, 26)).astype(np.float32)
    hy = Hydro(max_leaves=1, mlp_batch=B)
    try:
        hy.mlp_load(p)
        g, loss = hy.mlp_grad(torch.tensor(X, device="cuda"), torch.tensor(T, device="cuda"))
        again, _ = hy.mlp_grad(torch.tensor(X, device="cuda"), torch.tensor(T, device="cuda"))
        assert torch.equal(g, again)
        g, loss = g.cpu().numpy(), float(loss.item())
    finally:
        hy.close()
    lo, go = oracle.mlp_loss_grad(p, X.astype(np.float64), T.astype(np.float64), emulate=True)
    assert abs(loss - lo) <= 1e-4 * lo
    for name, (off, shape) in oracle.MLP_SLICES.items():
        n = int(np.prod(shape))
        d = np.abs(g[off:off + n] - go[off:off + n]).max() / np.abs(go[off:off + n]).max()
        print("grad %s %.1e" % (name, d), flush=True)
        assert d <= 1e-3, name
