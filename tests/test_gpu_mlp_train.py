"""Loss and gradient of the closure network at the edges of the training
kernel's tiles (rows below, at and beyond 16 and 64) and for every shape it is
built for, against the same network in FP64 with the operands of each product
rounded to BF16, as the matrix cores take them.  What is left is FP32 summation
and, rarely, an operand whose rounding flips by one BF16 step: 2^-8 of the
gradient's norm, 1e-5 of the loss (squares of outputs near 1)."""
import numpy as np
import pytest

from paper_2102_12559_amd import closure, inputs

pytestmark = pytest.mark.gpu


def reference(p, F, H, O, X, Y):
    import torch
    p, X, Y = (torch.as_tensor(a, dtype=torch.float64) for a in (p, X, Y))
    bf = lambda a: a.to(torch.float32).to(torch.bfloat16).to(torch.float64)
    w1, b1, w2, b2, w3, b3 = p.split([F * H, H, H * H, H, H * O, O])
    w1, w2, w3 = bf(w1.view(F, H)), bf(w2.view(H, H)), bf(w3.view(H, O))
    sg = torch.sigmoid
    z1 = bf(X) @ w1 + b1
    h1 = bf(z1 * sg(z1))
    z2 = h1 @ w2 + b2
    h2 = bf(z2 * sg(z2))
    e = h2 @ w3 + b3 - Y
    dy = 2 * e / e.numel()
    ds = lambda z: sg(z) * (1 + z * (1 - sg(z)))
    d2 = (bf(dy) @ w3.T) * ds(z2)
    d1 = (bf(d2) @ w2.T) * ds(z1)
    g = [bf(X).T @ bf(d1), d1.sum(0), h1.T @ bf(d2), d2.sum(0), h2.T @ bf(dy), dy.sum(0)]
    return float((e * e).mean()), torch.cat([a.reshape(-1) for a in g]).numpy()


@pytest.mark.parametrize("dim,nl,nh,hidden", [(2, 3, 4, 64), (2, 3, 6, 64), (2, 4, 6, 64), (3, 3, 4, 64),
                                              (2, 3, 5, 32), (2, 3, 6, 32), (3, 3, 4, 32)])
def test_gradient_at_tile_edges(dim, nl, nh, hidden):
    import torch
    from paper_2102_12559_amd import msl
    cfg = inputs.base_config(dim=dim, nx=8, ny=8, nz=8 if dim == 3 else 1, n_low=nl, n_high=nh, tau=0.7,
                             lift_mode=inputs.LIFT_MLP, store=inputs.STORE_FP32, mlp_hidden=hidden)
    s = msl.Solver(cfg)
    F, O, H, P = s.mlp_dims()
    rng = np.random.default_rng(nh)
    p = closure.init_params(F, H, O, seed=5).astype(np.float32)
    s.mlp_set_weights(p, np.zeros(F, np.float32), np.ones(F, np.float32), np.zeros(O, np.float32),
                      np.ones(O, np.float32))
    for n in (1, 15, 17, 64, 65, 130, 16384):
        X, Y = (rng.normal(0, 1, (n, k)).astype(np.float32) for k in (F, O))
        l, g = s.mlp_grad(torch.as_tensor(X), torch.as_tensor(Y))
        lr, gr = reference(p, F, H, O, X, Y)
        err = np.linalg.norm(g.cpu().numpy() - gr) / np.linalg.norm(gr)
        print(f"[case] {dim}D {nl}->{nh} H={H} n={n}: loss {abs(l / lr - 1):.1e} gradient {err:.1e}", flush=True)
        assert abs(l / lr - 1) < 1e-5 and err < 2.0 ** -8
    s.close()
