"""Both sets of a small 2D run in one launch: the populations are bit for bit
those of one launch per set (which timed steps keep), for every pair of sets,
storage type and relaxation model, on grids of one tile and of several, and on
both sides of the 2048 workgroups that one launch takes."""
import numpy as np
import pytest

from paper_2102_12559_amd import inputs

pytestmark = pytest.mark.gpu
P, Z, W = inputs.BC_PERIODIC, inputs.BC_OUTFLOW_ZG, inputs.BC_DIFFUSE_WALL


@pytest.mark.parametrize("store", [inputs.STORE_FP64, inputs.STORE_FP32, inputs.STORE_FP16_DEV, inputs.STORE_BF16_DEV])
@pytest.mark.parametrize("nl,nh,th,nx,ny,bc,extra", [
    (3, 4, 0, 64, 64, [P, P, P, P], {}),
    (3, 5, 0, 7, 5, [Z, Z, W, W], dict(tau2=0.9)),
    (3, 6, 0, 70, 33, [P, P, Z, Z], {}),
    (4, 5, 0, 130, 9, [P, P, P, P], {}),
    (4, 6, 0, 65, 30, [Z, Z, Z, Z], dict(tau2=0.9)),
    (5, 6, 0, 40, 12, [P, P, W, W], {}),
    (3, 4, 1, 66, 18, [P, P, W, W], {}),
    (3, 4, 0, 64, 4096, [P, P, P, P], {}),
    (3, 4, 0, 64, 8192, [P, P, P, P], {}),
])
def test_pair_equals_separate_launches(store, nl, nh, th, nx, ny, bc, extra):
    from paper_2102_12559_amd import msl
    cfg = inputs.base_config(dim=2, nx=nx, ny=ny, nz=1, n_low=nl, n_high=nh, tau=0.7, store=store, thermal=th, **extra)
    cfg["bc"] = list(bc) + [P, P]
    rho, u, T = inputs.smooth_random_flow(nx, ny, 1, umax=0.05, seed=nx + ny)
    mask = np.zeros((1, ny, nx), np.uint8)
    mask[:, : ny // 2, : nx // 2 + 1] = 1
    out = []
    for apart in (False, True):
        s = msl.Solver(cfg)
        s.set_mask(mask)
        s.init(rho, u, T)
        s.profile(apart, 1)
        s.step(21)
        out.append([s.get_populations(w, k).cpu().numpy() for w in range(2) for k in range(1 + th)])
        s.profile(False)
        s.close()
    print(f"[case] D2Q{nl * nl} + D2Q{nh * nh} thermal={th} store={store} {nx}x{ny}", flush=True)
    for a, b in zip(*out):
        assert np.array_equal(a, b, equal_nan=True)
