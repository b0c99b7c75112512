"""Ghost points of a 2D grid, mapped by the stream-collide launches: every face
rule beside every other, on grids narrower than a tile, just beyond one and
with rows outside the last tile, one and two sets, thermal and athermal,
against the oracle; FP64 within 1e-12, FP32 within 1e-5."""
import numpy as np
import pytest

from paper_2102_12559_amd import inputs
from tests.gpu_util import compare_macros, run_pair

pytestmark = pytest.mark.gpu
P, F, Z, W = inputs.BC_PERIODIC, inputs.BC_FIXED_EQ, inputs.BC_OUTFLOW_ZG, inputs.BC_DIFFUSE_WALL


@pytest.mark.parametrize("store,tol", [(inputs.STORE_FP64, 1e-12), (inputs.STORE_FP32, 1e-5)])
@pytest.mark.parametrize("nl,nh,th,nx,ny,bc", [
    (3, 0, 0, 4, 4, [P, P, P, P]),
    (3, 4, 0, 65, 5, [P, P, W, W]),
    (3, 5, 0, 66, 17, [Z, F, P, P]),
    (5, 0, 0, 63, 18, [P, P, W, F]),
    (6, 0, 0, 67, 16, [Z, Z, Z, W]),
    (4, 6, 0, 5, 33, [F, Z, Z, F]),
    (3, 5, 1, 6, 7, [P, P, Z, W]),
    (5, 6, 1, 66, 9, [P, P, P, P]),
    (5, 0, 1, 65, 6, [Z, Z, F, Z]),
])
def test_ghosts_match_oracle(store, tol, nl, nh, th, nx, ny, bc):
    cfg = inputs.base_config(dim=2, nx=nx, ny=ny, nz=1, n_low=nl, n_high=nh, tau=0.7, store=store, thermal=th)
    cfg["bc"] = list(bc) + [P, P]
    for f in range(4):
        cfg["bc_state"][f] = [1.0, 0.03 * (f > 1), 0.02 * (f < 2), 0.0, 1.0]   # a wall moves along itself
    rho, u, T = inputs.smooth_random_flow(nx, ny, 1, umax=0.05, seed=nx + ny)
    mask = np.zeros((1, ny, nx), np.uint8)
    if nh:
        mask[:, : ny // 2, : nx // 2 + 1] = 1
    s, o = run_pair(cfg, rho, u, T, mask, 3, tag=f"ghosts {bc}")
    compare_macros(s, o, tol, 1.0)
