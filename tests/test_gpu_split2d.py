"""The thermal FP64 D2Q25 and D2Q36 step, a wave per x node, against the
oracle: both relaxation models, a temperature-dependent viscosity, one and two
rows per workgroup (the latter needs 4096 row tiles; odd ny leaves a row of the
last one outside), two sets.  FP64: 1e-12."""
import numpy as np
import pytest

from paper_2102_12559_amd import inputs
from tests.gpu_util import compare_macros, run_pair

pytestmark = pytest.mark.gpu
P, F, Z, W = inputs.BC_PERIODIC, inputs.BC_FIXED_EQ, inputs.BC_OUTFLOW_ZG, inputs.BC_DIFFUSE_WALL


@pytest.mark.parametrize("nl,nh,nx,ny,bc,extra", [
    (5, 0, 66, 2049, [P, P, W, Z], {}),
    (5, 0, 66, 2047, [Z, F, P, P], {}),
    (5, 0, 65, 2100, [P, P, P, P], dict(tau2=0.9)),
    (5, 0, 4, 5, [P, P, P, P], dict(tau2=0.9)),
    (6, 0, 63, 4, [Z, Z, F, Z], dict(tau2=0.9)),
    (6, 0, 67, 6, [P, P, W, W], dict(tau_mode=1, mu_exp=0.7)),
    (3, 6, 130, 9, [P, P, Z, Z], dict(tau_mode=1, mu_exp=0.7, tau2=0.9)),
])
def test_split_matches_oracle(nl, nh, nx, ny, bc, extra):
    cfg = inputs.base_config(dim=2, nx=nx, ny=ny, nz=1, n_low=nl, n_high=nh, tau=0.7, store=inputs.STORE_FP64,
                             thermal=1, **extra)
    cfg["bc"] = list(bc) + [P, P]
    for f in range(4):
        cfg["bc_state"][f] = [1.0, 0.03 * (f > 1), 0.02 * (f < 2), 0.0, 1.0]
    rho, u, T = inputs.smooth_random_flow(nx, ny, 1, umax=0.05, seed=nx + ny, dT=0.02)
    mask = np.zeros((1, ny, nx), np.uint8)
    if nh:
        mask[:, : ny // 2, : nx // 2 + 1] = 1
    s, o = run_pair(cfg, rho, u, T, mask, 3, tag=f"split {bc} {extra}")
    compare_macros(s, o, 1e-12, 1.0)
