"""The 3D column walk at the ends of its columns and under every face rule,
FP32, against the oracle: one and two velocity sets on grids whose z extent is
shorter than, equal to and just beyond a column, whose y extent leaves rows of
a tile outside, with periodic, zero-gradient, fixed and diffuse y and z faces
(ghost rows and slabs mapped by the walk or stored) and periodic or
zero-gradient x faces.  rho, u within the FP32 bar of 1e-5."""
import numpy as np
import pytest

from paper_2102_12559_amd import inputs
from tests.gpu_util import compare_macros, run_pair

pytestmark = pytest.mark.gpu
P, F, Z, W = inputs.BC_PERIODIC, inputs.BC_FIXED_EQ, inputs.BC_OUTFLOW_ZG, inputs.BC_DIFFUSE_WALL


@pytest.mark.parametrize("nh,nx,ny,nz,bc", [
    (0, 67, 5, 4, [P, P, P, P, P, P]),
    (0, 5, 9, 17, [Z, Z, P, P, Z, Z]),
    (0, 66, 6, 9, [P, P, Z, F, P, P]),
    (4, 7, 6, 5, [P, P, P, P, P, P]),
    (4, 9, 5, 8, [P, P, W, W, P, P]),
    (4, 10, 6, 7, [Z, Z, P, P, W, W]),
    (4, 65, 4, 4, [P, P, F, Z, Z, F]),
])
def test_walk_matches_oracle(nh, nx, ny, nz, bc):
    cfg = inputs.base_config(dim=3, nx=nx, ny=ny, nz=nz, n_low=3, n_high=nh, tau=0.7, store=inputs.STORE_FP32)
    cfg["bc"] = list(bc)
    for f in range(6):
        cfg["bc_state"][f] = [1.0, 0.03, 0.02 * (f == 3), 0.01, 1.0]
    rho, u, T = inputs.smooth_random_flow(nx, ny, nz, umax=0.05, seed=nx + nz)
    mask = np.zeros((nz, ny, nx), np.uint8)
    if nh:
        mask[:, : ny // 2, : nx // 2 + 1] = 1
    s, o = run_pair(cfg, rho, u, T, mask, 3, tag=f"walk {bc}")
    compare_macros(s, o, 1e-5, 1.0)


def test_list_launch_equals_small_box():
    """A grid with more columns of the high-order set than the dense launch
    takes (live-column list), uniform along z: every slab holds what the same
    flow gives on a short box, bit for bit."""
    from paper_2102_12559_amd import msl
    nx, ny, out = 5, 6, []
    r2, u2, _ = inputs.smooth_random_flow(nx, ny, 1, umax=0.05, seed=2)
    for nz in (8, 33000):
        cfg = inputs.base_config(dim=3, nx=nx, ny=ny, nz=nz, n_low=3, n_high=4, tau=0.7, store=inputs.STORE_FP16_DEV)
        rho = np.repeat(r2, nz, axis=0)
        u = np.concatenate([np.repeat(u2, nz, axis=1), np.zeros((1, nz, ny, nx))])
        mask = np.zeros((nz, ny, nx), np.uint8)
        mask[:, :2, :3] = 1
        s = msl.Solver(cfg)
        s.set_mask(mask)
        s.init(rho, u, np.ones_like(rho))
        s.step(3)
        out.append([a.cpu().numpy() for a in s.macros()])
        s.close()
    for small, long in zip(out[0], out[1]):
        assert np.array_equal(long, np.broadcast_to(small[..., :1, :, :], long.shape))
