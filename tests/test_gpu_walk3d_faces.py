"""The 3D walks where test_gpu_walk3d.py does not take them, against the oracle:
columns of eight cells with a short last one (enough columns along z that the
launch keeps eight), in every storage type that walks; and the face rules in
16-bit storage, whose walk maps ghost rows and slabs by itself.  FP32 within
its bar of 1e-5, 16-bit deviations within the storage bar of 2e-3."""
import numpy as np
import pytest

from paper_2102_12559_amd import inputs
from tests.gpu_util import compare_macros, run_pair

pytestmark = pytest.mark.gpu
P, F, Z, W = inputs.BC_PERIODIC, inputs.BC_FIXED_EQ, inputs.BC_OUTFLOW_ZG, inputs.BC_DIFFUSE_WALL
BAR = {inputs.STORE_FP32: 1e-5, inputs.STORE_FP16_DEV: 2e-3, inputs.STORE_BF16_DEV: 2e-3}


def _run(store, nh, nx, ny, nz, bc, steps):
    cfg = inputs.base_config(dim=3, nx=nx, ny=ny, nz=nz, n_low=3, n_high=nh, tau=0.7, store=store)
    cfg["bc"] = list(bc)
    for f in range(6):
        cfg["bc_state"][f] = [1.0, 0.03, 0.02 * (f == 3), 0.01, 1.0]
    rho, u, T = inputs.smooth_random_flow(nx, ny, nz, umax=0.05, seed=nx + nz)
    mask = np.zeros((nz, ny, nx), np.uint8)
    if nh:
        mask[:, : ny // 2, : nx // 2 + 1] = 1
    s, o = run_pair(cfg, rho, u, T, mask, steps, tag=f"walk {bc}")
    compare_macros(s, o, BAR[store], 1.0)


@pytest.mark.parametrize("store", BAR)
@pytest.mark.parametrize("nh,nx,ny,nz,bc", [
    (4, 5, 6, 1029, [P, P, P, P, P, P]),      # 2 columns a slab: 258 of eight, the last of five cells
    (0, 66, 5, 513, [P, P, Z, F, Z, F]),      # 4 columns a slab: 260, the last of one cell
])
def test_short_last_column_of_eight(store, nh, nx, ny, nz, bc):
    _run(store, nh, nx, ny, nz, bc, 2)


@pytest.mark.parametrize("store", [inputs.STORE_FP16_DEV, inputs.STORE_BF16_DEV])
@pytest.mark.parametrize("nh,nx,ny,nz,bc", [
    (0, 67, 5, 4, [P, P, P, P, P, P]),
    (0, 5, 9, 17, [Z, Z, P, P, Z, Z]),
    (0, 66, 6, 9, [P, P, Z, F, P, P]),
    (4, 9, 5, 8, [P, P, W, W, P, P]),
    (4, 10, 6, 7, [Z, Z, P, P, W, W]),
    (4, 65, 4, 4, [P, P, F, Z, Z, F]),
    (4, 6, 7, 5, [F, Z, Z, Z, F, Z]),
])
def test_face_rules_16_bit(store, nh, nx, ny, nz, bc):
    _run(store, nh, nx, ny, nz, bc, 3)
