"""Slots on a fixed z face that reach a y edge, in 3D: the face's ghost rows
beyond the edge hold the face's own profile there, whatever the y faces' rule
(the highest axis out of range is resolved first), for sharp and smooth slots,
periodic, zero-gradient and fixed y faces, one and two sets, against the
oracle.  FP32 within its bar of 1e-5; 16-bit deviations within the storage bar
of 2e-3, which a row of a sharp slot in the place of a base row exceeds."""
import numpy as np
import pytest

from paper_2102_12559_amd import inputs
from tests.gpu_util import compare_macros, run_pair

pytestmark = pytest.mark.gpu
P, F, Z = inputs.BC_PERIODIC, inputs.BC_FIXED_EQ, inputs.BC_OUTFLOW_ZG
STORES = [(inputs.STORE_FP32, 1e-5), (inputs.STORE_FP16_DEV, 2e-3), (inputs.STORE_BF16_DEV, 2e-3)]


@pytest.mark.parametrize("store,tol", STORES)
@pytest.mark.parametrize("edge", [0.0, 1.5])
@pytest.mark.parametrize("nh,nx,ny,nz,bc,slots", [
    (0, 9, 6, 5, [P, P, P, P, F, F], {4: [0, 9, 0, 3], 5: [2, 7, 3, 6]}),
    (4, 67, 7, 6, [P, P, Z, Z, F, Z], {4: [0, 67, 0, 3]}),
    (4, 9, 6, 9, [Z, Z, Z, F, Z, F], {5: [1, 8, 0, 6]}),
    (0, 10, 5, 4, [Z, Z, F, F, F, F], {3: [0, 6, 0, 2], 4: [0, 10, 0, 5]}),
])
def test_slot_at_a_y_edge(store, tol, edge, nh, nx, ny, nz, bc, slots):
    cfg = inputs.base_config(dim=3, nx=nx, ny=ny, nz=nz, n_low=3, n_high=nh, tau=0.7, store=store)
    cfg["bc"] = list(bc)
    for f, s in slots.items():
        cfg["slot"][f] = s
        cfg["slot_state"][f] = [1.05, 0.04, -0.03, 0.05 if f % 2 == 0 else -0.05, 1.0]
        cfg["slot_edge"][f] = edge
    rho, u, T = inputs.smooth_random_flow(nx, ny, nz, umax=0.02, seed=nx + nz)
    mask = np.zeros((nz, ny, nx), np.uint8)
    if nh:
        mask[:, : ny // 2, : nx // 2 + 1] = 1
    s, o = run_pair(cfg, rho, u, T, mask, 4, tag=f"slot {bc} edge {edge}")
    compare_macros(s, o, tol, 1.0)
