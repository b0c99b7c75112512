"""Ghost rows in the D2Q9 kernel of large grids (tiles of eight rows, whose FP64
windows take two loads per lane): a flow uniform along x on a grid of 3072 such
tiles holds, in every column, what the same flow gives on a narrow grid, which
takes the four-row kernel checked against the oracle elsewhere.  FP64 within
1e-12, FP32 within 1e-5."""
import numpy as np
import pytest

from paper_2102_12559_amd import inputs

pytestmark = pytest.mark.gpu
P, F, Z, W = inputs.BC_PERIODIC, inputs.BC_FIXED_EQ, inputs.BC_OUTFLOW_ZG, inputs.BC_DIFFUSE_WALL


@pytest.mark.parametrize("store,tol", [(inputs.STORE_FP64, 1e-12), (inputs.STORE_FP32, 1e-5)])
@pytest.mark.parametrize("ylo,yhi", [(P, P), (Z, F), (W, Z)])
def test_wide_grid_equals_narrow_grid(store, tol, ylo, yhi):
    from paper_2102_12559_amd import msl
    ny, out = 20, []
    y = np.arange(ny)
    for nx in (8, 65536):
        cfg = inputs.base_config(dim=2, nx=nx, ny=ny, n_low=3, tau=0.7, store=store)
        cfg["bc"] = [P, P, ylo, yhi, P, P]
        cfg["bc_state"][2] = cfg["bc_state"][3] = [1.0, 0.04, 0.0, 0.0, 1.0]
        col = np.stack([1 + 0.02 * np.sin(0.9 * y), 0.05 * np.cos(0.7 * y), 0.03 * np.sin(0.4 * y + 1)])
        f = np.broadcast_to(col[:, None, :, None], (3, 1, ny, nx))
        s = msl.Solver(cfg)
        s.init(f[0], f[1:], np.ones((1, ny, nx)))
        s.step(3)
        out.append([a.cpu().numpy() for a in s.macros()])
        s.close()
    print(f"[case] store {store} faces {ylo} {yhi}", flush=True)
    for narrow, wide in zip(*out):
        assert np.max(np.abs(wide - narrow[..., :1])) <= tol
