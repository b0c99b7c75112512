"""The co-moving step at the edges of its tiles, in both lane layouts (point
columns on lanes of their own on small grids and for D2Q25; otherwise per x
node), against the oracle at the FP64 bar of the co-moving tests (1e-12 on the
frames and on the populations relative to the frame's rho W_i); and the pass
statistics of uniform flows, where every cell takes one pass (the reconstructed
frame differs from the old one by rounding, far below the 1e-14 that ends the
iteration)."""
import numpy as np
import pytest

from paper_2102_12559_amd import inputs
from tests.test_gpu_pond import _gpu, compare, pond_pair  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,thermal,qe,nx,ny", [
    (3, 1, 0, 18, 5), (4, 1, 1, 5, 4), (5, 1, 1, 17, 9), (6, 1, 0, 9, 5),
    (3, 1, 1, 67, 53), (4, 0, 0, 65, 54), (4, 1, 0, 68, 57), (5, 0, 0, 69, 55)])
def test_tiles_match_oracle(n, thermal, qe, nx, ny):
    cfg = inputs.base_config(nx=nx, ny=ny, n_low=n, tau=0.8, cfl=0.4, thermal=thermal, cv=1.5, pond=1)
    if qe:
        cfg["tau2"] = 0.5 + 1.5 * 0.3
    rho, u, T = inputs.smooth_random_flow(nx, ny, umax=0.15, seed=n + nx, drho=0.03, dT=0.03 if thermal else 0.0)
    u[0] += 0.6
    u[1] -= 0.2
    s, o = pond_pair(cfg, rho, u, T, 2, f"tiles n={n} {nx}x{ny}")
    compare(s, o, cfg)


@pytest.mark.parametrize("n,nx,ny", [(3, 18, 5), (4, 67, 53), (5, 69, 55), (6, 9, 5)])
def test_pass_statistics_of_a_uniform_flow(n, nx, ny):
    from paper_2102_12559_amd import msl
    cfg = inputs.base_config(nx=nx, ny=ny, n_low=n, tau=0.8, cfl=0.4, thermal=1, cv=1.5, pond=1)
    u = np.zeros((2, 1, ny, nx))
    u[0], u[1] = 0.7, -0.3
    s = msl.Solver(cfg)
    s.init(np.ones((1, ny, nx)), u, np.ones((1, ny, nx)))
    for steps in (1, 3):
        s.step(steps)
        mean, most = s.pond_iterations()
        assert mean == 1.0 and most == 1
