"""Both sets of a small 2D run in one launch, where test_gpu_pair2d.py does not
take it: every thermal pair of sets whose windows fit in LDS, with one and two
relaxation times, and both sides of the workgroup limits (1024 where a CU holds
one workgroup by the launch's LDS, 2048 otherwise).  Populations bit for bit
those of one launch per set, and the steps are counted as what they were."""
import numpy as np
import pytest

from paper_2102_12559_amd import inputs

pytestmark = pytest.mark.gpu
P, Z = inputs.BC_PERIODIC, inputs.BC_OUTFLOW_ZG
F64, F32, F16, BF16 = inputs.STORE_FP64, inputs.STORE_FP32, inputs.STORE_FP16_DEV, inputs.STORE_BF16_DEV


def _both(nl, nh, th, store, nx, ny, bc, extra, paired):
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
        s.step(5)
        assert s.paired_steps == (0 if apart or not paired else 5)
        out.append([s.get_populations(w, k).cpu().numpy() for w in range(2) for k in range(1 + th)])
        s.profile(False)
        s.close()
    print(f"[case] D2Q{nl * nl} + D2Q{nh * nh} thermal={th} store={store} {nx}x{ny} paired={paired}", flush=True)
    for a, b in zip(*out):
        assert np.all(np.isfinite(a)) and np.array_equal(a, b)


@pytest.mark.parametrize("tau2", [0.0, 0.9])
@pytest.mark.parametrize("store", [F64, F32, F16, BF16])
@pytest.mark.parametrize("nl,nh", [(3, 4), (3, 5), (3, 6), (4, 5), (4, 6), (5, 6)])
def test_thermal_pairs(nl, nh, store, tau2):
    # FP64 windows of f and g fit for D2Q9 and D2Q16 alone
    _both(nl, nh, 1, store, 70, 19, [P, P, Z, Z], dict(tau2=tau2), store != F64 or nh == 4)


@pytest.mark.parametrize("nl,nh,th,store,limit", [(3, 5, 0, F64, 1024), (3, 6, 1, F32, 1024), (3, 4, 0, F64, 2048)])
def test_workgroup_limits(nl, nh, th, store, limit):
    ny = 2 * limit   # tiles of four rows in both sets, one column of tiles
    _both(nl, nh, th, store, 40, ny, [P, P, P, P], {}, True)
    _both(nl, nh, th, store, 40, ny + 1, [P, P, P, P], {}, False)
