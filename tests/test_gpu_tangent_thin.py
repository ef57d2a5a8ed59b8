"""Forward mode on thin grids (needs a GPU): tiles that are mostly outside the
grid are not taken."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# 16 x 16 tiles hold 5.3 times the grid's nodes: measured 2.1 to 3 times the single steps' time
@pytest.mark.parametrize("nx,ny", [(3, 20000), (3, 100000), (100000, 3)])
def test_thin_grids_take_no_longer_than_single_steps(nx, ny):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_31347_amd import slbm as S
    F = 1e-2 * np.random.default_rng(1).standard_normal((2, ny, nx))
    p = dict(nx=nx, ny=ny, dx=1.0 / max(nx, ny), E=1.0, nu=0.3, domain=S.PERIODIC, target=1e-3 * F[::-1].copy(),
             fixed_force=F, tol=0.0, max_steps=300, control_kind=S.CTRL_E_SCALAR_SQ)
    ctx = S.solid_lbm_init(p)
    ms, out = {1: [], -1: []}, {}
    for _ in range(4):
        for tuning in (1, -1):
            S.solid_lbm_set_tuning(ctx, tuning, 0)
            rc, J, dJ, info = S.tangent_solve(ctx, np.array([1.05]), np.array([1.0]))
            ms[tuning].append(info.device_ms)
            out[tuning] = (J, dJ)
    assert out[1] == out[-1]
    assert min(ms[-1]) <= 1.5 * min(ms[1])
