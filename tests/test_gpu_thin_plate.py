"""Tall narrow plates (needs a GPU): where no panel shape suits the width the
sweeps run in LDS tiles, in their time; the fields are the single steps'."""
import numpy as np
import pytest

from paper_2609_31347_amd import inputs as I

pytestmark = pytest.mark.gpu


# panels of 60 x 5000 and 60 x 8000 took 1.24 times the LDS tiles' time per adjoint step; 40 x 4000 takes panels
@pytest.mark.parametrize("nx,ny", [(60, 5000), (60, 8000), (40, 4000)])
def test_adjoint_steps_take_no_longer_than_in_lds_tiles(nx, ny):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_31347_amd import slbm as S
    cp = I.clamped_plate(nx, ny, b=(ny - 5.0) / (nx - 4.0))
    F = 1e-2 * np.random.default_rng(1).standard_normal((2, ny, nx))
    p = dict(nx=nx, ny=ny, dx=cp["dx"], E=1.0, nu=0.3, domain=S.MASKED, node_mask=cp["active"].astype(np.uint8),
             link_bc=cp["bc"], link_wall=cp["wall"], link_normal=cp["normal"], target=1e-3 * F[::-1].copy(), tol=0.0,
             max_steps=31, control_kind=S.CTRL_FORCE_NODAL)
    ctx = S.solid_lbm_init(p)
    us, out = {6: [], -1: []}, {}
    for tuning in (1, 6, -1):
        S.solid_lbm_set_tuning(ctx, tuning, 0)
        rc, J, g, pi, ai = S.objective_and_grad(ctx, F)
        out[tuning] = (J, g)
    for _ in range(5):
        for tuning in us:
            S.solid_lbm_set_tuning(ctx, tuning, 0)
            us[tuning].append(S.solid_lbm_time_sweeps(ctx, 1, 480))
    for tuning in us:
        assert out[tuning][0] == out[1][0] and np.array_equal(out[tuning][1], out[1][1])
    assert min(us[-1]) <= 1.1 * min(us[6])
