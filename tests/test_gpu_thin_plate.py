"""Tall narrow plates (needs a GPU): in LDS tiles, where no panel shape suits the
width, and in panels the fields are the single steps'."""
import numpy as np
import pytest

from paper_2609_31347_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(60, 5000), (60, 8000), (40, 4000)])
def test_fields_of_narrow_plates(nx, ny):
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
    out = []
    for tuning in (1, -1):
        S.solid_lbm_set_tuning(ctx, tuning, 0)
        rc, J, g, pi, ai = S.objective_and_grad(ctx, F)
        out.append((J, g))
    assert out[0][0] == out[1][0] and np.array_equal(out[0][1], out[1][1])
