"""Modulus fields on thin periodic grids (needs a GPU): narrow columns of
many rows keep LDS tiles, flat ones take panels; the fields are the single
steps'."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# steps per launch tell the two apart: LDS tiles 8 up to 131072 nodes, panels 6 (GPU of 256 compute units)
@pytest.mark.parametrize("nx,ny,steps", [(3, 40000, 8), (15, 8700, 8), (40000, 3, 6)])
def test_thin_grids_with_a_modulus_field(nx, ny, steps):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_31347_amd import slbm as S
    rng = np.random.default_rng(nx)
    F = 1e-2 * rng.standard_normal((2, ny, nx))
    p = dict(nx=nx, ny=ny, dx=1.0 / max(nx, ny), E=1.0, nu=0.3, domain=S.PERIODIC, target=1e-3 * F[::-1].copy(),
             control_kind=S.CTRL_E_NODAL, fixed_force=F, tol=0.0, max_steps=48)
    E = 1.0 + 0.3 * np.tanh(rng.standard_normal((ny, nx)))
    out = []
    for tuning in (1, -1):
        ctx = S.solid_lbm_init(p)
        S.solid_lbm_set_tuning(ctx, tuning, 0)
        S.solid_lbm_set_launch_timing(ctx, 1)
        rc, J, g, pi, ai = S.objective_and_grad(ctx, E)
        out.append((J, g))
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert pi.fused_sweeps == steps * pi.fused_launches and ai.fused_sweeps == steps * ai.fused_launches
    assert out[0][0] == out[1][0] and np.array_equal(out[0][1], out[1][1])
