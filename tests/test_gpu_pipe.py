"""Wave pipeline of large periodic uniform grids (needs a GPU): its launches of
16 steps, and the wave strips that take a shorter rest, equal single sweeps bit
for bit at ragged last strips and row blocks, odd and even widths, and grids
narrower or flatter than a strip's halo."""
import numpy as np
import pytest

from paper_2609_31347_amd import inputs as I

pytestmark = pytest.mark.gpu

# (nx, ny): ragged strips and row blocks, odd width; whole strips; one strip that wraps onto itself;
# fewer rows than the halo wraps over; too flat for the pipeline (wave strips)
SIZES = ((1025, 777), (960, 800), (70, 9000), (23997, 20), (46669, 3))


@pytest.mark.parametrize("nx,ny", SIZES)
def test_pipeline_equals_single_steps_bit_for_bit(nx, ny):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_31347_amd import slbm as S
    dx = 1.0 / max(nx, ny)
    rng = np.random.default_rng(5)
    control = 1e-2 * rng.standard_normal((2, ny, nx))
    p = dict(nx=nx, ny=ny, dx=dx, E=1.0, nu=0.3, domain=0, target=1e-3 * control[::-1].copy(), tol=0.0, max_steps=14,
             control_kind=S.CTRL_FORCE_NODAL)

    def fields(tuning):
        ctx = S.solid_lbm_init(p)
        S.solid_lbm_set_tuning(ctx, tuning, 0)
        S.solid_lbm_set_control(ctx, control)
        S.solid_lbm_run_steps(ctx, 38)           # 2 launches of 16 and, before the last step, strips of 4 and 1
        pops = S.solid_lbm_get_field(ctx, S.FIELD_POPS)
        S.primal_solve(ctx, control)
        S.solid_lbm_run_adjoint_steps(ctx, 31)   # 16, 8 and 6
        return pops, S.solid_lbm_get_field(ctx, S.FIELD_ADJ_POPS)
    ref, got = fields(1), fields(-1)
    assert np.abs(ref[0]).max() > 0 and np.abs(ref[1]).max() > 0
    assert np.array_equal(ref[0], got[0])
    assert np.array_equal(ref[1], got[1])
