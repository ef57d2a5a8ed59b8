"""Residual checks in panel launches with a modulus per node (needs a GPU): a
solve that converges stops where single steps stop, with the same outputs, on
grids of several panels with a ragged last one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# one short launch, one whole, two, three; halos of 14, 12 and 12 steps; odd sizes, since a period-2 mode of even ones
# keeps checks at odd intervals from passing
@pytest.mark.parametrize("nx,ny,tol", [(61, 47, 1e-6), (157, 149, 1e-4), (131, 139, 1e-4)])
@pytest.mark.parametrize("K", [5, 14, 20, 33])
def test_converged_solves_stop_where_single_steps_do(nx, ny, tol, K):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_31347_amd import slbm as S
    rng = np.random.default_rng(nx)
    F = 1e-2 * rng.standard_normal((2, ny, nx))
    F -= F.mean((1, 2), keepdims=True)               # a mean force has no steady state on the torus
    E = 1.0 + 0.3 * np.tanh(rng.standard_normal((ny, nx)))
    p = dict(nx=nx, ny=ny, dx=1.0 / max(nx, ny), E=1.0, nu=0.3, domain=S.PERIODIC, target=1e-3 * F[::-1].copy(),
             control_kind=S.CTRL_E_NODAL, fixed_force=F, tol=tol, max_steps=200000, check_interval=K)
    out = []
    for tuning in (1, -1):
        ctx = S.solid_lbm_init(p)
        S.solid_lbm_set_tuning(ctx, tuning, 0)
        rc, J, g, pi, ai = S.objective_and_grad(ctx, E)
        assert rc == 0 and pi.converged and ai.converged
        out.append((J, pi.steps, ai.steps, np.asarray(g), S.solid_lbm_get_field(ctx, S.FIELD_POPS),
                    S.solid_lbm_get_field(ctx, S.FIELD_ADJ_POPS), pi.residual, ai.residual))
    a, b = out
    assert a[:3] == b[:3]
    for k in (3, 4, 5):
        assert np.array_equal(a[k], b[k])
    for k in (6, 7):                                 # sums over panels instead of blocks
        assert abs(a[k] - b[k]) <= 1e-9 * abs(a[k])
