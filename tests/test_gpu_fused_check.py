"""Residual checks as the first sweep of a fused tile launch (needs a GPU):
stop step, residual, J, gradient and populations are those of single-step
launches, whose checks are launches of their own."""
import numpy as np
import pytest

from paper_2609_31347_amd import inputs as I

pytestmark = pytest.mark.gpu


# check intervals below, at and above the steps of a launch (2, 3, 8, 9, 12, 13 and more than one poll's 64 steps),
# solves that converge, one that stops at max_steps on a check, just after one and between two, and the
# coefficient-of-variation test
@pytest.mark.parametrize("K,max_steps,cv", [(2, 10 ** 6, False), (3, 10 ** 6, False), (8, 10 ** 6, False),
                                            (9, 10 ** 6, False), (12, 10 ** 6, False), (13, 10 ** 6, False),
                                            (70, 10 ** 6, False), (1, 10 ** 6, False), (10, 40, False),
                                            (10, 41, False), (10, 45, False), (10, 10 ** 6, True)])
@pytest.mark.parametrize("what", ["periodic", "plate", "plate_E"])
def test_fused_checks_stop_where_single_steps_do(what, K, max_steps, cv):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_31347_amd import slbm as S
    if what == "periodic":
        nx, ny = 30, 26
        dx = 1.0 / 30
        F = I.grf(nx, ny, dx, 0.05, 0.1, 5, comps=2)
        p = dict(nx=nx, ny=ny, dx=dx, domain=S.PERIODIC, target=1e-3 * F[::-1].copy(),
                 control_kind=S.CTRL_FORCE_NODAL)
        control = F
    else:
        cp = I.paper_plate(20)
        ny, nx = cp["active"].shape
        p = dict(nx=nx, ny=ny, dx=cp["dx"], domain=S.MASKED, node_mask=cp["active"].astype(np.uint8),
                 link_bc=cp["bc"], link_wall=cp["wall"], link_normal=cp["normal"], target=cp["target"])
        if what == "plate":
            control = cp["F"] * 1.1
            p.update(control_kind=S.CTRL_FORCE_NODAL)
        else:
            control = 0.1 * (1.0 + 0.3 * np.tanh(I.grf(nx, ny, cp["dx"], 1.0, 0.2, 9)[0]))
            p.update(control_kind=S.CTRL_E_NODAL, fixed_force=cp["F"])
    p.update(E=1.0 if what == "periodic" else 0.1, nu=0.3 if what == "periodic" else 0.7, tol=1e-7,
             max_steps=max_steps, check_interval=K, convergence=S.CONV_CV if cv else S.CONV_KLAG)
    out = []
    for tuning in (1, -1):
        ctx = S.solid_lbm_init(p)
        S.solid_lbm_set_tuning(ctx, tuning, 0)
        rc, J, g, pi, ai = S.objective_and_grad(ctx, control)
        out.append((rc, J, pi.steps, ai.steps, np.asarray(g), S.solid_lbm_get_field(ctx, S.FIELD_POPS),
                    S.solid_lbm_get_field(ctx, S.FIELD_ADJ_POPS), pi.residual, ai.residual))
        # a second solve on the same context
        assert S.objective_and_grad(ctx, control)[1] == J
    a, b = out
    assert a[0] == b[0] == (1 if max_steps < 100 else 0)
    assert a[1:4] == b[1:4]
    for k in (4, 5, 6):
        assert np.array_equal(a[k], b[k])
    # the residual's sums run over tiles instead of blocks; the CV test takes a difference of nearly equal sums
    for k in (7, 8):
        assert abs(a[k] - b[k]) <= (1e-5 if cv else 1e-9) * abs(a[k])
