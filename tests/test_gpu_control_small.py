"""Refused controls in device memory (needs a GPU): the flags of the test do not
outlive the call."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_31347_amd import slbm
    return slbm


def problem(S, n=64):
    F = 1e-2 * np.random.default_rng(1).standard_normal((2, n, n))
    return dict(nx=n, ny=n, dx=1 / n, E=1.0, nu=0.3, domain=S.PERIODIC, target=1e-3 * F[::-1].copy(), fixed_force=F,
                tol=0.0, max_steps=9, control_kind=S.CTRL_E_NODAL)


def test_refusals_leave_no_trace(S):
    import torch
    ctx = S.solid_lbm_init(problem(S))
    good = 1.0 + 0.3 * np.tanh(np.random.default_rng(2).standard_normal((64, 64)))
    bads = []
    for at, v, code in ((0, -1.0, S.EINVAL), (5, np.nan, S.ENONFINITE), (-1, 0.0, S.EINVAL), (9, np.inf, S.ENONFINITE)):
        b = good.copy()
        b.reshape(-1)[at] = v
        bads.append((b, code))
    J = S.objective_and_grad(ctx, good, want_grad=False)[1]
    for b, code in bads + bads[::-1]:
        for _ in range(2):
            with pytest.raises(S.SlbmError) as e:
                S.solid_lbm_set_control(ctx, torch.tensor(b, device="cuda"))
            assert e.value.code == code
        assert S.objective_and_grad(ctx, torch.tensor(good, device="cuda"), want_grad=False)[1] == J

