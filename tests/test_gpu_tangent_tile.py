"""Fused tangent launches (needs a GPU): J and its derivative after a fixed step
count against the primal's J and its central difference."""
import numpy as np
import pytest

from paper_2609_31347_amd import inputs as I

pytestmark = pytest.mark.gpu


# 7, 5 and 3 steps per launch by size, 3 in several rounds of workgroups; step counts with a shorter last launch,
# a single step left over, and fewer than one launch; plates and the torus (narrower than a region too)
@pytest.mark.parametrize("domain,nx,ny,steps", [("plate", 48, 29, 30), ("plate", 200, 120, 31), ("plate", 300, 180, 29),
                                                ("plate", 400, 240, 30), ("plate", 64, 39, 2), ("plate", 64, 39, 1),
                                                ("periodic", 13, 9, 30), ("periodic", 65, 50, 44)])
@pytest.mark.parametrize("kind", ["scalar", "E"])
def test_tangent_matches_difference_quotient(domain, nx, ny, steps, kind):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_31347_amd import slbm as S
    if domain == "plate":
        cp = I.clamped_plate(nx, ny)
        p = dict(nx=nx, ny=ny, dx=cp["dx"], domain=S.MASKED, node_mask=cp["active"].astype(np.uint8),
                 link_bc=cp["bc"], link_wall=cp["wall"], link_normal=cp["normal"])
    else:
        p = dict(nx=nx, ny=ny, dx=1.0 / nx, domain=S.PERIODIC)
    F = I.grf(nx, ny, p["dx"], 0.05, 0.1, 3, comps=2)
    p.update(E=1.0, nu=0.3, target=1e-6 * F[::-1].copy(), tol=0.0, max_steps=steps, fixed_force=F,
             control_kind=S.CTRL_E_SCALAR_SQ if kind == "scalar" else S.CTRL_E_NODAL)
    if kind == "scalar":
        c, d = np.array([1.05]), np.array([1.0])
    else:
        c = 1.0 + 0.3 * np.tanh(I.grf(nx, ny, p["dx"], 1.0, 0.2, 9)[0])
        d = I.grf(nx, ny, p["dx"], 1.0, 0.3, 11)[0]
    ctx = S.solid_lbm_init(p)
    _, J, dJ, info = S.tangent_solve(ctx, c, d)
    assert info.steps == steps
    J_of = lambda x: S.objective_and_grad(ctx, x, want_grad=False)[1]        # noqa: E731
    J0 = J_of(c)
    assert abs(J - J0) <= 1e-12 * abs(J0)
    # five-point quotient: truncation O(eps^4), rounding about 1e-16 |J| / eps
    eps = 1e-3 if kind == "scalar" else 3e-3
    q = (8 * (J_of(c + eps * d) - J_of(c - eps * d)) - (J_of(c + 2 * eps * d) - J_of(c - 2 * eps * d))) / (12 * eps)
    assert abs(dJ - q) <= 1e-7 * abs(q) + 1e-11 * abs(J0)
