"""Batches whose instances check at different intervals (needs a GPU): every
instance keeps its own schedule, so its stop steps, J and gradient are those
of the same problem alone, in the wave-strip and the tiled class."""
import numpy as np
import pytest

from paper_2609_31347_amd import inputs as I

pytestmark = pytest.mark.gpu


# intervals around the strips' 8 and the tiles' 6 steps, a check every step, and runs that end at max_steps: on a
# check of some instances, between checks of others; one class alone and both
@pytest.mark.parametrize("kinds", ["strips", "tiles", "both"])
@pytest.mark.parametrize("max_steps", [200000, 56, 57])
def test_instances_keep_their_own_check_schedules(kinds, max_steps):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_31347_amd import slbm as S
    probs, controls = [], []
    if kinds != "tiles":
        for n, K in ((32, 1), (40, 7), (33, 8), (48, 9), (64, 50)):
            F = I.grf(n, n, 1.0 / n, 0.05, 0.1, K, comps=2)
            probs.append(dict(nx=n, ny=n, dx=1.0 / n, E=1.0, nu=0.3, domain=S.PERIODIC, target=1e-3 * F[::-1].copy(),
                              control_kind=S.CTRL_FORCE_NODAL, check_interval=K))
            controls.append(F)
    if kinds != "strips":
        for n, K in ((16, 5), (20, 6), (24, 7), (16, 28)):
            cp = I.paper_plate(n)
            ny, nx = cp["active"].shape
            probs.append(dict(nx=nx, ny=ny, dx=cp["dx"], E=0.1, nu=0.7, domain=S.MASKED,
                              node_mask=cp["active"].astype(np.uint8), link_bc=cp["bc"], link_wall=cp["wall"],
                              link_normal=cp["normal"], target=cp["target"], control_kind=S.CTRL_FORCE_NODAL,
                              check_interval=K))
            controls.append(cp["F"] * 1.1)
    for p in probs:
        p.update(tol=1e-6, max_steps=max_steps)
    batch = S.solid_lbm_batch_init(probs)
    rc, J, grads, pi, ai = S.batch_objective_and_grad(batch, controls)
    assert rc == (1 if max_steps < 100 else 0)
    for i, (p, c) in enumerate(zip(probs, controls)):
        ctx = S.solid_lbm_init(p)
        S.solid_lbm_set_tuning(ctx, 1, 0)
        rc1, J1, g1, pi1, ai1 = S.objective_and_grad(ctx, c)
        assert (pi[i].steps, ai[i].steps) == (pi1.steps, ai1.steps), i
        assert J[i] == J1 and np.array_equal(np.asarray(grads[i]), np.asarray(g1)), i
