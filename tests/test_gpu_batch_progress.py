"""Progress reports of a batch whose classes run at their own pace (needs a
GPU): step and residual come from the instances that still run."""
import numpy as np
import pytest

from paper_2609_31347_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_reports_leave_out_stopped_instances():
    """A plate without a load passes its first check, step 1009, long before the
    periodic instance gets there; every report is of the periodic instance, whose
    checks fall on multiples of 16."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_31347_amd import slbm as S
    n = 512
    F = I.grf(n, n, 1 / n, 0.05, 0.1, 5, comps=2)
    strips = dict(nx=n, ny=n, dx=1 / n, E=1.0, nu=0.3, domain=S.PERIODIC, target=1e-3 * F[::-1].copy(),
                  control_kind=S.CTRL_FORCE_NODAL, check_interval=16)
    cp = I.clamped_plate(64, 39)
    plate = dict(nx=64, ny=39, dx=cp["dx"], E=1.0, nu=0.3, domain=S.MASKED, node_mask=cp["active"].astype(np.uint8),
                 link_bc=cp["bc"], link_wall=np.zeros_like(cp["wall"]), link_normal=cp["normal"],
                 target=1e-3 + np.zeros((2, 39, 64)), control_kind=S.CTRL_FORCE_NODAL, check_interval=1009)
    steps = 3000

    def reports(probs, controls):
        for p in probs:
            p.update(tol=1e-14, max_steps=steps)
        batch = S.solid_lbm_batch_init(probs)
        seen = []
        S.solid_lbm_batch_set_progress(batch, lambda ph, st, r: seen.append((ph, st, r)), 0.0)
        _, _, _, pi, _ = S.batch_objective_and_grad(batch, controls, want_grad=False)
        return seen, pi
    seen, pi = reports([strips, plate], [F, np.zeros((2, 39, 64))])
    assert [x.steps for x in pi] == [steps, 1009]
    alone, _ = reports([strips], [F])
    res = {st: r for _, st, r in alone}
    print("reports", len(seen), "alone", len(alone), flush=True)
    assert len(seen) >= 10 and len(alone) >= 10
    for _, st, r in seen:
        assert st % 16 == 0
        if st in res:
            assert r == res[st]
