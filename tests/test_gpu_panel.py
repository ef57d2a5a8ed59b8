"""Register panels (needs a GPU): launches of several steps equal single
sweeps bit for bit, in every shape that the automatic choice takes on a GPU of
256 compute units, with ragged last panels and grids narrower than a panel,
and on plates with panels that lie wholly outside, Dirichlet holes, and rims
too dense for the boundary waves."""
import numpy as np
import pytest

from paper_2609_31347_amd import inputs as I

pytestmark = pytest.mark.gpu

# (rows per lane, halo) by size: (3,6), (4,8), (4,7), (6,12), (6,10), (8,12), (6,8), the wave pipeline; a 40-column grid
# that its 64-column regions wrap onto
SIZES = ((300, 300), (501, 333), (448, 448), (480, 470), (512, 512), (600, 600), (192, 2048), (700, 700), (40, 5000))
E_SIZES = ((401, 299), (501, 333), (480, 470), (700, 651))      # the last in several rounds of workgroups


def fields(S, problem, control, tuning, steps, adjoint_steps):
    ctx = S.solid_lbm_init(problem)
    S.solid_lbm_set_tuning(ctx, tuning, 0)
    S.solid_lbm_set_control(ctx, control)
    S.solid_lbm_run_steps(ctx, steps)
    pops = S.solid_lbm_get_field(ctx, S.FIELD_POPS)
    S.primal_solve(ctx, control)
    S.solid_lbm_run_adjoint_steps(ctx, adjoint_steps)
    return pops, S.solid_lbm_get_field(ctx, S.FIELD_ADJ_POPS)


@pytest.mark.parametrize("nx,ny,efield", [(*s, False) for s in SIZES] + [(*s, True) for s in E_SIZES])
def test_panels_equal_single_steps_bit_for_bit(nx, ny, efield):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_31347_amd import slbm as S
    dx = 1.0 / max(nx, ny)
    F = I.grf(nx, ny, dx, 0.05, 0.1, 21, comps=2)
    p = dict(nx=nx, ny=ny, dx=dx, E=1.0, nu=0.3, domain=0, target=1e-3 * F[::-1].copy(), tol=0.0, max_steps=14)
    if efield:
        control = 1.0 + 0.3 * np.tanh(I.grf(nx, ny, dx, 1.0, 0.2, 9)[0])
        p.update(control_kind=S.CTRL_E_NODAL, fixed_force=F)
    else:
        control = F
        p.update(control_kind=S.CTRL_FORCE_NODAL)
    # 2 launches of 12 (or 3 of 10, 4 of 8, ...), a shorter one, and a last single step
    ref = fields(S, p, control, 1, 37, 29)
    got = fields(S, p, control, -1, 37, 29)
    assert np.abs(ref[0]).max() > 0 and np.abs(ref[1]).max() > 0
    assert np.array_equal(ref[0], got[0])
    assert np.array_equal(ref[1], got[1])


def perforated(nx, ny, pitch):
    """A rectangular plate with a one-node hole every `pitch` nodes, all walls clamped."""
    active = np.zeros((ny, nx), bool)
    active[2:-2, 2:-2] = True
    active[4:-4:pitch, 4:-4:pitch] = False
    dx = 1.0 / nx
    X, Y = I.grid(nx, ny, dx)
    zero = lambda kind, xw, yw: (np.zeros((2,) + xw.shape), np.zeros((2,) + xw.shape))      # noqa: E731
    bc, wall, nrm = I._links(active, X, Y, dx, lambda xo, yo: np.full(xo.shape, I.DIRICHLET, np.uint8), zero)
    return dict(nx=nx, ny=ny, dx=dx, active=active, bc=bc, wall=wall, normal=nrm)


# (2, 8), (3, 8), (4, 8) and (4, 6) in one and several rounds by size; the paper's plate with two holes; a
# perforated plate of up to 256 boundary nodes a region, and one beyond (LDS tiles)
@pytest.mark.parametrize("what,size,efield", [("clamped", 384, False), ("clamped", 385, True), ("clamped", 512, True),
                                              ("clamped", 560, False), ("clamped", 701, True), ("clamped", 900, False),
                                              ("paper", 400, False), ("paper", 400, True), ("holes", 24, False),
                                              ("holes", 24, True), ("holes", 5, False)])
def test_plate_panels_equal_single_steps_bit_for_bit(what, size, efield):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_31347_amd import slbm as S
    if what == "clamped":
        cp = I.clamped_plate(size, int(np.ceil(0.6 * size)))
    elif what == "paper":
        cp = I.paper_plate(size)
    else:
        cp = perforated(330, 290, size)
    ny, nx = cp["active"].shape
    F = I.grf(nx, ny, cp["dx"], 0.05, 0.1, 5, comps=2) * cp["active"]
    p = dict(nx=nx, ny=ny, dx=cp["dx"], E=1.0, nu=0.3, domain=S.MASKED, node_mask=cp["active"].astype(np.uint8),
             link_bc=cp["bc"], link_wall=cp["wall"], link_normal=cp["normal"], target=1e-3 * F[::-1] * cp["active"],
             tol=0.0, max_steps=14)
    if efield:
        control = 1.0 + 0.3 * np.tanh(I.grf(nx, ny, cp["dx"], 1.0, 0.2, 9)[0])
        p.update(control_kind=S.CTRL_E_NODAL, fixed_force=F)
    else:
        control = F
        p.update(control_kind=S.CTRL_FORCE_NODAL)
    ref = fields(S, p, control, 1, 37, 29)
    got = fields(S, p, control, -1, 37, 29)
    assert np.abs(ref[0]).max() > 0 and np.abs(ref[1]).max() > 0
    assert np.array_equal(ref[0], got[0])
    assert np.array_equal(ref[1], got[1])
