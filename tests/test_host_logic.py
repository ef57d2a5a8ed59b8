"""The library's host side on a stubbed HIP runtime (hip_stub.c; no GPU): waits
after a failed launch, kernel attributes of every device, memory of launch plans, which kernels are chosen."""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, os, sys
sys.modules["torch"] = None                    # its own HIP runtime would answer first
stub = ctypes.CDLL({stub!r}, mode=ctypes.RTLD_GLOBAL)
for f in ("stub_what", "stub_where"):
    getattr(stub, f).restype = ctypes.c_size_t
sys.path.insert(0, {root!r})
import numpy as np
from paper_2609_31347_amd import inputs as I, slbm as S
LAUNCH, SYNC, ATTR, ALLOC, READ = 1, 2, 3, 4, 5
def log():
    return [(stub.stub_op(i), stub.stub_what(i), stub.stub_where(i)) for i in range(stub.stub_size())]
def kernels(call):
    stub.stub_reset(-1)
    call()
    return [what for op, what, _ in log() if op == LAUNCH]
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    """The stub, under the runtime's name, so that the library binds to it."""
    d = tmp_path_factory.mktemp("hip_stub")
    out, vers = os.path.join(d, "libamdhip64.so.7"), os.path.join(d, "versions")
    with open(vers, "w", encoding="utf-8") as f:
        f.write("hip_4.2 { *; };\nhip_4.3 { hipGraph*; hipStreamBeginCapture; hipStreamEndCapture; };\n")
    subprocess.run(["gcc", "-O1", "-fPIC", "-shared", "-Wall", "-Wl,-soname,libamdhip64.so.7",
                    "-Wl,--version-script," + vers, "-o", out, os.path.join(HERE, "hip_stub.c")], check=True)
    return out


def run(stub, code):
    src = PRELUDE.format(stub=stub, root=ROOT) + textwrap.dedent(code)
    r = subprocess.run([sys.executable, "-c", src], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


def test_a_batch_waits_for_both_streams_when_a_launch_fails(stub):
    """Kernels of the other class may still run on their stream: the call that
    reports the error returns only after they have ended, like every other call."""
    out = run(stub, """
        n = 32
        cp = I.clamped_plate(32, 20)
        probs = [dict(nx=n, ny=n, dx=1 / n, E=1.0, nu=0.3, target=np.ones((2, n, n)), control_kind=S.CTRL_FORCE_NODAL),
                 dict(nx=32, ny=20, dx=cp["dx"], E=1.0, nu=0.3, domain=S.MASKED,
                      node_mask=cp["active"].astype(np.uint8), link_bc=cp["bc"], link_wall=cp["wall"],
                      link_normal=cp["normal"], target=np.ones((2, 20, 32)), control_kind=S.CTRL_FORCE_NODAL)]
        for p in probs:
            p.update(tol=1e-10, max_steps=200, check_interval=10)
        controls = [np.ones((2, n, n)), np.ones((2, 20, 32))]
        b = S.solid_lbm_batch_init(probs)
        S.batch_objective_and_grad(b, controls, want_grad=False)      # builds the launch plans
        stub.stub_reset(-1)
        S.batch_objective_and_grad(b, controls, want_grad=False)
        whole = log()
        streams = {w for op, _, w in whole if op == LAUNCH}
        assert len(streams) == 2                                     # one per class
        other = [w for w in streams if w][0]
        mine = [i for i, e in enumerate(e for e in whole if e[0] == LAUNCH) if e[2] == other]
        for at in (mine[0], mine[len(mine) // 2], mine[-1], mine[len(mine) // 2] + 1):
            stub.stub_reset(at)
            try:
                S.batch_objective_and_grad(b, controls, want_grad=False)
            except S.SlbmError as e:
                assert e.code == S.EHIP
            else:
                raise AssertionError("no error")
            part = log()
            for s in streams:
                last = max([i for i, e in enumerate(part) if e[0] == LAUNCH and e[2] == s], default=-1)
                assert any(e[0] == SYNC and e[2] in (s, 2 ** 64 - 1) for e in part[last + 1:]), (at, s)
        stub.stub_reset(-1)
        S.batch_objective_and_grad(b, controls, want_grad=False)      # the batch is usable afterwards
        assert len(log()) == len(whole)
        print("ok")
    """)
    assert out.strip() == "ok"


@pytest.mark.parametrize("what", ["forward, staged", "forward, from memory", "weight gradient"])
def test_convolutions_raise_the_lds_limit_on_every_device(stub, what):
    """The limit of dynamic LDS is set on each device before the first launch
    there, and once."""
    out = run(stub, f"""
        what = {what!r}
        """ + """
        L, P = S.LIB, ctypes.c_void_p
        buf = (ctypes.c_char * 64)()
        p = P(ctypes.addressof(buf))
        def call():
            if what == "weight gradient":
                L.slbm_conv3x3_backward_weight_workspace.restype = ctypes.c_int64
                n = L.slbm_conv3x3_backward_weight_workspace(8, 32, 39, 64, 1)
                return L.slbm_conv3x3_backward_weight_ws(p, p, p, p, 8, 32, 32, 39, 64, 1, p, ctypes.c_int64(n), None)
            return L.slbm_conv3x3_forward(p, p, p, p, None, 8, 32, 32, 39, 64, 0, 1 if "staged" in what else 40, None)
        for dev, sets in ((0, 1), (1, 1), (0, 0), (5, 1), (1, 0), (70, 1), (70, 1)):
            stub.stub_device(dev)
            stub.stub_reset(-1)
            assert call() == 0
            seen = log()
            attrs = [e for e in seen if e[0] == ATTR]
            assert len(attrs) == sets and all(e[2] == dev for e in attrs), (dev, attrs)
            assert [e[0] for e in seen][:sets + 1] == [ATTR] * sets + [LAUNCH]
            assert all(e[1] == seen[sets][1] for e in attrs)          # of the kernel that is launched
        print("ok")
    """)
    assert out.strip() == "ok"


def test_panel_plans_take_memory_for_rim_tiles_only(stub):
    """The first solve of a 1000 x 600 plate allocates less for its panels than the
    16 KiB per 20 x 20 tile of the LDS tiles' plan."""
    out = run(stub, """
        cp = I.clamped_plate(1000, 600)
        p = dict(nx=1000, ny=600, dx=cp["dx"], E=1.0, nu=0.3, domain=S.MASKED, node_mask=cp["active"].astype(np.uint8),
                 link_bc=cp["bc"], link_wall=cp["wall"], link_normal=cp["normal"], target=np.ones((2, 600, 1000)),
                 control_kind=S.CTRL_FORCE_NODAL, tol=0.0, max_steps=13)
        taken = {}
        for tuning in (-1, 6):
            ctx = S.solid_lbm_init(p)
            S.solid_lbm_set_tuning(ctx, tuning, 0)
            stub.stub_reset(-1)
            S.objective_and_grad(ctx, np.ones((2, 600, 1000)), want_grad=False)
            taken[tuning] = sum(n for op, n, _ in log() if op == ALLOC)
        print(taken[-1], taken[6], flush=True)
        assert 0 < taken[-1] < taken[6]
    """)
    panels, tiles = (int(v) for v in out.split())
    assert panels < 0.6 * tiles


def test_kernel_attributes_are_set_once_per_context(stub):
    """Solves after the first set none: pipeline, panels and tiles of plates."""
    out = run(stub, """
        def problem(nx, ny, **more):
            return dict(nx=nx, ny=ny, dx=1 / nx, E=1.0, nu=0.3, target=np.ones((2, ny, nx)), tol=0.0, max_steps=40,
                        control_kind=S.CTRL_FORCE_NODAL, **more)
        def plate(nx, ny):
            cp = I.clamped_plate(nx, ny)
            p = problem(nx, ny, domain=S.MASKED, node_mask=cp["active"].astype(np.uint8), link_bc=cp["bc"],
                        link_wall=cp["wall"], link_normal=cp["normal"])
            return dict(p, dx=cp["dx"])
        for p in (problem(900, 900), plate(64, 39), plate(400, 240)):
            ctx = S.solid_lbm_init(p)
            sets = []
            for _ in range(2):
                stub.stub_reset(-1)
                S.objective_and_grad(ctx, np.ones((2, p["ny"], p["nx"])))
                sets.append(sum(op == ATTR for op, _, _ in log()))
            assert sets[0] > 0 and sets[1] == 0, (p["nx"], sets)
        print("ok")
    """)
    assert out.strip() == "ok"


@pytest.mark.parametrize("nx,ny,tiles", [(60, 5000, True), (60, 8000, True), (40, 4000, False), (400, 240, False)])
def test_narrow_plates_run_in_lds_tiles(stub, nx, ny, tiles):
    """Columns whose width suits no panel shape launch the kernels that an explicit
    6 steps per launch does (LDS tiles); others have panels."""
    out = run(stub, f"nx, ny, tiles = {nx}, {ny}, {tiles}" + """
cp = I.clamped_plate(nx, ny, b=(ny - 5.0) / (nx - 4.0) if ny > nx else 0.6)
p = dict(nx=nx, ny=ny, dx=cp["dx"], E=1.0, nu=0.3, domain=S.MASKED, node_mask=cp["active"].astype(np.uint8),
         link_bc=cp["bc"], link_wall=cp["wall"], link_normal=cp["normal"], target=np.ones((2, ny, nx)), tol=0.0,
         max_steps=48, control_kind=S.CTRL_FORCE_NODAL)
ctx = S.solid_lbm_init(p)
used = []
for tuning in (6, -1):
    S.solid_lbm_set_tuning(ctx, tuning, 0)
    S.objective_and_grad(ctx, np.ones((2, ny, nx)))               # builds the launch plan
    used.append(set(kernels(lambda: S.objective_and_grad(ctx, np.ones((2, ny, nx))))))
assert (used[0] == used[1]) == tiles
print("ok")
""")
    assert out.strip() == "ok"


@pytest.mark.parametrize("nx,ny,steps", [(3, 20000, 1), (100000, 3, 1), (17, 20000, 1), (3, 4000, 3), (96, 96, 7),
                                         (600, 600, 3)])
def test_tangent_launches(stub, nx, ny, steps):
    """Tiles of several tangent steps, single steps on thin grids, and single steps
    wherever the caller set one step per launch."""
    out = run(stub, f"nx, ny, steps = {nx}, {ny}, {steps}" + """
F = np.ones((2, ny, nx))
ctx = S.solid_lbm_init(dict(nx=nx, ny=ny, dx=1 / nx, E=1.0, nu=0.3, target=F, fixed_force=F, tol=0.0, max_steps=210,
                            control_kind=S.CTRL_E_SCALAR_SQ))
one = np.array([1.0])
def launches(tuning):
    S.solid_lbm_set_tuning(ctx, tuning, 0)
    return kernels(lambda: S.tangent_solve(ctx, one, one))
single, auto = launches(1), launches(-1)
assert len(single) >= 210
assert len(single) - len(auto) == (210 - 210 // steps)
assert (set(single) == set(auto)) == (steps == 1)
print("ok")
""")
    assert out.strip() == "ok"


@pytest.mark.parametrize("B,H,W,dil,memory", [(32, 39, 64, 8, True), (32, 39, 64, 4, False), (4, 39, 64, 8, False),
                                              (32, 512, 1, 1, True), (64, 256, 10, 2, True), (32, 200, 20, 1, False)])
def test_form_of_the_forward_convolution(stub, B, H, W, dil, memory):
    """From memory where staging the tiles' regions costs more: the kernel is that of
    a dilation whose region cannot be staged at all."""
    out = run(stub, f"B, H, W, dil, memory = {B}, {H}, {W}, {dil}, {memory}" + """
P = ctypes.c_void_p
p = P(ctypes.addressof((ctypes.c_char * 64)()))
def call(d):
    return kernels(lambda: S.LIB.slbm_conv3x3_forward(p, p, p, p, None, B, 32, 32, H, W, 0, d, None))
assert len(call(dil)) == 1
assert (call(dil) == call(60)) == memory
print("ok")
""")
    assert out.strip() == "ok"


@pytest.mark.parametrize("kind", ["E", "force"])
def test_device_controls_are_tested_with_one_launch_and_one_read(stub, kind):
    """New memory holds all ones, so no flag of the test is set."""
    out = run(stub, f"kind = {kind!r}" + """
stub.stub_fill(255)
n = 24
F = np.ones((2, n, n))
ctx = S.solid_lbm_init(dict(nx=n, ny=n, dx=1 / n, E=1.0, nu=0.3, target=F, fixed_force=F, tol=0.0, max_steps=4,
                            zero_mean_projection=0, control_kind=S.CTRL_E_NODAL if kind == "E" else S.CTRL_FORCE_NODAL))
c = F[0].copy() if kind == "E" else F
def counts(where):
    stub.stub_reset(-1)
    assert S.LIB.solid_lbm_set_control(ctx.handle, ctypes.c_void_p(c.ctypes.data), None, where) == 0
    ops = [op for op, _, _ in log()]
    return ops.count(LAUNCH), ops.count(READ)
counts(S.PTR_DEVICE)                                               # the first resets the flags
host, device = counts(S.PTR_HOST), counts(S.PTR_DEVICE)
assert host[1] == 0 and device == (host[0] + 1, 1), (host, device)
print("ok")
""")
    assert out.strip() == "ok"
