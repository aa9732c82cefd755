"""GPU tests of lbm_step_ws: several time steps per launch, between the
lattice's buffer and a workspace lent for the call.  Lattice.step takes it where
lbm_step_workspace offers one; states, residuals, time and the random stream of
FP16 storage must be those of lbm_step bit for bit.  Shapes: bricks of each
thread count, remainder bricks, axes of one and two nodes, axes that a brick
spans (periodic and walled), and boxes next to the size limits on both sides."""
import ctypes
import sys

import numpy as np
import pytest

import lbm_inputs
from lbm_inputs import face

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

from paper_1611_03329_amd import Batch, Lattice, lbm  # noqa: E402

WALL, PER = face("wall", "adiabatic"), face("periodic", "periodic")
HOT, COLD = face("wall", "isothermal", 0.4), face("wall", "isothermal", -0.3)


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _single(lat, n):
    assert lbm.library().lbm_step(lat._h, n) == 0, lbm.library().lbm_last_error()


def _workspace(lat, n=100):
    need = ctypes.c_size_t()
    assert lbm.library().lbm_step_workspace(lat._h, n, ctypes.byref(need)) == 0
    return need.value


FLOW = {
    "cavity": ((16, 12, 10), [HOT, COLD, WALL, WALL, WALL, WALL]),
    "ragged": ((23, 13, 11), [HOT, COLD, PER, PER, WALL, WALL]),
    "periodic": ((9, 7, 5), [PER] * 6),
    "cube32": ((32, 32, 32), [HOT, COLD, WALL, WALL, WALL, WALL]),
    "long": ((100, 20, 19), [PER, PER, HOT, COLD, PER, PER]),
    "flat": ((2, 30, 1), [WALL, WALL, HOT, COLD, PER, PER]),
    "largest": ((44, 44, 44), [HOT, COLD, WALL, WALL, PER, PER]),
}


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("name", sorted(FLOW))
def test_two_steps_per_launch_equal_single_steps(name, prec):
    shape, faces = FLOW[name]
    q = 15 if name in ("ragged", "flat") else 19
    wl = lbm_inputs.cavity(shape, lattice=q, rayleigh=1e3, seed=3, s_nu_set=1.2)
    wl["faces"] = faces
    _say(f"case passes {name} {prec}")
    with Lattice(wl, prec, check_interval=7) as a, Lattice(wl, prec, check_interval=7) as b:
        f, g = lbm_inputs.random_state(q, a.shape, 5, amp=0.01)
        a.set_state(f, g)
        b.set_state(f, g)
        if name in ("cavity", "periodic", "cube32"):
            assert _workspace(b) > 0
        for n in (4, 9, 3, 18):
            _single(a, n)
            b.step(n)
            for x, y in zip(a.get_state(), b.get_state()):
                assert torch.equal(x, y), (name, prec, n)
            assert a.time == b.time and a.residual() == b.residual()


@pytest.mark.parametrize("interval", [1, 2, 3, 4, 10])
def test_checks_inside_passes_equal_single_steps(interval):
    """Snapshot and compare steps on either side of a pass, at each alignment."""
    wl = lbm_inputs.cavity((40, 21, 24), rayleigh=1e4, seed=6)
    _say(f"case checks every {interval}")
    with Lattice(wl, "fp64", check_interval=interval) as a, Lattice(wl, "fp64", check_interval=interval) as b:
        for n in (4, 21, 6, 20, 1, 13):
            _single(a, n)
            b.step(n)
            assert a.residual() == b.residual(), (interval, a.time)
            for x, y in zip(a.get_state(), b.get_state()):
                assert torch.equal(x, y), (interval, a.time)


MELT = {
    "slab": ((400, 6, 6), None),
    "walls": ((30, 4, 11), [HOT, WALL, WALL, COLD, PER, PER]),
    "wide": ((120, 16, 15), None),
    "point": ((1, 3, 2), [PER] * 6),
}


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("name", sorted(MELT))
def test_enthalpy_passes_equal_single_steps(name, prec):
    shape, faces = MELT[name]
    wl = lbm_inputs.melting(*shape, alpha_ratio=12.0)
    if faces:
        wl["faces"] = faces
    _say(f"case enthalpy passes {name} {prec}")
    with Lattice(wl, prec) as a, Lattice(wl, prec) as b:
        g = np.random.default_rng(4).uniform(-0.3, 0.3, (7,) + a.shape)
        a.set_state(None, g)
        b.set_state(None, g)
        assert _workspace(b) > 0
        for n in (4, 5, 17, 50):
            _single(a, n)
            b.step(n)
            assert torch.equal(a.get_state()[1], b.get_state()[1]), (name, prec, n)
            assert a.time == b.time


def test_workspace_is_offered_only_where_it_is_used():
    small = lbm_inputs.cavity(16, seed=2)
    with Lattice(small, "fp32") as lat:
        assert _workspace(lat, 4) > 0 and _workspace(lat, 3) == 0
        # a workspace that is too small is not used
        ws = torch.full((1024,), 7, dtype=torch.uint8, device="cuda")
        assert lbm.library().lbm_step_ws(lat._h, 8, ctypes.c_void_p(ws.data_ptr()), ctypes.c_size_t(1024)) == 0
        torch.cuda.synchronize()
        assert lat.time == 8 and bool((ws == 7).all())
        with Batch(0) as batch:
            batch.add(lat)
            assert _workspace(lat) == 0
    for wl, prec in ((lbm_inputs.cavity(96), "fp32"), (lbm_inputs.channel((16, 8, 6)), "fp64")):
        with Lattice(wl, prec) as lat:
            assert _workspace(lat) == 0


@pytest.mark.parametrize("kind", ["flow", "enthalpy"])
def test_unusable_workspaces_are_refused(kind):
    wl = lbm_inputs.cavity(16, seed=2) if kind == "flow" else lbm_inputs.melting(400, 6, 6)
    with Lattice(wl, "fp32") as lat:
        need = _workspace(lat)
        room = torch.empty(need + 512, dtype=torch.uint8, device="cuda")
        host = np.empty(need + 512, dtype=np.uint8)
        for ws in (room.data_ptr() + 16, -(-host.ctypes.data // 256) * 256, lat._base):
            err = lbm.library().lbm_step_ws(lat._h, 8, ctypes.c_void_p(ws), ctypes.c_size_t(need))
            assert err == 1 and lat.time == 0
        aligned = -(-room.data_ptr() // 256) * 256
        assert lbm.library().lbm_step_ws(lat._h, 8, ctypes.c_void_p(aligned), ctypes.c_size_t(need)) == 0
        assert lat.time == 8


def test_steps_in_a_captured_graph_equal_eager_steps():
    wl = lbm_inputs.cavity((16, 12, 10), seed=9)
    stream = torch.cuda.Stream()
    with Lattice(wl, "fp32", stream=stream) as a, Lattice(wl, "fp32", stream=stream) as b:
        with torch.cuda.stream(stream):
            a.step(8)
            b.step(8)
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                b.step(8)
            for _ in range(3):
                graph.replay()
                _single(a, 8)
                torch.cuda.synchronize()
                for x, y in zip(a.get_state(), b.get_state()):
                    assert torch.equal(x, y)


MARCH = {
    # FP32: rows of 64 lanes x 2 and x 4 nodes, FP64: x 2
    "wide_rows": ((1040, 79, 75), [HOT, COLD, PER, PER, PER, PER]),
    "one_row": ((256, 65, 64), [WALL, HOT, COLD, WALL, WALL, HOT]),
    "ragged": ((258, 55, 75), [PER, PER, HOT, WALL, PER, PER]),
    "periodic": ((1026, 33, 31), [PER] * 6),
    "thin": ((4096, 257, 1), [HOT, WALL, PER, PER, COLD, HOT]),
}


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("name", sorted(MARCH))
def test_enthalpy_marching_passes_equal_single_steps(name, prec):
    shape, faces = MARCH[name]
    wl = lbm_inputs.melting(*shape, alpha_ratio=12.0)
    wl["faces"] = faces
    _say(f"case enthalpy marching passes {name} {prec}")
    with Lattice(wl, prec) as a, Lattice(wl, prec) as b:
        g = torch.rand((7,) + a.shape, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(3))
        g = 0.6 * g - 0.3
        a.set_state(None, g)
        b.set_state(None, g)
        assert _workspace(b) > 0
        for n in (4, 7, 6):
            _single(a, n)
            b.step(n)
            assert torch.equal(a.get_state()[1], b.get_state()[1]), (name, prec, n)
            assert a.time == b.time
