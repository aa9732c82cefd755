"""GPU test of the step count that drives FP16 rounding: passes of several steps
take and advance the device's, as single steps do, also after steps that a
graph has replayed (which the host does not see)."""
import ctypes

import pytest

import lbm_inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

from paper_1611_03329_amd import Lattice, lbm  # noqa: E402


def _single(lat, n):
    assert lbm.library().lbm_step(lat._h, n) == 0, lbm.library().lbm_last_error()


@pytest.mark.parametrize("prec", ["fp16", "fp32"])
def test_passes_after_replayed_steps_equal_single_steps(prec):
    print(f"case passes after replays {prec}", flush=True)
    wl = lbm_inputs.cavity((16, 12, 10), seed=9)
    stream = torch.cuda.Stream()
    with Lattice(wl, prec, stream=stream) as a, Lattice(wl, prec, stream=stream) as b:
        with torch.cuda.stream(stream):
            graph = torch.cuda.CUDAGraph()
            torch.cuda.synchronize()
            with torch.cuda.graph(graph, stream=stream):
                b.step(8)
            for n in (4, 7, 9, 12):
                for _ in range(3):
                    graph.replay()
                _single(a, 24)
                torch.cuda.synchronize()
                _single(a, n)
                b.step(n)
                if n == 7:  # back to the parity the graph was captured at
                    _single(a, 1)
                    b.step(1)
                if n == 9:
                    _single(a, 3)
                    b.step(3)
                for x, y in zip(a.get_state(), b.get_state()):
                    assert torch.equal(x, y), (prec, n)


@pytest.mark.parametrize("prec", ["fp16", "fp64"])
def test_a_workspace_passed_under_capture_is_left_alone(prec):
    print(f"case workspace under capture {prec}", flush=True)
    wl = lbm_inputs.cavity((16, 12, 10), seed=9)
    stream = torch.cuda.Stream()
    need = ctypes.c_size_t()
    with Lattice(wl, prec, stream=stream) as a, Lattice(wl, prec, stream=stream) as b:
        assert lbm.library().lbm_step_workspace(b._h, 8, ctypes.byref(need)) == 0 and need.value > 0
        room = torch.full((need.value + 256,), 7, dtype=torch.uint8, device="cuda")
        ws = ctypes.c_void_p(-(-room.data_ptr() // 256) * 256)
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                assert lbm.library().lbm_step_ws(b._h, 8, ws, need) == 0
            for _ in range(3):
                graph.replay()
                _single(a, 8)
                torch.cuda.synchronize()
                for x, y in zip(a.get_state(), b.get_state()):
                    assert torch.equal(x, y), prec
        assert bool((room == 7).all())
