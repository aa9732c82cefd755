"""GPU test of passes of several steps on boxes that reach each of their kernels
(pass_shapes.py): states, residuals and time are those of lbm_step bit for bit, and
a workspace is offered exactly where the table says so."""
import ctypes

import pytest

import lbm_inputs
import pass_shapes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

from paper_1611_03329_amd import Lattice, lbm  # noqa: E402


def _single(lat, n):
    assert lbm.library().lbm_step(lat._h, n) == 0, lbm.library().lbm_last_error()


def _offered(lat):
    need = ctypes.c_size_t()
    assert lbm.library().lbm_step_workspace(lat._h, 8, ctypes.byref(need)) == 0
    return need.value > 0


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("name", sorted(pass_shapes.FLOW))
def test_flow_passes_equal_single_steps(name, prec):
    shape, q, faces, threads = pass_shapes.FLOW[name]
    wl = lbm_inputs.cavity(shape, lattice=q, rayleigh=1e3, seed=3, s_nu_set=1.2)
    wl["faces"] = faces
    print(f"case pass shapes {name} {prec}", flush=True)
    with Lattice(wl, prec, check_interval=5) as a, Lattice(wl, prec, check_interval=5) as b:
        assert _offered(b) == (threads[prec] > 0)
        f, g = lbm_inputs.random_state(q, a.shape, 5, amp=0.01)
        a.set_state(f, g)
        b.set_state(f, g)
        for n in (4, 11, 8):
            _single(a, n)
            b.step(n)
            for x, y in zip(a.get_state(), b.get_state()):
                assert torch.equal(x, y), (name, prec, n)
            assert a.time == b.time and a.residual() == b.residual()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("table,name", [(t, n) for t in ("MELT", "MARCH") for n in sorted(getattr(pass_shapes, t))])
def test_enthalpy_passes_equal_single_steps(table, name, prec):
    shape, faces, kernel = getattr(pass_shapes, table)[name]
    wl = lbm_inputs.melting(*shape, alpha_ratio=12.0)
    wl["faces"] = faces
    print(f"case enthalpy pass shapes {name} {prec}", flush=True)
    with Lattice(wl, prec) as a, Lattice(wl, prec) as b:
        assert _offered(b) == (kernel[prec] > 0)
        g = torch.rand((7,) + a.shape, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(3))
        g = 0.6 * g - 0.3
        a.set_state(None, g)
        b.set_state(None, g)
        for n in (4, 13, 6):
            _single(a, n)
            b.step(n)
            assert torch.equal(a.get_state()[1], b.get_state()[1]), (name, prec, n)
            assert a.time == b.time
