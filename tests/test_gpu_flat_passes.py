"""GPU test of two-step passes over enthalpy boxes of one plane (k_march2's FLAT
form): bit for bit the single steps, with the plane its own z neighbour or between
two walls, filled and ragged rows and tiles."""
import ctypes

import pytest

import lbm_inputs
from lbm_inputs import face

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

from paper_1611_03329_amd import Lattice, lbm  # noqa: E402

WALL, PER = face("wall", "adiabatic"), face("periodic", "periodic")
HOT, COLD = face("wall", "isothermal", 0.4), face("wall", "isothermal", -0.3)

FLAT = {
    "slab": ((1024, 1030, 1), [HOT, COLD, PER, PER, PER, PER]),
    "walls": ((2050, 515, 1), [WALL, HOT, COLD, WALL, HOT, COLD]),
    "periodic": ((898, 1201, 1), [PER] * 6),
    "wide": ((32770, 33, 1), [PER, PER, WALL, HOT, PER, PER]),
}


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("name", sorted(FLAT))
def test_passes_over_one_plane_equal_single_steps(name, prec):
    shape, faces = FLAT[name]
    wl = lbm_inputs.melting(*shape, alpha_ratio=12.0)
    wl["faces"] = faces
    print(f"case flat passes {name} {prec}", flush=True)
    need = ctypes.c_size_t()
    with Lattice(wl, prec) as a, Lattice(wl, prec) as b:
        g = torch.rand((7,) + a.shape, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(3))
        g = 0.6 * g - 0.3
        a.set_state(None, g)
        b.set_state(None, g)
        assert lbm.library().lbm_step_workspace(b._h, 4, ctypes.byref(need)) == 0 and need.value > 0
        for n in (4, 7, 6):
            assert lbm.library().lbm_step(a._h, n) == 0
            b.step(n)
            assert torch.equal(a.get_state()[1], b.get_state()[1]), (name, prec, n)
