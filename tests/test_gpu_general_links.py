"""GPU test of FP16 storage with a moving lid and an open face on D3Q19, whose odd
step takes element indices in its gather and byte offsets in its scatter: alone
and in a batch the states are the same, bit for bit, in plain and check steps."""
import pytest

import lbm_inputs
from lbm_inputs import face

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

from paper_1611_03329_amd import Batch, Lattice  # noqa: E402

LID = face("wall", "adiabatic", 0.0, (0.02, 0.0, 0.01))


@pytest.mark.parametrize("shape", [(20, 13, 11), (5, 1, 3), (64, 64, 64), (65, 64, 64)])
def test_a_lattice_steps_as_in_a_batch(shape):
    print(f"case general links {shape}", flush=True)
    wl = lbm_inputs.cavity(shape, rayleigh=1e3, seed=5, s_nu_set=1.2)
    wl["faces"][5] = LID
    wl["faces"][1] = face("outlet", "outflow")
    with Lattice(wl, "fp16", check_interval=4) as a, Lattice(wl, "fp16") as b, Batch(4) as batch:
        f, g = lbm_inputs.random_state(19, a.shape, 8, amp=0.01)
        a.set_state(f, g)
        b.set_state(f, g)
        batch.add(b)
        for n in (5, 8):
            a.step(n)
            batch.step(n)
            for x, y in zip(a.get_state(), b.get_state()):
                assert torch.equal(x, y), (shape, n)
