"""GPU test of lbm_set_state over whole and ragged node blocks: the state comes
back as it was given (FP64: to the rounding of the shift by the rest state;
FP32 and FP16 to the rounding of their storage)."""
import numpy as np
import pytest

import lbm_inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

from paper_1611_03329_amd import Lattice  # noqa: E402

# unit roundoff of each storage, relative to the largest departure stored: flow
# populations, temperature populations
EPS = {"fp64": (2.0 ** -52, 2.0 ** -52), "fp32": (2.0 ** -23, 2.0 ** -23), "fp16": (2.0 ** -10, 2.0 ** -23)}


@pytest.mark.parametrize("prec", sorted(EPS))
@pytest.mark.parametrize("q", [19, 15])
@pytest.mark.parametrize("shape", [(1, 1, 1), (32, 32, 1), (41, 25, 1), (64, 33, 3)])
def test_state_comes_back(shape, q, prec):
    print(f"case state {shape} D3Q{q} {prec}", flush=True)
    with Lattice(lbm_inputs.periodic_box(shape, lattice=q), prec) as lat:
        f, g = lbm_inputs.random_state(q, lat.shape, 7, amp=0.05)
        lat.set_state(torch.from_numpy(f), torch.from_numpy(g))
        for got, want, eps in zip(lat.get_state(), (f, g), EPS[prec]):
            # departures from the rest state are below 1, the values too
            assert np.max(np.abs(got.cpu().numpy() - want)) <= 2.0 * eps, (shape, q, prec)
