"""GPU test of the tile order of single lattices: states small enough for the
last-level cache are stepped in one contiguous range of tiles per XCD, larger
FP32 and FP64 ones in runs of tiles per XCD at odd parity.  The order changes no
value, so a lattice must be bit for bit the member of a batch that walks the
same tiles in hardware order.  Shapes: the smallest of the ranges in each
precision, tile counts that ranges and runs do not divide, and general-rule
channels."""
import sys

import pytest

import lbm_inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

from paper_1611_03329_amd import Batch, Lattice  # noqa: E402

CASES = {
    "fp32_smallest": (lbm_inputs.cavity(64, seed=5), "fp32"),
    "fp32_ragged": (lbm_inputs.cavity((65, 63, 65), seed=6), "fp32"),
    "fp64_ragged": (lbm_inputs.cavity((67, 64, 65), lattice=15, seed=7), "fp64"),
    "fp16_smallest": (lbm_inputs.cavity((128, 128, 64), seed=8), "fp16"),
    "fp32_channel": (lbm_inputs.channel((130, 47, 44)), "fp32"),
    "fp32_runs": (lbm_inputs.cavity((167, 161, 160), seed=9), "fp32"),
    "fp64_runs": (lbm_inputs.cavity((130, 131, 127), seed=10), "fp64"),
    "fp64_runs_channel": (lbm_inputs.channel((257, 99, 97)), "fp64"),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_tile_order_changes_no_state(name):
    wl, prec = CASES[name]
    print(f"case order {name}", flush=True)
    sys.stdout.flush()
    with Lattice(wl, prec) as a, Lattice(wl, prec) as b:
        with Batch(0) as batch:
            batch.add(b)
            a.step(5)
            batch.step(5)
            for x, y in zip(a.get_state(), b.get_state()):
                assert torch.equal(x, y), name
