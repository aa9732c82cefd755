"""CPU test of the workspace that Lattice.step lends: it is memory of the device
the lattice was created on, also after the program has made another one current."""
import contextlib
import types

import pytest

from paper_1611_03329_amd import Lattice, lbm

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("own", [True, False])
def test_the_workspace_is_on_the_lattices_device(monkeypatch, own):
    home = torch.device("cuda:1")
    asked = []

    def empty(n, dtype, device):
        asked.append(device)
        return types.SimpleNamespace(data_ptr=lambda: 512)

    def workspace(handle, n, need):
        need._obj.value = 1 << 20
        return 0

    lat = object.__new__(Lattice)
    lat._h, lat._passes, lat.batch = None, True, None
    lat.device, lat.buf = torch.device("cuda"), types.SimpleNamespace(device=home)
    lat.stream = types.SimpleNamespace(cuda_stream=64)
    monkeypatch.setattr(torch, "empty", empty)
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda device=None: asked.append(device) or types.SimpleNamespace(cuda_stream=64 if own else 32))
    monkeypatch.setattr(torch.cuda, "stream", lambda s: contextlib.nullcontext())
    monkeypatch.setattr(lbm, "_lib", types.SimpleNamespace(lbm_step_workspace=workspace,
                                                           lbm_step_ws=lambda h, n, ws, size: 0))
    lat.step(8)
    assert asked == [home, home]
