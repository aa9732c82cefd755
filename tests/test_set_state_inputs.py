"""Lattice.set_state and its caller's tensors: what the caller's stream still has to
write into them comes first, and they have been read when it returns, whichever
stream the lattice runs on and whichever stream they are freed to or written from
next."""
import types

import numpy as np
import pytest

import lbm_inputs
from paper_1611_03329_amd import Lattice, lbm

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("own, capturing", [(True, False), (False, False), (False, True)])
def test_the_inputs_have_been_read_on_return(monkeypatch, own, capturing):
    """On the caller's own stream too: a tensor of another stream may be freed
    to that stream, or refilled there, as soon as the call returns."""
    calls = []

    class Stream:
        cuda_stream = 64

        def synchronize(self):
            calls.append("wait")

        def wait_stream(self, other):
            calls.append("order")

    lat = object.__new__(Lattice)
    lat.stream, lat.device, lat.shape, lat.q, lat._h = Stream(), torch.device("cpu"), (2, 3, 4), 15, None
    lat.buf = torch.empty(0)
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda device=None: lat.stream if own else types.SimpleNamespace(cuda_stream=32))
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: capturing)
    monkeypatch.setattr(lbm, "_lib", types.SimpleNamespace(lbm_set_state=lambda *a: calls.append("copy") or 0))
    lat.set_state(np.zeros((15, 2, 3, 4)), np.zeros((7, 2, 3, 4)))
    assert calls == ([] if own or capturing else ["order"]) + ["copy", "wait"]


@pytest.mark.gpu
def test_inputs_of_another_stream_may_change_on_return():
    if not torch.cuda.is_available():  # pragma: no cover - CPU container
        pytest.skip("no GPU")
    print("case set_state from a loader's stream", flush=True)
    side = torch.cuda.Stream()
    with Lattice(lbm_inputs.periodic_box((96, 96, 96)), "fp64") as lat:
        f, g = (torch.from_numpy(a) for a in lbm_inputs.random_state(19, lat.shape, 3, amp=0.05))
        with torch.cuda.stream(side):
            df, dg = f.cuda(), g.cuda()
        side.synchronize()
        for _ in range(3):
            lat.step(50)
            lat.set_state(df, dg)
            with torch.cuda.stream(side):
                df.fill_(7.0)
                dg.fill_(7.0)
            got = [x.cpu() for x in lat.get_state()]
            side.synchronize()
            # departures from the rest state are below 1
            assert all(float((x - y).abs().max()) <= 2.0 ** -51 for x, y in zip(got, (f, g)))
            with torch.cuda.stream(side):
                df.copy_(f)
                dg.copy_(g)
            side.synchronize()


@pytest.mark.gpu
def test_inputs_still_being_written_come_first():
    if not torch.cuda.is_available():  # pragma: no cover - CPU container
        pytest.skip("no GPU")
    print("case set_state after work of the caller's stream", flush=True)
    with Lattice(lbm_inputs.periodic_box((48, 40, 32)), "fp64", stream=torch.cuda.Stream()) as lat:
        f, g = (torch.from_numpy(a).cuda() for a in lbm_inputs.random_state(19, lat.shape, 3, amp=0.05))
        df, dg = torch.zeros_like(f), torch.zeros_like(g)
        x = torch.ones(4096, 4096, device="cuda")
        torch.cuda.synchronize()
        for _ in range(40):  # work that the copies below wait for
            x = x @ x * 1e-4
        df.copy_(f)
        dg.copy_(g)
        lat.set_state(df, dg)
        got = lat.get_state()
        assert all(float((a - b).abs().max()) <= 2.0 ** -51 for a, b in zip(got, (f, g)))
