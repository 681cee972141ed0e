"""Which stream CpdpState waits for before it reads a result on the host."""
from types import SimpleNamespace

import pytest
import torch

from paper_2607_21224_amd import cpdp, state


@pytest.mark.parametrize("state_device,current,waits", [(1, 0, True), (0, 0, False)])
def test_count_unsynced_waits_for_the_launch_stream(monkeypatch, state_device, current, waits):
    """The count is launched on the current stream of the current device; with
    the state on another device, reading the word does not wait for that one."""
    order = []
    word = SimpleNamespace(item=lambda: order.append("read") or 0)
    st = SimpleNamespace(params=SimpleNamespace(device=torch.device("cuda", state_device)),
                         anchor=None, W=2, P=8, ld=8, param_dt="f32", _count=word)
    launched = SimpleNamespace(synchronize=lambda: order.append("wait"))
    monkeypatch.setattr(state, "_on", lambda stream: launched)
    monkeypatch.setattr(cpdp, "cpdp_count_unsynced", lambda *a, **k: order.append("launch"))
    monkeypatch.setattr(torch.cuda, "current_device", lambda: current)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: launched)
    assert state.CpdpState.count_unsynced(st) == 0
    assert order == ["launch"] + ["wait"] * waits + ["read"]
