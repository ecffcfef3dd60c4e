"""Which devices the Python binding takes (no GPU needed: the current device is
given by hand and nothing is enqueued)."""
import pytest
import torch

import paper_2607_09385_amd as steel


@pytest.fixture(autouse=True)
def on_device_0(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)


@pytest.mark.parametrize("device,index", [(1, 1), ("cuda:1", 1), (torch.device("cuda", 1), 1), (0, 0)])
def test_device_given_by_index_or_name(device, index):
    scope = steel._on(device)
    assert isinstance(scope, torch.cuda.device) and scope.idx == index


def test_current_device_is_not_switched():
    assert not isinstance(steel._on(torch.device("cuda", 0)), torch.cuda.device)


@pytest.mark.parametrize("device", ["cpu", "cpu:0", torch.device("cpu"), torch.device("cpu", 0),
                                    torch.device("meta", 0)], ids=str)
def test_other_devices_are_refused(device):
    """Their memory must not reach a kernel, whatever their index."""
    with pytest.raises(ValueError, match="Expected a cuda device"):
        steel._on(device)


@pytest.mark.parametrize("device", [torch.device("cpu", 0), "cpu:0"], ids=str)
def test_index_and_plan_on_the_host_are_refused(device):
    with pytest.raises(ValueError, match="Expected a cuda device"):
        steel.block_index(None, 1, 1, 64, 64, device=device)
    with pytest.raises(ValueError, match="Expected a cuda device"):
        steel.Plan(None, 1, 1, 1, 64, 64, device=device)
