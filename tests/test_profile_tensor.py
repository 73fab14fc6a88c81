"""The plane profiles' host tensor: the binding refuses one that the library
would write past or that is no host memory, before it calls it, and the
Solver's does not depend on the default device."""
import pytest
import torch

from paper_2401_17074_amd import _binding as C


@pytest.mark.parametrize("sums", [
    torch.empty((5, 13), dtype=torch.float32), torch.empty((4, 13), dtype=torch.float64),
    torch.empty((6, 13), dtype=torch.float64), torch.empty((13, 5), dtype=torch.float64).T,
    torch.empty((5, 13), dtype=torch.float64, device="meta")])
def test_refused(sums, monkeypatch):
    monkeypatch.setattr(C.lib, "tslb_stats_profile", lambda *a: pytest.fail("called"))
    monkeypatch.setattr(C, "_stream", lambda s: None)
    with pytest.raises(ValueError):
        C.tslb_stats_profile_into(None, sums, 5)


def test_accepted(monkeypatch):
    monkeypatch.setattr(C, "_stream", lambda s: None)
    with pytest.raises(C.TslbError):  # the library's own refusal of the NULL handle
        C.tslb_stats_profile_into(None, torch.empty((5, 13), dtype=torch.float64), 5)


@pytest.mark.gpu
def test_default_device():
    import workloads as W
    from helpers import gpu_solver
    s = gpu_solver(W.Case("default", 8, 6, 5, 0.6))
    s.stats_begin(profile_axis=1)
    s.stats_sample()
    host, _ = s.stats_profile()
    with torch.device("cuda"):
        there, ns = s.stats_profile()
    s.close()
    assert host.device.type == "cpu" and there.device.type == "cuda"
    assert ns == 1 and torch.equal(there.cpu(), host) and bool((host[:, 0] == 40).all())
