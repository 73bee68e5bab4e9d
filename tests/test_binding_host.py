"""Checks of the Python binding that come before any call into the library (no GPU)."""
import pytest
import torch

from paper_2502_21231_amd import bs_attn as B


def test_host_workspace_is_refused_before_the_library_sees_it(monkeypatch):
    """A workspace on the host has no stream: the binding raises instead of handing its address and
    the current GPU's stream to a device copy."""
    class Untouched:
        def __getattr__(self, name):
            return lambda *a: pytest.fail(f"{name} was called")
    monkeypatch.setattr(B, "load_library", lambda *a: Untouched())
    monkeypatch.setattr(B, "_raw_stream", lambda index: 0)
    with pytest.raises((ValueError, RuntimeError)):  # torch: not a GPU, or no GPU at all
        B.bs_read_device_status(torch.zeros(256, dtype=torch.uint8))
