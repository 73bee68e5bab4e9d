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


def test_make_dims_reads_the_first_three_sizes():
    """Views with trailing dimensions (a head_dim that is split further) are taken as before."""
    q, k = torch.zeros(5, 4, 64, 1, dtype=torch.bfloat16), torch.zeros(7, 2, 64, 1, dtype=torch.bfloat16)
    d = B.make_dims(q, k)
    assert (d.total_q, d.total_k, d.hq, d.hkv, d.head_dim, d.dtype) == (5, 7, 4, 2, 64, B.BS_BF16)
    d = B.make_dims(q[..., 0], None)
    assert (d.total_q, d.total_k, d.hq, d.hkv, d.head_dim) == (5, 0, 4, 1, 64)
