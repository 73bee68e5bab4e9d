"""The merge on both sides of its rule for the order of blocks: float32 rows of head_dim 128 below
and from 65,536 on, ragged counts, against the float64 oracle."""
import numpy as np
import pytest
import torch

from oracle import attention as A
from paper_2502_21231_amd import bs_attn as B
from tests.parity_util import check_close, check_lse, f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 5])
@pytest.mark.parametrize("T,hq", [(2047, 32), (2048, 32), (9363, 7), (65537, 1)])
def test_merge_rows(gpu, T, hq, n):
    g = torch.Generator().manual_seed(T + n)
    o = torch.randn(n, T, hq, 128, generator=g)
    l = torch.randn(n, hq, T, generator=g) * 3
    l[n - 1, :, ::5] = -float("inf")
    l[:, 0, 3] = -float("inf")
    out = torch.full((T, hq, 128), 7.0, device=gpu)
    lse = torch.full((hq, T), 7.0, device=gpu)
    B.bs_lse_merge(o.cuda(), l.cuda(), out=out, lse=lse)
    o_ref, l_ref = A.lse_merge(o.numpy(), l.numpy())
    # float32 weights and sums of n <= 5 terms below 6: a few units of 2^-24
    check_close("O", f64(out), o_ref, 1e-5)
    check_lse("LSE", f64(lse), l_ref, 1e-5)
