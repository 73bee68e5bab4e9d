"""The forward of few queries per segment over many keys: rows of a KV group packed into one
product block, the keys cut into equal ranges over the workgroups, pieces merged.  Against the
float64 oracle with the bf16 bounds, through both entry points (same bits), and on the general
path that a workspace without room for the pieces takes."""
import numpy as np
import pytest
import torch

from oracle import attention as A
from paper_2502_21231_amd import bs_attn as B
from paper_2502_21231_amd import inputs
from tests.parity_util import TOL, check_close, check_lse, f64, make_qkv, scale_for, to_gpu

pytestmark = pytest.mark.gpu
BF = TOL[torch.bfloat16]

# (query lengths, key lengths): one long segment (many pieces), edges of the 128/256-key blocks,
# segments without keys or queries, more queries than keys, many one-block segments
SHAPES = [
    ([1], [5003]),
    ([1, 1, 1, 1, 1, 1], [1, 127, 128, 129, 1025, 3000]),
    ([2, 0, 3, 1, 4], [255, 77, 0, 257, 2]),
    ([4, 4, 1], [3, 700, 4100]),
    ([1] * 70, list(range(1, 141, 2))),
    ([50, 9], [4000, 600]),  # several 32-row blocks
]


@pytest.mark.parametrize("hq,hkv,d,causal", [(8, 1, 128, True), (8, 8, 64, True), (12, 2, 128, False),
                                             (16, 2, 64, True), (7, 7, 128, True)])
@pytest.mark.parametrize("shape", range(len(SHAPES)))
def test_few_queries_match_oracle(gpu, shape, hq, hkv, d, causal):
    lq, lk = SHAPES[shape]
    cq, ck = (torch.from_numpy(inputs.cu_seqlens(x)) for x in (lq, lk))
    q, k, v, _ = make_qkv(31 + shape, sum(lq), sum(lk), hq, hkv, d, torch.bfloat16, with_do=False)
    qg, kg, vg, cqg, ckg = to_gpu(q, k, v, cq, ck)
    mx, sc = max(lq + lk), scale_for(d)
    o_ref, lse_ref = A.varlen_fwd(q, k, v, cq.numpy(), ck.numpy(), causal, sc)
    dims = B.make_dims(qg, kg)
    size = B.bs_attn_workspace_size(B.BS_OP_VARLEN_FWD, dims, len(lq), mx)
    plan_only = B.bs_attn_workspace_size(B.BS_OP_PACKED_CHUNK_FWD, dims, len(lq), mx)
    assert size > plan_only  # this path's sizes: there is room for the pieces
    got = {}
    for name, bytes_ in (("pieces", size), ("plan", plan_only)):
        ws = torch.empty(bytes_, dtype=torch.uint8, device=gpu)
        out = torch.full_like(qg, 7.0)
        lse = torch.full((hq, sum(lq)), 7.0, device=gpu)
        B.bs_attn_varlen_fwd(qg, kg, vg, cqg, ckg, mx, causal, sc, out=out, lse=lse, workspace=ws)
        assert B.bs_read_device_status(ws) == B.BS_OK
        check_close(name + " O", f64(out), o_ref, BF["o"], bf16_out=True)
        check_lse(name + " LSE", f64(lse), lse_ref, BF["lse"])
        got[name] = (out, lse)
    out = torch.full_like(qg, 7.0)
    lse = torch.full((hq, sum(lq)), 7.0, device=gpu)
    B.bs_attn_varlen_fwd_noalloc(qg, kg, vg, cqg, ckg, mx, causal, sc, out=out, lse=lse)
    assert torch.equal(out.view(torch.int16), got["pieces"][0].view(torch.int16))
    assert torch.equal(lse.view(torch.int32), got["pieces"][1].view(torch.int32))


@pytest.mark.parametrize("n", [257, 1023, 1024, 1025])
def test_many_sequences(gpu, n):
    """Sequences beyond the first wave of the table, and a full table of 1024 (1025: the general
    path); some without keys or queries."""
    hq, hkv, d, sc = 2, 1, 64, scale_for(64)
    rng = np.random.default_rng(n)
    lk = [int(x) for x in rng.integers(0, 60, n)]
    lq = [int(x) for x in rng.integers(0, 3, n)]
    lk[0], lk[255], lk[256], lk[n - 1], lq[n - 1], lq[n // 2] = 0, 300, 0, 77, 1, 0
    cq, ck = (torch.from_numpy(inputs.cu_seqlens(x)) for x in (lq, lk))
    q, k, v, _ = make_qkv(37, sum(lq), sum(lk), hq, hkv, d, torch.bfloat16, with_do=False)
    qg, kg, vg, cqg, ckg = to_gpu(q, k, v, cq, ck)
    dims, mx = B.make_dims(qg, kg), max(lq + lk)
    few, general = (B.bs_attn_workspace_size(op, dims, n, mx)
                    for op in (B.BS_OP_VARLEN_FWD, B.BS_OP_PACKED_CHUNK_FWD))
    assert (few != general) == (n <= 1024)
    out, lse = torch.full_like(qg, 7.0), torch.full((hq, sum(lq)), 7.0, device=gpu)
    B.bs_attn_varlen_fwd(qg, kg, vg, cqg, ckg, mx, True, sc, out=out, lse=lse)
    o_ref, lse_ref = A.varlen_fwd(q, k, v, cq.numpy(), ck.numpy(), True, sc)
    check_close("O", f64(out), o_ref, BF["o"], bf16_out=True)
    check_lse("LSE", f64(lse), lse_ref, BF["lse"])


def test_few_queries_bad_cu_seqlens_writes_nothing(gpu):
    q, k, v, _ = make_qkv(14, 4, 900, 8, 2, 128, torch.bfloat16, with_do=False)
    qg, kg, vg = to_gpu(q, k, v)
    cq = torch.tensor([0, 1, 2, 4], dtype=torch.int32, device=gpu)
    dims = B.make_dims(qg, kg)
    for bad, code in (([0, 600, 500, 900], 2), ([1, 50, 100, 900], 1), ([0, 50, 90, 899], 3),
                      ([0, 10, 890, 900], 4)):
        ck = torch.tensor(bad, dtype=torch.int32, device=gpu)
        ws = B.alloc_workspace(B.BS_OP_VARLEN_FWD, dims, gpu, 3, 850)
        out = torch.full_like(qg, 7.0)
        B.bs_attn_varlen_fwd(qg, kg, vg, cq, ck, 850, True, 0.1, out=out, workspace=ws)
        with pytest.raises(B.BsError) as e:
            B.bs_read_device_status(ws)
        assert e.value.status == B.BS_ERR_DEVICE_STATUS and f"code {code}" in str(e.value)
        assert torch.all(out == 7.0)


def test_few_queries_graph_replays(gpu):
    """Captured and replayed with new lengths and contents in the same buffers."""
    hq, hkv, d, n = 16, 2, 128, 5
    lk0, lk1 = [900, 40, 1300, 7, 257], [10, 1200, 301, 990, 3]
    sc = scale_for(d)
    assert sum(lk0) == sum(lk1)
    cq = torch.arange(n + 1, dtype=torch.int32, device=gpu)
    q, k, v, _ = make_qkv(51, n, sum(lk0), hq, hkv, d, torch.bfloat16, with_do=False)
    qg, kg, vg = to_gpu(q, k, v)
    ck = torch.from_numpy(inputs.cu_seqlens(lk0)).cuda()
    out, lse = torch.empty_like(qg), torch.empty(hq, n, device=gpu)
    call = lambda o, l: B.bs_attn_varlen_fwd_noalloc(qg, kg, vg, cq, ck, 1300, True, sc, out=o, lse=l)
    call(out, lse)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(out, lse)
    for lens in (lk0, lk1, lk0):
        ck.copy_(torch.from_numpy(inputs.cu_seqlens(lens)))
        out.fill_(7.0)
        g.replay()
        torch.cuda.synchronize()
        want, want_l = torch.empty_like(qg), torch.empty(hq, n, device=gpu)
        call(want, want_l)
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(lse, want_l)
        o_ref, _ = A.varlen_fwd(q, k, v, cq.cpu().numpy(), inputs.cu_seqlens(lens), True, sc)
        check_close("O", f64(out), o_ref, BF["o"], bf16_out=True)


def test_max_seqlen_far_above_the_lengths(gpu):
    """max_seqlen is only a bound (a context's length): the pieces follow the longest segment that has
    queries, as with the exact maximum, bit for bit."""
    hq, hkv, d, sc = 32, 8, 128, scale_for(128)
    lk = [int(x) for x in np.random.default_rng(3).integers(1, 700, 67)]
    lk[5], lk[6] = 4000, 6000
    lq = [1 + i % 3 for i in range(67)]
    lq[6] = 0  # the longest has none
    cq, ck = (torch.from_numpy(inputs.cu_seqlens(x)) for x in (lq, lk))
    q, k, v, _ = make_qkv(38, sum(lq), sum(lk), hq, hkv, d, torch.bfloat16, with_do=False)
    qg, kg, vg, cqg, ckg = to_gpu(q, k, v, cq, ck)
    dims, got = B.make_dims(qg, kg), []
    for mx in (max(lk), sum(lk), 131072):
        sizes = [B.bs_attn_workspace_size(op, dims, 67, mx) for op in (B.BS_OP_VARLEN_FWD, B.BS_OP_PACKED_CHUNK_FWD)]
        assert sizes[0] != sizes[1]  # this path
        got.append(B.bs_attn_varlen_fwd(qg, kg, vg, cqg, ckg, mx, True, sc))
    o_ref, lse_ref = A.varlen_fwd(q, k, v, cq.numpy(), ck.numpy(), True, sc)
    check_close("O", f64(got[0][0]), o_ref, BF["o"], bf16_out=True)
    check_lse("LSE", f64(got[0][1]), lse_ref, BF["lse"])
    for out, lse in got[1:]:
        assert torch.equal(out, got[0][0]) and torch.equal(lse, got[0][1])
