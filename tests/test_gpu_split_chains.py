"""Kernels of few workgroups: they plan for themselves and split each work item's chain of tiles
(key tiles in the forward and dQ, query tiles x heads of the group in dK/dV) over several
workgroups whose float32 partials a second kernel combines.  Every output against the float64
oracle with the bf16 bounds, with a workspace that has room for the partials and with one that
has not, and the device's status for rejected cu_seqlens."""
import numpy as np
import pytest
import torch

from oracle import attention as A
from paper_2502_21231_amd import bs_attn as B
from paper_2502_21231_amd import inputs
from tests.parity_util import TOL, check_close, check_lse, f64, make_qkv, scale_for, to_gpu

pytestmark = pytest.mark.gpu
BF = TOL[torch.bfloat16]


def plan_only(op, dims, nseq):
    """Bytes of a workspace without the partials' room (a header, two int32 arrays, the items and,
    backward, D), from the layout documented in the header."""
    r = lambda x: (x + 255) // 256 * 256
    fwd = -(-dims.total_q // 128) + nseq
    bwd = -(-dims.total_k // 128) + nseq
    n = 256 + r(4 * (nseq + 2)) + r(4 * (nseq + 1))
    if op == B.BS_OP_VARLEN_BWD:
        return n + r(48 * max(fwd, bwd)) + r(4 * dims.hq * dims.total_q)
    return n + r(48 * fwd)


CASES = [  # lengths, hq, hkv, d, causal
    ([1500], 2, 1, 128, True),
    ([1, 700, 0, 129, 64, 900], 1, 1, 64, True),
    ([300, 800, 40], 6, 2, 128, False),
    ([1100, 96, 97], 8, 1, 128, True),
    ([257, 1023], 3, 3, 64, False),
]


@pytest.mark.parametrize("lens,hq,hkv,d,causal", CASES)
def test_split_varlen_matches_oracle(gpu, lens, hq, hkv, d, causal):
    T, n, mx, sc = sum(lens), len(lens), max(lens), scale_for(d)
    cu = torch.from_numpy(inputs.cu_seqlens(lens))
    q, k, v, do = make_qkv(61, T, T, hq, hkv, d, torch.bfloat16)
    qg, kg, vg, dog, cug = to_gpu(q, k, v, do, cu)
    o_ref, lse_ref = A.varlen_fwd(q, k, v, cu.numpy(), cu.numpy(), causal, sc)
    o_in, lse_in = torch.from_numpy(o_ref).to(torch.bfloat16), torch.from_numpy(lse_ref).float()
    want = A.varlen_bwd(q, k, v, o_in, lse_in, do, cu.numpy(), cu.numpy(), causal, sc)
    dims = B.make_dims(qg, kg)
    for op in (B.BS_OP_VARLEN_FWD, B.BS_OP_VARLEN_BWD):
        full, small = B.bs_attn_workspace_size(op, dims, n, mx), plan_only(op, dims, n)
        assert full > small or op == B.BS_OP_VARLEN_FWD  # the chains are split (dK/dV: always)
        for size in (full, small):
            ws = torch.empty(size, dtype=torch.uint8, device=gpu)
            if op == B.BS_OP_VARLEN_FWD:
                out, lse = B.bs_attn_varlen_fwd(qg, kg, vg, cug, cug, mx, causal, sc, workspace=ws)
                check_close("O", f64(out), o_ref, BF["o"], bf16_out=True)
                check_lse("LSE", f64(lse), lse_ref, BF["lse"])
            else:
                got = B.bs_attn_varlen_bwd(qg, kg, vg, o_in.cuda(), lse_in.cuda(), dog, cug, cug, mx,
                                           causal, sc, workspace=ws)
                for name, g, r in zip(("dQ", "dK", "dV"), got, want):
                    check_close(name, f64(g), r, BF["grad"], bf16_out=True)
            assert B.bs_read_device_status(ws) == B.BS_OK


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lens,hq,hkv", [
    ([512, 1, 0, 129, 33], 64, 32),     # 11 items: 704 and 352 workgroups, the longest allowed
    ([40, 300, 64, 7], 94, 47),         # 8 items: 752 and 376, just below 768 and 384
    ([40, 300, 64, 7], 96, 48),         # 768 and 384: by the list
    ([513, 100, 29], 64, 32),           # 9 items: 576 and 288, but one segment is too long
])
def test_more_workgroups_than_slots(gpu, lens, hq, hkv, d):
    """Grids somewhat above what the chip holds at once, on both sides of the rule's lines."""
    T, mx, sc = sum(lens), max(lens), scale_for(d)
    cu = torch.from_numpy(inputs.cu_seqlens(lens))
    q, k, v, do = make_qkv(64, T, T, hq, hkv, d, torch.bfloat16)
    qg, kg, vg, dog, cug = to_gpu(q, k, v, do, cu)
    o_ref, lse_ref = A.varlen_fwd(q, k, v, cu.numpy(), cu.numpy(), True, sc)
    o_in, lse_in = torch.from_numpy(o_ref).to(torch.bfloat16), torch.from_numpy(lse_ref).float()
    want = A.varlen_bwd(q, k, v, o_in, lse_in, do, cu.numpy(), cu.numpy(), True, sc)
    out, lse = B.bs_attn_varlen_fwd(qg, kg, vg, cug, cug, mx, True, sc)
    check_close("O", f64(out), o_ref, BF["o"], bf16_out=True)
    check_lse("LSE", f64(lse), lse_ref, BF["lse"])
    got = B.bs_attn_varlen_bwd(qg, kg, vg, o_in.cuda(), lse_in.cuda(), dog, cug, cug, mx, True, sc)
    for name, g, r in zip(("dQ", "dK", "dV"), got, want):
        check_close(name, f64(g), r, BF["grad"], bf16_out=True)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("tq,tk,diag", [(700, 1300, 600), (130, 2000, 900), (900, 500, -300)])
def test_split_chunks_fold_and_accumulate(gpu, d, tq, tk, diag):
    """Ring steps: the forward folded into a running state (replaced, accumulated, written out in
    bf16), dQ, dK and dV added into accumulators that already hold values."""
    hq, hkv, sc = 4, 2, scale_for(d)
    q, k, v, do = make_qkv(62, tq, tk, hq, hkv, d, torch.bfloat16)
    _, k2, v2, _ = make_qkv(63, tq, tk, hq, hkv, d, torch.bfloat16)
    qg, kg, vg, dog, k2g, v2g = to_gpu(q, k, v, do, k2, v2)
    o_run = torch.full((tq, hq, d), float("nan"), device=gpu)
    l_run = torch.full((hq, tq), float("nan"), device=gpu)
    p1 = A.chunk_fwd(q, k, v, 5000 + diag, 5000, True, sc)
    p2 = A.chunk_fwd(q, k2, v2, 9000, 5000, True, sc)
    B.bs_attn_chunk_fwd_merge(qg, kg, vg, 5000 + diag, 5000, o_run, l_run, False, True, sc)
    check_close("step 1 O", f64(o_run), p1[0], BF["o"])
    check_lse("step 1 LSE", f64(l_run), p1[1], BF["lse"])
    out = torch.empty_like(qg)
    B.bs_attn_chunk_fwd_merge(qg, k2g, v2g, 9000, 5000, o_run, l_run, True, True, sc, out=out)
    o_ref, l_ref = A.lse_merge(np.stack([p1[0], p2[0]]), np.stack([p1[1], p2[1]]))
    check_close("step 2 O", f64(out), o_ref, BF["o"], bf16_out=True)
    check_lse("step 2 LSE", f64(l_run), l_ref, BF["lse"])
    o_in, l_in = torch.from_numpy(o_ref).to(torch.bfloat16), torch.from_numpy(l_ref).float()
    acc = [torch.full(x.shape, 0.5, device=gpu) for x in (qg, kg, vg)]
    B.bs_attn_chunk_bwd(qg, kg, vg, o_in.cuda(), l_in.cuda(), dog, 5000 + diag, 5000, True, sc,
                        dq_accum=acc[0], dk=acc[1], dv=acc[2], kv_accumulate=True)
    want = A.chunk_bwd(q, k, v, o_in, l_in, do, 5000 + diag, 5000, True, sc)
    for name, g, r in zip(("dQ", "dK", "dV"), acc, want):
        check_close(name, f64(g), np.asarray(r) + 0.5, BF["grad"])


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("tq,tk,diag", [(326, 2463, 0), (379, 1569, -127), (200, 900, -500), (1500, 400, -1300)])
def test_split_chunks_that_see_few_keys(gpu, d, tq, tk, diag):
    """Chunks whose offsets hide most keys (all of them in the third): fewer parts than the room
    in the workspace is for."""
    test_split_chunks_fold_and_accumulate(gpu, d, tq, tk, diag)


@pytest.mark.parametrize("n", [65, 255, 256, 257])
def test_many_segments(gpu, n):
    """Segments beyond the first wave, and a full table of 256 (257: by the list), empty ones and
    equal sizes among them: every segment's tiles are found once, whatever its place."""
    hq, hkv, d, sc = 1, 1, 64, scale_for(64)
    lens = [int(x) for x in np.random.default_rng(n).integers(0, 40, n)]
    lens[0], lens[63], lens[64], lens[n - 1] = 0, 200, 7, 131
    lens[n // 2] = 0
    T, mx = sum(lens), max(lens)
    cu = torch.from_numpy(inputs.cu_seqlens(lens))
    q, k, v, do = make_qkv(66, T, T, hq, hkv, d, torch.bfloat16)
    qg, kg, vg, dog, cug = to_gpu(q, k, v, do, cu)
    o_ref, lse_ref = A.varlen_fwd(q, k, v, cu.numpy(), cu.numpy(), True, sc)
    o_in, lse_in = torch.from_numpy(o_ref).to(torch.bfloat16), torch.from_numpy(lse_ref).float()
    want = A.varlen_bwd(q, k, v, o_in, lse_in, do, cu.numpy(), cu.numpy(), True, sc)
    pos = torch.zeros(n, dtype=torch.int64, device=gpu)  # (the varlen entry may take few_bf16.hip)
    out, lse = torch.full_like(qg, 7.0), torch.full((hq, T), 7.0, device=gpu)
    B.bs_attn_packed_chunk_fwd(qg, kg, vg, cug, cug, pos, pos, mx, True, sc, out=out, lse=lse)
    check_close("O", f64(out), o_ref, BF["o"], bf16_out=True)
    check_lse("LSE", f64(lse), lse_ref, BF["lse"])
    got = [torch.full_like(x, 7.0) for x in (qg, kg, vg)]
    B.bs_attn_varlen_bwd(qg, kg, vg, o_in.cuda(), lse_in.cuda(), dog, cug, cug, mx, True, sc, dq=got[0],
                         dk=got[1], dv=got[2])
    for name, g, r in zip(("dQ", "dK", "dV"), got, want):
        check_close(name, f64(g), r, BF["grad"], bf16_out=True)


def test_split_bad_cu_seqlens_writes_nothing(gpu):
    q, k, v, do = make_qkv(64, 900, 900, 2, 1, 128, torch.bfloat16)
    qg, kg, vg, dog = to_gpu(q, k, v, do)
    dims = B.make_dims(qg, kg)
    lse = torch.zeros(2, 900, device=gpu)
    for bad, code in (([0, 600, 500, 900], 2), ([1, 50, 100, 900], 1), ([0, 50, 90, 899], 3),
                      ([0, 10, 890, 900], 4)):
        cu = torch.tensor(bad, dtype=torch.int32, device=gpu)
        for op in (B.BS_OP_VARLEN_FWD, B.BS_OP_VARLEN_BWD):
            ws = B.alloc_workspace(op, dims, gpu, 3, 850)
            outs = [torch.full_like(x, 7.0) for x in (qg, kg, vg)]
            if op == B.BS_OP_VARLEN_FWD:
                B.bs_attn_varlen_fwd(qg, kg, vg, cu, cu, 850, True, 0.1, out=outs[0], workspace=ws)
            else:
                B.bs_attn_varlen_bwd(qg, kg, vg, qg, lse, dog, cu, cu, 850, True, 0.1, dq=outs[0],
                                     dk=outs[1], dv=outs[2], workspace=ws)
            with pytest.raises(B.BsError) as e:
                B.bs_read_device_status(ws)
            assert f"code {code}" in str(e.value)
            assert all(torch.all(x == 7.0) for x in outs)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("hq,hkv", [(8, 8), (4, 1)])
@pytest.mark.parametrize("lk", [[2048], [2000, 1000], [0, 5000, 3]])
def test_no_queries_over_long_keys(gpu, lk, hq, hkv, dtype):
    """Segments that all lack queries (a rank with none of this batch's): nothing to write in the
    forward, a running state without rows left alone, dK = dV = 0."""
    d, n, mx, sc = 128, len(lk), max(lk), scale_for(128)
    cq = torch.zeros(n + 1, dtype=torch.int32, device=gpu)
    ck = torch.from_numpy(inputs.cu_seqlens(lk)).cuda()
    pos = torch.zeros(n, dtype=torch.int64, device=gpu)
    q, k, v, do = to_gpu(*make_qkv(65, 0, sum(lk), hq, hkv, d, dtype))
    dims = B.make_dims(q, k)
    ws = B.alloc_workspace(B.BS_OP_VARLEN_FWD, dims, gpu, n, mx)
    out, lse = B.bs_attn_varlen_fwd(q, k, v, cq, ck, mx, True, sc, workspace=ws)
    assert out.shape == (0, hq, d) and lse.shape == (hq, 0)
    assert B.bs_read_device_status(ws) == B.BS_OK
    B.bs_attn_varlen_fwd_noalloc(q, k, v, cq, ck, mx, True, sc)
    ws = B.alloc_workspace(B.BS_OP_PACKED_CHUNK_FWD, dims, gpu, n, mx)
    B.bs_attn_packed_chunk_fwd(q, k, v, cq, ck, pos, pos, mx, True, sc, workspace=ws)
    assert B.bs_read_device_status(ws) == B.BS_OK
    o_run = torch.empty(0, hq, d, device=gpu)
    for accumulate in (False, True):
        B.bs_attn_packed_chunk_fwd_merge(q, k, v, cq, ck, pos, pos, mx, o_run, lse, accumulate, True,
                                         sc, out=out, workspace=ws)
        assert B.bs_read_device_status(ws) == B.BS_OK
    dk, dv = torch.full_like(k, 7.0), torch.full_like(v, 7.0)
    ws = B.alloc_workspace(B.BS_OP_VARLEN_BWD, dims, gpu, n, mx)
    B.bs_attn_varlen_bwd(q, k, v, out, lse, do, cq, ck, mx, True, sc, dk=dk, dv=dv, workspace=ws)
    assert B.bs_read_device_status(ws) == B.BS_OK
    assert not dk.any() and not dv.any()
