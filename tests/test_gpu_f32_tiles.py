"""float32 attention at the edges of its tiles (64-query items split into 32-row blocks, 128-key
tiles of four 32-key blocks; 32-key items over 128-query tiles of four 32-row blocks): every
output against the float64 oracle.  Bound: 1e-5 plus 1e-5 of the reference value (168 units of
2^-24, far above what the at most 300-term sums here reach)."""
import numpy as np
import pytest
import torch

from oracle import attention as A
from paper_2502_21231_amd import bs_attn as B
from paper_2502_21231_amd import inputs
from tests.parity_util import check_close, check_lse, f64, make_qkv, scale_for, to_gpu

pytestmark = pytest.mark.gpu

EDGES = [1, 31, 32, 33, 63, 64, 65, 95, 97, 127, 128, 129, 160, 257]


@pytest.mark.parametrize("d,hq,hkv,causal", [(64, 3, 3, True), (64, 8, 4, True), (128, 6, 2, True),
                                             (128, 8, 8, False), (64, 16, 2, False)])
def test_f32_tile_edges(gpu, d, hq, hkv, causal):
    T, sc = sum(EDGES), scale_for(d)
    cu = torch.from_numpy(inputs.cu_seqlens(EDGES))
    q, k, v, do = make_qkv(21, T, T, hq, hkv, d, torch.float32)
    qg, kg, vg, dog, cug = to_gpu(q, k, v, do, cu)
    out, lse = B.bs_attn_varlen_fwd(qg, kg, vg, cug, cug, max(EDGES), causal, sc)
    o_ref, lse_ref = A.varlen_fwd(q, k, v, cu.numpy(), cu.numpy(), causal, sc)
    check_close("O", f64(out), o_ref, 1e-5, rel=1e-5)
    check_lse("LSE", f64(lse), lse_ref, 1e-5)
    o_in, lse_in = torch.from_numpy(o_ref).float(), torch.from_numpy(lse_ref).float()
    grads = B.bs_attn_varlen_bwd(qg, kg, vg, o_in.cuda(), lse_in.cuda(), dog, cug, cug, max(EDGES),
                                 causal, sc)
    want = A.varlen_bwd(q, k, v, o_in, lse_in, do, cu.numpy(), cu.numpy(), causal, sc)
    for name, g, r in zip(("dQ", "dK", "dV"), grads, want):
        check_close(name, f64(g), r, 1e-5, rel=1e-5)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("tq,tk,diag", [(65, 129, 40), (130, 33, -20), (33, 300, 267), (70, 64, -200)])
def test_f32_chunk_edges(gpu, d, tq, tk, diag):
    """One chunk whose diagonal crosses, misses or clears its tiles; dQ, dK and dV added into
    accumulators that already hold values."""
    hq, hkv, sc = 4, 2, scale_for(d)
    q, k, v, do = make_qkv(22, tq, tk, hq, hkv, d, torch.float32)
    qg, kg, vg, dog = to_gpu(q, k, v, do)
    out, lse = B.bs_attn_chunk_fwd(qg, kg, vg, 1000 + diag, 1000, True, sc)
    o_ref, lse_ref = A.chunk_fwd(q, k, v, 1000 + diag, 1000, True, sc)
    check_close("O", f64(out), o_ref, 1e-5, rel=1e-5)
    check_lse("LSE", f64(lse), lse_ref, 1e-5)
    o_in, lse_in = torch.from_numpy(o_ref).float(), torch.from_numpy(lse_ref).float()
    acc = [torch.full(x.shape, 0.5, device=gpu) for x in (qg, kg, vg)]
    B.bs_attn_chunk_bwd(qg, kg, vg, o_in.cuda(), lse_in.cuda(), dog, 1000 + diag, 1000, True, sc,
                        dq_accum=acc[0], dk=acc[1], dv=acc[2], kv_accumulate=True)
    want = A.chunk_bwd(q, k, v, o_in, lse_in, do, 1000 + diag, 1000, True, sc)
    for name, g, r in zip(("dQ", "dK", "dV"), acc, want):
        check_close(name, f64(g), np.asarray(r) + 0.5, 1e-5, rel=1e-5)


@pytest.mark.parametrize("d,hq,hkv,causal", [(64, 8, 1, True), (128, 6, 2, False)])
def test_f32_split_dkdv(gpu, d, hq, hkv, causal):
    """Few key tiles and a group of heads: each dK/dV item's steps are shared by several workgroups
    (the workspace has room for their sums), or not (a workspace without it)."""
    lens = [500, 1, 333]
    T, sc = sum(lens), scale_for(d)
    cu = torch.from_numpy(inputs.cu_seqlens(lens))
    q, k, v, do = make_qkv(23, T, T, hq, hkv, d, torch.float32)
    o_ref, lse_ref = A.varlen_fwd(q, k, v, cu.numpy(), cu.numpy(), causal, sc)
    o_in, lse_in = torch.from_numpy(o_ref).float(), torch.from_numpy(lse_ref).float()
    want = A.varlen_bwd(q, k, v, o_in, lse_in, do, cu.numpy(), cu.numpy(), causal, sc)
    qg, kg, vg, dog, cug, og, lg = to_gpu(q, k, v, do, cu, o_in, lse_in)
    size = B.bs_attn_workspace_size(B.BS_OP_VARLEN_BWD, B.make_dims(qg, kg), 3, 500)
    for bytes_ in (size, size - 4096):
        ws = torch.empty(bytes_, dtype=torch.uint8, device=gpu)
        got = B.bs_attn_varlen_bwd(qg, kg, vg, og, lg, dog, cug, cug, 500, causal, sc, workspace=ws)
        for name, g, r in zip(("dQ", "dK", "dV"), got, want):
            check_close(name, f64(g), r, 1e-5, rel=1e-5)


@pytest.mark.parametrize("over", ["q", "k", "v", "out", "do", "shifted"])
def test_f32_dq_over_an_input(gpu, over):
    """dq in the place of an input, whole or shifted by some rows into a buffer that both share: the
    gradients of separate buffers, and nothing written where cu_seqlens is rejected."""
    lens, h, d, sc = [150, 0, 33, 257], 4, 64, scale_for(64)
    T, mx = sum(lens), max(lens)
    cu = torch.from_numpy(inputs.cu_seqlens(lens)).cuda()
    q, k, v, do = to_gpu(*make_qkv(25, T, T, h, h, d, torch.float32))
    out, lse = B.bs_attn_varlen_fwd(q, k, v, cu, cu, mx, True, sc)
    want = B.bs_attn_varlen_bwd(q, k, v, out, lse, do, cu, cu, mx, True, sc)
    t = {"q": q, "k": k, "v": v, "out": out, "do": do}
    if over == "shifted":
        both = torch.empty(T + 40, h, d, device=gpu)
        t["q"], dq = both[40:], both[:T]
        t["q"].copy_(q)
    else:
        dq = t[over]
    def bwd(c):
        return B.bs_attn_varlen_bwd(t["q"], t["k"], t["v"], t["out"], lse, t["do"], c, c, mx, True, sc, dq=dq)
    kept = dq.clone()
    bwd(torch.tensor([0, 10, 5, 20, T], dtype=torch.int32, device=gpu))
    assert torch.equal(dq, kept)
    for g, r in zip(bwd(cu), want):
        assert torch.equal(g, r)
