"""Timed cases of the library's public entry points.

Each case is one piece of work that a program built on this package has it do: the attention of
a training step over a packed buffer, a device's share of a context-parallel ring, a serving
step over a key/value cache, the merge of ring partials, the loss head.  `listed()` names the
cases, `draw()` makes more of the same ranges, `prepare()` makes what the program holds before
the call (inputs drawn on the GPU, outputs and workspaces that it keeps), `run()` is one pass,
`exact()` the same result in float64 by plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2502_21231_amd import bs_attn as B
from paper_2502_21231_amd import inputs
from paper_2502_21231_amd.ring import ChunkRing

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # The headline training step: one 32K-token buffer of log-normal lengths, 7B-shaped heads.
        dict(name="train_packed_32k", kind="train", mix="lognormal", total=32768, median=1024,
             lens_seed=0, hq=32, hkv=32, d=128, dtype="bf16", causal=True),
        # The largest step: a long-tailed 128K-token buffer with 32K..64K sequences among short
        # ones, 70B-shaped grouped-query heads.
        dict(name="train_long_gqa_128k", kind="train", mix="long", total=131072, median=0,
             lens_seed=0, hq=64, hkv=8, d=128, dtype="bf16", causal=True),
        # The smallest step: two short sequences on a few heads (one rank of a tensor-parallel
        # group, the last micro-batch of an epoch, a unit test of a training loop).
        dict(name="train_small_512", kind="train", mix="lognormal", total=512, median=256,
             lens_seed=1, hq=8, hkv=8, d=128, dtype="bf16", causal=True),
        # An 8K-token micro-batch of a small model with 64-wide heads.
        dict(name="train_d64_8k", kind="train", mix="lognormal", total=8191, median=768,
             lens_seed=7, hq=16, hkv=16, d=64, dtype="bf16", causal=True),
        # A full-precision step (reference runs and convergence checks in float32).
        dict(name="train_f32_2k", kind="train", mix="lognormal", total=2048, median=512,
             lens_seed=5, hq=8, hkv=4, d=64, dtype="f32", causal=True),
        # One device's share of a ring over a long sequence: the own shard and three past ones,
        # received on a copy stream, running merge, backward.
        dict(name="ring_4x4k", kind="ring", shard=4096, n=4, hq=32, hkv=32, d=128, dtype="bf16"),
        # One device's share of a zig-zag split packed batch (two parts of each subsequence),
        # 141B-shaped grouped-query heads, float32 key/value gradient accumulators.
        dict(name="zigzag_packed_2dev", kind="zigzag", lens="16384,8192,4120,260", n_dev=2, dev=0,
             hq=48, hkv=8, d=128, dtype="bf16"),
        # Serving, decode: one new token of each of 32 sequences over its cache.
        dict(name="serve_decode_32", kind="serve", seqs=32, q_max=1, past=8192, lens_seed=4,
             hq=64, hkv=8, d=128, dtype="bf16"),
        # Serving, prefill: ragged prompts, the later part of each over what is cached already.
        dict(name="serve_prefill_16", kind="serve", seqs=16, q_max=1024, past=2048, lens_seed=5,
             hq=32, hkv=8, d=128, dtype="bf16"),
        # Ring partials combined after the last step instead of as they arrive.
        dict(name="merge_8x8k", kind="merge", n=8, tokens=8192, hq=32, d=128, dtype="bf16"),
        # The loss head over the 128,256-entry vocabulary.
        dict(name="xent_4k_128256", kind="xent", rows=4096, vocab=128256, dtype="bf16", grad=True),
        # The loss head of an odd vocabulary (rows without 16-byte alignment).
        dict(name="xent_2k_32003", kind="xent", rows=2048, vocab=32003, dtype="bf16", grad=True),
    ]


HEADS = [(8, 8), (32, 32), (64, 8), (48, 8), (16, 16), (12, 4), (7, 7), (40, 8), (32, 4), (16, 2)]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["train", "train", "train", "ring", "zigzag", "serve", "serve", "merge",
                       "xent", "xent"])
    hq, hkv = rng.choice(HEADS)
    d = rng.choice([128, 128, 64])
    if kind == "train":
        dtype = rng.choice(["bf16"] * 5 + ["f32"])
        total = _log_int(rng, 256, 4096 if dtype == "f32" else 32768)
        return dict(kind=kind, mix="lognormal", total=total,
                    median=_log_int(rng, 64, max(128, total // 4)), lens_seed=rng.randrange(1000),
                    hq=hq, hkv=hkv, d=d, dtype=dtype, causal=rng.random() < 0.85)
    if kind == "ring":
        return dict(kind=kind, shard=_log_int(rng, 500, 8192), n=rng.randint(2, 5), hq=hq, hkv=hkv,
                    d=d, dtype="bf16")
    if kind == "zigzag":
        n_dev = rng.randint(2, 4)
        lens = [2 * n_dev * _log_int(rng, 30, 8192 // n_dev) for _ in range(rng.randint(1, 5))]
        return dict(kind=kind, lens=",".join(str(x) for x in lens), n_dev=n_dev,
                    dev=rng.randrange(n_dev), hq=hq, hkv=hkv, d=d, dtype="bf16")
    if kind == "serve":
        q_max = 1 if rng.random() < 0.5 else _log_int(rng, 2, 1024)
        return dict(kind=kind, seqs=_log_int(rng, 1, 64), q_max=q_max, past=_log_int(rng, 256, 16384),
                    lens_seed=rng.randrange(1000), hq=hq, hkv=hkv, d=d, dtype="bf16")
    if kind == "merge":
        return dict(kind=kind, n=rng.randint(2, 12), tokens=_log_int(rng, 100, 8192), hq=hq, d=d,
                    dtype=rng.choice(["bf16", "bf16", "f32"]))
    vocab = _log_int(rng, 4000, 262144)
    if rng.random() < 0.6:
        vocab = (vocab + 63) // 64 * 64
    rows = _log_int(rng, 64, max(65, min(8192, (1 << 29) // vocab)))
    return dict(kind=kind, rows=rows, vocab=vocab, dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]),
                grad=rng.random() < 0.85)


# ---------------------------------------------------------------- lengths of a case

def _train_lens(c):
    if c["mix"] == "long":
        return inputs.mixed_long_short_lengths(c["lens_seed"], c["total"])
    return inputs.lognormal_packed_lengths(c["lens_seed"], c["total"], c["median"],
                                           lo=min(32, c["total"]), hi=c["total"])


def _serve_lens(c):
    """New and cached tokens of each sequence: cached lengths spread evenly up to `past` over
    their logarithm's upper octaves, new ones up to q_max."""
    rng = np.random.default_rng([c["lens_seed"], 77])
    past = np.exp(rng.uniform(math.log(max(1, c["past"] // 8)), math.log(c["past"]), c["seqs"]))
    new = rng.integers(max(1, c["q_max"] // 8), c["q_max"], size=c["seqs"], endpoint=True)
    return [int(x) for x in new], [int(p) + int(x) for p, x in zip(past, new)]


def _zigzag_lens(c):
    return [int(x) for x in c["lens"].split(",")]


def _zigzag_calls(c):
    """(kv device, segment table) of the ring's packed calls, the own parts first."""
    lens, n, dev = _zigzag_lens(c), c["n_dev"], c["dev"]
    return [((dev - s) % n, inputs.zigzag_step(lens, n, dev, (dev - s) % n, crossed))
            for s in range(n) for crossed in (False, True)]


# ---------------------------------------------------------------- inputs

def _normal(seed, tid, shape, dtype, std=1.0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000003 + tid * 7919)
    x = torch.empty(shape, dtype=dtype, device="cuda")
    flat = x.view(-1)
    for lo in range(0, flat.numel(), 1 << 28):
        hi = min(flat.numel(), lo + (1 << 28))
        flat[lo:hi] = (torch.randn(hi - lo, generator=g, device="cuda") * std).to(dtype)
    return x


def _qkvd(c, seed, tq, tk):
    dt = DTYPES[c["dtype"]]
    return (_normal(seed, 0, (tq, c["hq"], c["d"]), dt), _normal(seed, 1, (tk, c["hkv"], c["d"]), dt),
            _normal(seed, 2, (tk, c["hkv"], c["d"]), dt), _normal(seed, 3, (tq, c["hq"], c["d"]), dt))


def _cu(lens):
    return torch.from_numpy(inputs.cu_seqlens(lens)).cuda()


def _ring_inputs(c, seed):
    dt = DTYPES[c["dtype"]]
    shard, n = c["shard"], c["n"]
    q = _normal(seed, 0, (shard, c["hq"], c["d"]), dt)
    do = _normal(seed, 3, (shard, c["hq"], c["d"]), dt)
    ks = [_normal(seed, 100 + s, (shard, c["hkv"], c["d"]), dt) for s in range(n)]
    vs = [_normal(seed, 200 + s, (shard, c["hkv"], c["d"]), dt) for s in range(n)]
    return q, do, ks, vs, (n - 1) * shard, [(n - 1 - s) * shard for s in range(n)]


def _zigzag_inputs(c, seed):
    """Q and dO of this device's parts, and per device the K and V of its parts."""
    dt = DTYPES[c["dtype"]]
    T = sum(2 * (x // (2 * c["n_dev"])) for x in _zigzag_lens(c))
    q = _normal(seed, 0, (T, c["hq"], c["d"]), dt)
    do = _normal(seed, 3, (T, c["hq"], c["d"]), dt)
    ks = [_normal(seed, 100 + s, (T, c["hkv"], c["d"]), dt) for s in range(c["n_dev"])]
    vs = [_normal(seed, 200 + s, (T, c["hkv"], c["d"]), dt) for s in range(c["n_dev"])]
    return q, do, ks, vs


def _merge_inputs(c, seed):
    n, T, hq, d = c["n"], c["tokens"], c["hq"], c["d"]
    o = _normal(seed, 0, (n, T, hq, d), DTYPES[c["dtype"]], std=0.05)
    # log-sum-exp of some thousands of scores of N(0, 1) vectors
    lse = 9.0 + _normal(seed, 1, (n, hq, T), torch.float32, std=0.5)
    return o, lse


def _xent_inputs(c, seed):
    return inputs.xent_inputs(seed, c["rows"], c["vocab"], dtype=DTYPES[c["dtype"]], device="cuda")


def prepare(case, seed):
    c, kind = case, case["kind"]
    st = dict(case=c)
    if kind == "train":
        lens = _train_lens(c)
        T, nseq, mx = sum(lens), len(lens), max(lens)
        q, k, v, do = _qkvd(c, seed, T, T)
        dims = B.make_dims(q, k)
        st.update(q=q, k=k, v=v, do=do, cu=_cu(lens), mx=mx, out=torch.empty_like(q),
                  lse=torch.empty(c["hq"], T, dtype=torch.float32, device="cuda"),
                  dq=torch.empty_like(q), dk=torch.empty_like(k), dv=torch.empty_like(v),
                  ws_f=B.alloc_workspace(B.BS_OP_VARLEN_FWD, dims, "cuda", nseq, mx),
                  ws_b=B.alloc_workspace(B.BS_OP_VARLEN_BWD, dims, "cuda", nseq, mx))
    elif kind == "serve":
        new, full = _serve_lens(c)
        q, k, v, _ = _qkvd(c, seed, sum(new), sum(full))
        st.update(q=q, k=k, v=v, cq=_cu(new), ck=_cu(full), mx=max(full), out=torch.empty_like(q),
                  lse=torch.empty(c["hq"], sum(new), dtype=torch.float32, device="cuda"))
    elif kind == "ring":
        q, do, ks, vs, q_pos, k_pos = _ring_inputs(c, seed)
        st.update(ring=ChunkRing(q, do, ks, vs, q_pos, k_pos))
    elif kind == "zigzag":
        q, do, ks, vs = _zigzag_inputs(c, seed)
        calls = []
        for dev, (cu_q, cu_k, q_pos, k_pos, rows) in _zigzag_calls(c):
            r = torch.from_numpy(rows).cuda()
            k = ks[dev][r].contiguous()
            calls.append(dict(k=k, v=vs[dev][r].contiguous(), cu_q=torch.from_numpy(cu_q).cuda(),
                              cu_k=torch.from_numpy(cu_k).cuda(), q_pos=torch.from_numpy(q_pos).cuda(),
                              k_pos=torch.from_numpy(k_pos).cuda(),
                              mx=int(max(np.diff(cu_q).max(), np.diff(cu_k).max())),
                              dk=torch.empty(k.shape, dtype=torch.float32, device="cuda"),
                              dv=torch.empty(k.shape, dtype=torch.float32, device="cuda")))
        dims, nseq, mx = B.make_dims(q, calls[0]["k"]), 2 * len(_zigzag_lens(c)), calls[0]["mx"]
        st.update(q=q, do=do, calls=calls, out=torch.empty_like(q), dq=torch.empty_like(q),
                  o_run=torch.empty(q.shape, dtype=torch.float32, device="cuda"),
                  dq_acc=torch.empty(q.shape, dtype=torch.float32, device="cuda"),
                  lse=torch.empty(c["hq"], q.shape[0], dtype=torch.float32, device="cuda"),
                  ws_f=B.alloc_workspace(B.BS_OP_PACKED_CHUNK_FWD, dims, "cuda", nseq, mx),
                  ws_b=B.alloc_workspace(B.BS_OP_PACKED_CHUNK_BWD, dims, "cuda", nseq, mx))
    elif kind == "merge":
        o, lse = _merge_inputs(c, seed)
        st.update(parts=o, lses=lse, out=torch.empty_like(o[0]), lse=torch.empty_like(lse[0]))
    else:
        z, y = _xent_inputs(c, seed)
        n = c["rows"]
        st.update(z=z, y=y, loss=torch.empty(n, dtype=torch.float32, device="cuda"),
                  lse=torch.empty(n, dtype=torch.float32, device="cuda"),
                  dz=torch.empty_like(z) if c["grad"] else None)
    return st


def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind == "train":
        B.bs_attn_varlen_fwd(s["q"], s["k"], s["v"], s["cu"], s["cu"], s["mx"], c["causal"],
                             out=s["out"], lse=s["lse"], workspace=s["ws_f"])
        B.bs_attn_varlen_bwd(s["q"], s["k"], s["v"], s["out"], s["lse"], s["do"], s["cu"], s["cu"],
                             s["mx"], c["causal"], dq=s["dq"], dk=s["dk"], dv=s["dv"],
                             workspace=s["ws_b"])
        return dict(out=s["out"], lse=s["lse"], dq=s["dq"], dk=s["dk"], dv=s["dv"])
    if kind == "serve":
        B.bs_attn_varlen_fwd_noalloc(s["q"], s["k"], s["v"], s["cq"], s["ck"], s["mx"], True,
                                     out=s["out"], lse=s["lse"])
        return dict(out=s["out"], lse=s["lse"])
    if kind == "ring":
        out, lse = s["ring"].forward()
        dq, dk, dv = s["ring"].backward()
        return dict(out=out, lse=lse, dq=dq, dk=dk, dv=dv)
    if kind == "zigzag":
        calls = s["calls"]
        for i, x in enumerate(calls):
            B.bs_attn_packed_chunk_fwd_merge(
                s["q"], x["k"], x["v"], x["cu_q"], x["cu_k"], x["q_pos"], x["k_pos"], x["mx"],
                s["o_run"], s["lse"], i > 0, out=s["out"] if i == len(calls) - 1 else None,
                workspace=s["ws_f"])
        s["dq_acc"].zero_()
        for x in calls:
            x["dk"].zero_()
            x["dv"].zero_()
            B.bs_attn_packed_chunk_bwd(
                s["q"], x["k"], x["v"], s["out"], s["lse"], s["do"], x["cu_q"], x["cu_k"],
                x["q_pos"], x["k_pos"], x["mx"], dq_accum=s["dq_acc"], dk=x["dk"], dv=x["dv"],
                kv_accumulate=True, workspace=s["ws_b"])
        B.bs_dq_finalize(s["dq_acc"], s["dq"])
        return dict(out=s["out"], lse=s["lse"], dq=s["dq"], dk=[x["dk"] for x in calls],
                    dv=[x["dv"] for x in calls])
    if kind == "merge":
        B.bs_lse_merge(s["parts"], s["lses"], out=s["out"], lse=s["lse"])
        return dict(out=s["out"], lse=s["lse"])
    loss, lse, dz = B.bs_softmax_xent(s["z"], s["y"], grad_scale=1.0 / c["rows"], loss=s["loss"],
                                      lse=s["lse"], dlogits=s["dz"], with_grad=c["grad"])
    return dict(loss=loss, lse=lse, dlogits=dz) if c["grad"] else dict(loss=loss, lse=lse)


# ---------------------------------------------------------------- work and tolerance

def _pairs_seg(lq, lk, diag, causal=True):
    """Visible (query, key) pairs: key j and query i with j <= i + diag."""
    if not causal:
        return lq * lk
    i = np.arange(lq, dtype=np.int64)
    return int(np.clip(i + diag + 1, 0, lk).sum())


def _pairs(c):
    kind = c["kind"]
    if kind == "train":
        return sum(_pairs_seg(x, x, 0, c["causal"]) for x in _train_lens(c))
    if kind == "serve":
        return sum(_pairs_seg(a, b, b - a) for a, b in zip(*_serve_lens(c)))
    if kind == "ring":
        s, n = c["shard"], c["n"]
        return s * (s + 1) // 2 + (n - 1) * s * s
    return sum(_pairs_seg(int(cq[i + 1] - cq[i]), int(ck[i + 1] - ck[i]), int(qp[i] - kp[i]))
               for _, (cq, ck, qp, kp, _r) in _zigzag_calls(c) for i in range(len(qp)))


def work(case):
    c, kind = case, case["kind"]
    es = 2 if c["dtype"] == "bf16" else 4
    if kind == "xent":
        n = c["rows"] * c["vocab"]
        return dict(bytes=n * es * (2 if c["grad"] else 1) + c["rows"] * 16, flops=0)
    if kind == "merge":
        rows = c["tokens"] * c["hq"]
        return dict(bytes=(c["n"] + 1) * rows * (c["d"] * es + 4), flops=0)
    hq, hkv, d = c["hq"], c["hkv"], c["d"]
    pairs = _pairs(c)
    if kind == "serve":
        new, full = _serve_lens(c)
        return dict(bytes=2 * sum(new) * hq * d * es + 2 * sum(full) * hkv * d * es
                    + 4 * hq * sum(new), flops=4 * d * hq * pairs)
    if kind == "train":
        tq = tk = sum(_train_lens(c))
        kv_out = es
    elif kind == "ring":
        tq, tk, kv_out = c["shard"], c["shard"] * c["n"], es
    else:
        tq = sum(2 * (x // (2 * c["n_dev"])) for x in _zigzag_lens(c))
        tk, kv_out = tq * c["n_dev"], 4
    # q, dO, out, dQ; lse; k, v; dK, dV
    return dict(bytes=4 * tq * hq * d * es + 4 * hq * tq + 2 * tk * hkv * d * (es + kv_out),
                flops=14 * d * hq * pairs)


def tolerance(case):
    """About four times the error of each path against float64, measured on the listed cases
    and on drawn ones: bf16 attention 2.0e-3 to 3.1e-3 (dK), float32 attention 3e-7 to 7.4e-7
    (dK), merge 1.7e-3, cross-entropy gradients 2.7e-4 (bf16) and 1e-7 (float32)."""
    bf16 = case["dtype"] == "bf16"
    if case["kind"] == "xent":
        return dict(rel=1.2e-3, max=0.02) if bf16 and case["grad"] else dict(rel=2e-6)
    if not bf16:
        return dict(rel=4e-6)
    return dict(rel=7e-3, max=0.05) if case["kind"] == "merge" else dict(rel=1.2e-2, max=0.15)


# ---------------------------------------------------------------- float64 reference

_MOST_SCORES = 2.5e10  # (query, key, head) triples that the float64 reference computes


def _attend(q, do, pieces, causal, scale, grad):
    """Plain softmax attention of the queries q [lq, hq, d] over several key pieces
    (k, v, diag, dk, dv): key j of a piece is visible to query i iff j <= i + diag.  dk, dv of a
    piece are added into.  Returns out, lse, dq in float64."""
    lq, hq, d = q.shape
    hkv = pieces[0][0].shape[1]
    g = hq // hkv
    out = torch.zeros(lq, hq, d, dtype=torch.float64, device=q.device)
    lse = torch.full((hq, lq), -math.inf, dtype=torch.float64, device=q.device)
    dq = torch.zeros_like(out)
    n = max(1, 2048 // g)
    for h in range(hkv):
        heads = slice(h * g, (h + 1) * g)
        kk = [(p[0][:, h].double(), p[1][:, h].double()) for p in pieces]
        for r0 in range(0, lq, n):
            r1 = min(lq, r0 + n)
            rows = torch.arange(r0, r1, device=q.device)
            qb = q[r0:r1, heads].double().transpose(0, 1).reshape(-1, d)
            scores, used = [], []
            for (k, _), (_k, _v, diag, _dk, _dv) in zip(kk, pieces):
                seen = min(k.shape[0], r1 - 1 + diag + 1) if causal else k.shape[0]
                if seen <= 0:
                    used.append(0)
                    continue
                used.append(seen)
                s = (qb @ k[:seen].t()) * scale
                if causal:
                    hidden = torch.arange(seen, device=q.device)[None, :] > rows[:, None] + diag
                    s = s.view(g, r1 - r0, seen).masked_fill_(hidden, -math.inf).view(-1, seen)
                scores.append(s)
            if not scores:
                continue
            m = torch.stack([s.max(1).values for s in scores]).max(0).values
            ps = [s.sub_(m[:, None]).exp_() for s in scores]
            tot = sum(p.sum(1) for p in ps)
            ob = torch.zeros_like(qb)
            seen = [(x, i) for i, x in enumerate(used) if x]
            for p, (x, i) in zip(ps, seen):
                p.div_(tot[:, None])
                ob += p @ kk[i][1][:x]
            out[r0:r1, heads] = ob.view(g, -1, d).transpose(0, 1)
            lse[heads, r0:r1] = (m + tot.log()).view(g, -1)
            if not grad:
                continue
            dob = do[r0:r1, heads].double().transpose(0, 1).reshape(-1, d)
            dvec = (dob * ob).sum(1, keepdim=True)
            dqb = torch.zeros_like(qb)
            for p, (x, i) in zip(ps, seen):
                pieces[i][4][:x, h] += p.t() @ dob
                ds = p.mul_((dob @ kk[i][1][:x].t()).sub_(dvec))
                dqb += ds @ kk[i][0][:x]
                pieces[i][3][:x, h] += (ds.t() @ qb) * scale
            dq[r0:r1, heads] = (dqb * scale).view(g, -1, d).transpose(0, 1)
    return out, lse, dq


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "xent":
        z, y = _xent_inputs(c, seed)
        loss, lse, dz = [], [], []
        for r0 in range(0, c["rows"], 256):
            zb, yb = z[r0:r0 + 256].double(), y[r0:r0 + 256]
            ok = yb != -100
            lb = torch.logsumexp(zb, 1)
            at = yb.clamp(min=0)[:, None]
            loss.append(torch.where(ok, lb - zb.gather(1, at)[:, 0], torch.zeros_like(lb)))
            lse.append(lb)
            if c["grad"]:
                p = (zb - lb[:, None]).exp_()
                p.scatter_add_(1, at, torch.full_like(lb, -1.0)[:, None])
                dz.append((p * ok[:, None] / c["rows"]).to(torch.float64))
        r = dict(loss=torch.cat(loss), lse=torch.cat(lse))
        return dict(r, dlogits=torch.cat(dz)) if c["grad"] else r
    if kind == "merge":
        o, lse = _merge_inputs(c, seed)
        l64 = lse.double()
        tot = torch.logsumexp(l64, 0)
        w = (l64 - tot).exp()  # [n, hq, T]
        out = sum(o[i].double() * w[i].t()[:, :, None] for i in range(c["n"]))
        return dict(out=out, lse=tot)
    if _pairs(c) * c["hq"] > _MOST_SCORES:
        return None
    hq, hkv, d = c["hq"], c["hkv"], c["d"]
    scale = 1.0 / math.sqrt(d)

    def zeros(*shape):
        return torch.zeros(shape, dtype=torch.float64, device="cuda")

    if kind in ("train", "serve"):
        new, full = (_train_lens(c), _train_lens(c)) if kind == "train" else _serve_lens(c)
        tq, tk, grad = sum(new), sum(full), kind == "train"
        q, k, v, do = _qkvd(c, seed, tq, tk)
        out, lse, dq = zeros(tq, hq, d), zeros(hq, tq), zeros(tq, hq, d)
        dk, dv = zeros(tk, hkv, d), zeros(tk, hkv, d)
        a = b = 0
        for lq, lk in zip(new, full):
            sq, sk = slice(a, a + lq), slice(b, b + lk)
            out[sq], lse[:, sq], dq[sq] = _attend(
                q[sq], do[sq], [(k[sk], v[sk], lk - lq, dk[sk], dv[sk])], c.get("causal", True),
                scale, grad)
            a, b = a + lq, b + lk
        return dict(out=out, lse=lse, dq=dq, dk=dk, dv=dv) if grad else dict(out=out, lse=lse)
    if kind == "ring":
        q, do, ks, vs, q_pos, k_pos = _ring_inputs(c, seed)
        dk = [zeros(*k.shape) for k in ks]
        dv = [zeros(*k.shape) for k in ks]
        out, lse, dq = _attend(q, do, [(ks[i], vs[i], q_pos - k_pos[i], dk[i], dv[i])
                                       for i in range(c["n"])], True, scale, True)
        return dict(out=out, lse=lse, dq=dq, dk=dk, dv=dv)
    q, do, ks, vs = _zigzag_inputs(c, seed)
    T = q.shape[0]
    out, lse, dq = zeros(T, hq, d), zeros(hq, T), zeros(T, hq, d)
    calls = []
    for dev, (cu_q, cu_k, q_pos, k_pos, rows) in _zigzag_calls(c):
        r = torch.from_numpy(rows).cuda()
        calls.append((ks[dev][r], vs[dev][r], cu_q, cu_k, q_pos, k_pos, zeros(len(rows), hkv, d),
                      zeros(len(rows), hkv, d)))
    for i in range(2 * len(_zigzag_lens(c))):  # query segment i is the same in every call
        sq = slice(int(calls[0][2][i]), int(calls[0][2][i + 1]))
        pieces = []
        for k, v, _cu, cu_k, q_pos, k_pos, dk, dv in calls:
            sk = slice(int(cu_k[i]), int(cu_k[i + 1]))
            pieces.append((k[sk], v[sk], int(q_pos[i] - k_pos[i]), dk[sk], dv[sk]))
        out[sq], lse[:, sq], dq[sq] = _attend(q[sq], do[sq], pieces, True, scale, True)
    return dict(out=out, lse=lse, dq=dq, dk=[x[6] for x in calls], dv=[x[7] for x in calls])
