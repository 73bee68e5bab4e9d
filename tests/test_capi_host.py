"""Host-side checks of the C ABI that need no GPU: the library loads, exports every
entry point the header declares, and rejects bad arguments before touching the device."""
import ctypes
import os
import re

import pytest

from paper_2502_21231_amd import bs_attn as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "bs_attn.h")


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(bs_\w+)\s*\(", text)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(B.LIB_PATH):
        pytest.fail("libbs_attn.so is not built (run __graft_entry__.build())")
    return B.load_library()


def test_exports_every_declared_symbol(lib):
    names = declared_functions()
    assert len(names) == 19, names
    assert set(names) == set(B.EXPORTS)
    for n in names:
        assert hasattr(lib, n), n


FAKE = 4096  # a non-null, aligned address that the validation rejects before any use


def dims(**kw):
    d = dict(total_q=128, total_k=128, hq=4, hkv=2, head_dim=128, dtype=B.BS_BF16)
    d.update(kw)
    return B.bs_dims(**d)


def fwd(lib, d, ws_bytes=1 << 30, scale=0.1, q=FAKE, cu=FAKE):
    return lib.bs_attn_varlen_fwd(ctypes.byref(d), q, FAKE, FAKE, cu, cu, 1, 128, 1, scale, FAKE,
                                  FAKE, FAKE, ws_bytes, None)


def test_rejects_bad_arguments_without_device(lib):
    assert fwd(lib, dims(head_dim=96)) == B.BS_ERR_UNSUPPORTED
    assert "head_dim" in B.bs_last_error()
    assert fwd(lib, dims(dtype=7)) == B.BS_ERR_UNSUPPORTED
    assert fwd(lib, dims(hq=6, hkv=4)) == B.BS_ERR_INVALID_ARG
    assert fwd(lib, dims(hkv=0)) == B.BS_ERR_INVALID_ARG
    assert fwd(lib, dims(hq=8192, hkv=8)) == B.BS_ERR_INVALID_ARG  # above the 4096-head limit
    assert fwd(lib, dims(total_q=-1)) == B.BS_ERR_INVALID_ARG
    assert fwd(lib, dims(), q=None) == B.BS_ERR_INVALID_ARG
    assert "q is NULL" in B.bs_last_error()
    assert fwd(lib, dims(), q=FAKE + 2) == B.BS_ERR_INVALID_ARG
    assert fwd(lib, dims(), scale=float("nan")) == B.BS_ERR_INVALID_ARG
    assert fwd(lib, dims(), scale=-1.0) == B.BS_ERR_INVALID_ARG
    assert fwd(lib, dims(), cu=None) == B.BS_ERR_INVALID_ARG
    assert fwd(lib, dims(), ws_bytes=16) == B.BS_ERR_WORKSPACE
    assert "smaller" in B.bs_last_error()
    d = dims()
    assert lib.bs_lse_merge(ctypes.byref(d), FAKE, FAKE, 0, FAKE, FAKE, None) == B.BS_ERR_INVALID_ARG
    # the packed chunk ops need the per-segment positions as well as cu_seqlens
    assert lib.bs_attn_packed_chunk_fwd(ctypes.byref(d), FAKE, FAKE, FAKE, FAKE, FAKE, None, FAKE, 1,
                                        128, 1, 0.1, FAKE, FAKE, FAKE, 1 << 30, None) == B.BS_ERR_INVALID_ARG
    assert "q_pos" in B.bs_last_error()
    assert lib.bs_attn_packed_chunk_bwd(ctypes.byref(d), FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE,
                                        FAKE, FAKE, FAKE, 1, 128, 1, 0.1, None, FAKE, FAKE, 0, FAKE,
                                        1 << 30, None) == B.BS_ERR_INVALID_ARG
    assert "dq_accum" in B.bs_last_error()
    assert lib.bs_read_device_status(None, None) == B.BS_ERR_WORKSPACE
    assert lib.bs_copy_async(None, FAKE, 64, None) == B.BS_ERR_INVALID_ARG
    assert lib.bs_copy_async(FAKE, FAKE + 32, 64, None) == B.BS_ERR_INVALID_ARG
    assert "overlap" in B.bs_last_error()
    assert lib.bs_copy_async(None, None, 0, None) == B.BS_OK  # nothing to copy: nothing enqueued


def test_softmax_xent_rejects_bad_arguments(lib):
    def xent(rows=4, vocab=1000, dtype=B.BS_BF16, logits=FAKE, labels=FAKE, g=1.0, loss=FAKE,
             dlogits=None):
        return lib.bs_softmax_xent(rows, vocab, dtype, logits, labels, -100, g, loss, None,
                                   dlogits, None)

    assert xent(dtype=5) == B.BS_ERR_UNSUPPORTED
    assert xent(rows=-1) == B.BS_ERR_INVALID_ARG
    assert xent(rows=1 << 30) == B.BS_ERR_INVALID_ARG
    assert xent(vocab=0) == B.BS_ERR_INVALID_ARG
    assert xent(vocab=1 << 31) == B.BS_ERR_INVALID_ARG
    assert xent(g=float("inf")) == B.BS_ERR_INVALID_ARG
    assert xent(logits=None) == B.BS_ERR_INVALID_ARG
    assert xent(loss=None) == B.BS_ERR_INVALID_ARG
    assert xent(logits=FAKE + 1) == B.BS_ERR_INVALID_ARG  # bf16 needs 2-byte alignment
    assert "aligned" in B.bs_last_error()
    assert xent(labels=FAKE + 4) == B.BS_ERR_INVALID_ARG  # int64 labels need 8-byte alignment
    assert xent(loss=FAKE + 2) == B.BS_ERR_INVALID_ARG
    # a gradient buffer that overlaps the logits without being them
    assert xent(dlogits=FAKE + 64) == B.BS_ERR_INVALID_ARG
    assert "overlaps" in B.bs_last_error()
    assert xent(rows=0, logits=None, labels=None, loss=None) == B.BS_OK  # nothing to do


def test_running_merge_rejects_bad_state(lib):
    """The forward steps that fold into a running (O, LSE) need both running buffers; the
    optional final output must not overlap the running O."""
    d = dims()
    qn = 128 * 4 * 128  # total_q * hq * head_dim

    def chunk(o_run=FAKE, lse_run=FAKE, out=None, ws_bytes=1 << 30):
        return lib.bs_attn_chunk_fwd_merge(ctypes.byref(d), FAKE, FAKE, FAKE, 0, 0, 1, 0.1, o_run,
                                           lse_run, 1, out, FAKE, ws_bytes, None)

    assert chunk(o_run=None) == B.BS_ERR_INVALID_ARG
    assert "o_run is NULL" in B.bs_last_error()
    assert chunk(lse_run=None) == B.BS_ERR_INVALID_ARG
    assert "lse_run is NULL" in B.bs_last_error()
    assert chunk(o_run=FAKE + 8) == B.BS_ERR_INVALID_ARG
    assert "aligned" in B.bs_last_error()
    # bf16 out of qn * 2 bytes starting inside the float32 o_run, or o_run starting inside out
    assert chunk(o_run=1 << 20, out=(1 << 20) + qn * 4 - 16) == B.BS_ERR_INVALID_ARG
    assert "overlaps" in B.bs_last_error()
    assert chunk(o_run=(1 << 20) + qn * 2 - 16, out=1 << 20) == B.BS_ERR_INVALID_ARG
    # adjacent buffers pass that check and stop at the (too small) workspace, enqueueing nothing
    assert chunk(o_run=1 << 20, out=(1 << 20) + qn * 4, ws_bytes=16) == B.BS_ERR_WORKSPACE
    assert chunk(o_run=(1 << 20) + qn * 2, out=1 << 20, ws_bytes=16) == B.BS_ERR_WORKSPACE
    assert lib.bs_attn_packed_chunk_fwd_merge(ctypes.byref(d), FAKE, FAKE, FAKE, FAKE, FAKE, None,
                                              FAKE, 1, 128, 1, 0.1, FAKE, FAKE, 0, None, FAKE,
                                              1 << 30, None) == B.BS_ERR_INVALID_ARG
    assert "q_pos" in B.bs_last_error()
    assert lib.bs_attn_packed_chunk_fwd_merge(ctypes.byref(d), FAKE, FAKE, FAKE, FAKE, FAKE, FAKE,
                                              FAKE, 1, 128, 1, 0.1, None, FAKE, 0, None, FAKE,
                                              1 << 30, None) == B.BS_ERR_INVALID_ARG
    assert "o_run is NULL" in B.bs_last_error()


def test_workspace_size_grows_with_problem(lib):
    small = B.bs_attn_workspace_size(B.BS_OP_VARLEN_FWD, dims(), 1, 128)
    big = B.bs_attn_workspace_size(B.BS_OP_VARLEN_FWD, dims(total_q=4096, total_k=4096), 1, 4096)
    bwd = B.bs_attn_workspace_size(B.BS_OP_VARLEN_BWD, dims(total_q=4096, total_k=4096), 1, 4096)
    assert 0 < small < big < bwd
    # the backward holds D [hq, T]; the float32 varlen backward also a dQ accumulator [T, hq, d]
    assert bwd >= 4 * 4096 * 4
    f32 = B.bs_attn_workspace_size(B.BS_OP_VARLEN_BWD,
                                   dims(total_q=4096, total_k=4096, dtype=B.BS_F32), 1, 4096)
    assert f32 >= bwd + 4096 * 4 * 128 * 4
    assert lib.bs_attn_workspace_size(9, ctypes.byref(dims()), 1, 1) == 0
    # the packed chunk backward adds into the caller's dQ accumulator: no dQ buffer of its own
    pk = B.bs_attn_workspace_size(B.BS_OP_PACKED_CHUNK_BWD,
                                  dims(total_q=4096, total_k=4096, dtype=B.BS_F32), 1, 4096)
    assert bwd <= pk < f32


def test_noalloc_forward_rejects_sizes_beyond_its_scratch(lib):
    """The allocation-free forward checks the plan size against its fixed scratch array on the
    host and enqueues nothing: 2^28 bf16 query tokens need 2M work items of 48 B."""
    def call(d, n=1, cu=FAKE):
        return lib.bs_attn_varlen_fwd_noalloc(ctypes.byref(d), FAKE, FAKE, FAKE, cu, cu, n, 1 << 28,
                                              1, 0.1, FAKE, FAKE, None)
    assert call(dims(total_q=1 << 28, total_k=1 << 28)) == B.BS_ERR_WORKSPACE
    assert "allocation-free" in B.bs_last_error()
    assert call(dims(head_dim=96)) == B.BS_ERR_UNSUPPORTED
    assert call(dims(), cu=None) == B.BS_ERR_INVALID_ARG
    assert call(dims(), n=-1) == B.BS_ERR_INVALID_ARG


def test_few_query_forward_is_weighed_against_the_self_planned_one(lib):
    """Which forward a call takes shows in its workspace: the packed op never takes the few-query
    kernel and otherwise asks for the same.  Decoding takes it; short batches of self-attention,
    which the self-planned kernel does in one launch, and long chains that it splits, do not."""
    def few(total_q, total_k, hq, hkv, n, longest):
        d = dims(total_q=total_q, total_k=total_k, hq=hq, hkv=hkv)
        a, b = (B.bs_attn_workspace_size(op, d, n, longest)
                for op in (B.BS_OP_VARLEN_FWD, B.BS_OP_PACKED_CHUNK_FWD))
        return a != b
    assert few(32, 100000, 64, 8, 32, 8192)
    assert few(1, 16384, 64, 8, 1, 16384)
    assert few(70, 4900, 12, 2, 70, 139)
    for call in ((512, 512, 8, 8, 2, 452), (408, 408, 16, 16, 2, 294), (454, 454, 12, 4, 4, 197),
                 (170, 170, 40, 8, 1, 170), (256, 14012, 32, 32, 2, 8192)):
        assert not few(*call), call


def test_short_segments_are_not_split_for_a_loose_max_seqlen(lib):
    """max_seqlen is only a bound (a buffer's or a context's length): 32 segments of 83 tokens on
    average ask for the room of unsplit chains whatever it says, as with their exact maximum."""
    d = dims(total_q=2660, total_k=2660, hq=4, hkv=1)
    size = lambda op, mx: B.bs_attn_workspace_size(op, d, 32, mx)
    for mx in (2660, 131072):
        assert size(B.BS_OP_PACKED_CHUNK_FWD, mx) == size(B.BS_OP_PACKED_CHUNK_FWD, 139)
    # one segment may be as long as its buffer: its chains are split
    one = dims(total_q=2660, total_k=2660, hq=4, hkv=1)
    assert (B.bs_attn_workspace_size(B.BS_OP_PACKED_CHUNK_FWD, one, 1, 131072)
            > B.bs_attn_workspace_size(B.BS_OP_PACKED_CHUNK_FWD, one, 32, 131072))


def test_many_short_segments_stay_with_the_list(lib):
    """Batches of many short sequences, and prompts of tens of tokens, beyond the self-planned lines: the
    few-query kernel would read their keys once per row block.  Decoding of as many takes it."""
    def few(total_q, total_k, hq, hkv, n, longest, head_dim=128):
        d = dims(total_q=total_q, total_k=total_k, hq=hq, hkv=hkv, head_dim=head_dim)
        a, b = (B.bs_attn_workspace_size(op, d, n, longest)
                for op in (B.BS_OP_VARLEN_FWD, B.BS_OP_PACKED_CHUNK_FWD))
        return a != b
    for call in ((7674, 7674, 32, 32, 126, 107), (12454, 12454, 32, 8, 199, 104), (9074, 9074, 64, 8, 178, 88, 64),
                 (889, 54580, 16, 16, 39, 2193), (268, 21591, 32, 32, 16, 2119, 64)):
        assert not few(*call), call
    for call in ((114, 5380, 64, 64, 114, 79), (192, 10544, 64, 64, 192, 95), (344, 25356, 16, 8, 344, 120)):
        assert few(*call), call
