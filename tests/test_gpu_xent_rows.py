"""Cross-entropy rows that start anywhere: head and tail entries around the 16-byte chunks, the
edges of every register-resident form (chunks of a row: 512, 2048, 4096, 8192, 16384, beyond),
logits and gradients that lie differently modulo 16 bytes, more rows than workgroups.  Bounds of
tests/test_gpu_xent.py."""
import numpy as np
import pytest
import torch

from oracle.xent import softmax_xent
from paper_2502_21231_amd import bs_attn as B
from paper_2502_21231_amd import inputs
from tests.parity_util import check_close, f64
from tests.test_gpu_xent import LSE_TOL, check_row_results

pytestmark = pytest.mark.gpu

CHUNKS = [1, 511, 512, 513, 2048, 2049, 4096, 4097, 8192, 8193, 16384, 16385, 21000]


def place(n, vocab, dtype, shift, gpu):
    """An [n, vocab] contiguous tensor that starts `shift` entries after a 16-byte boundary."""
    buf = torch.full((n * vocab + 64,), 7.0, dtype=dtype, device=gpu)
    return buf[shift:shift + n * vocab].view(n, vocab), buf


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("chunks", CHUNKS)
def test_rows_at_every_alignment(gpu, dtype, chunks):
    per = 8 if dtype == torch.bfloat16 else 4
    rows = 2 * per + 1  # every alignment of an odd row length
    for extra, shift_z, shift_d in ((0, 0, 0), (per - 1, 1, 1), (3, per - 1, per - 1), (1, 0, 1)):
        vocab = chunks * per + extra
        z, y = inputs.xent_inputs(chunks, rows, vocab, dtype=dtype, ignore_every=6)
        y[0], y[1], y[2], y[-1] = 0, vocab - 1, vocab // 2, -100
        zg, zbuf = place(rows, vocab, dtype, shift_z, gpu)
        dg, dbuf = place(rows, vocab, dtype, shift_d, gpu)
        zg.copy_(z)
        before = zbuf.clone()
        g = 0.25
        loss, lse, dz = B.bs_softmax_xent(zg, y.cuda(), -100, g, dlogits=dg)
        check_row_results(f"{chunks} {extra} {shift_z}", loss, lse, dz, z, y.numpy(), g, -100,
                          dtype == torch.bfloat16)
        assert torch.equal(zbuf, before)  # nothing but the gradient's rows was written
        assert (dbuf[:shift_d] == 7).all() and (dbuf[shift_d + rows * vocab:] == 7).all()
        if shift_z != shift_d:
            continue  # (the streamed form; the calls below take the register form)
        l2, s2, none = B.bs_softmax_xent(zg, y.cuda(), -100, g, with_grad=False)
        assert none is None
        if chunks <= 8192:  # beyond, a loss-only call sums in another order
            assert torch.equal(l2, loss) and torch.equal(s2, lse)
        check_row_results("loss only", l2, s2, None, z, y.numpy(), g, -100, False)
        l3, s3, d3 = B.bs_softmax_xent(zg, y.cuda(), -100, g, dlogits=zg)  # in place
        assert torch.equal(l3, loss) and torch.equal(s3, lse) and torch.equal(d3, dz)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_more_rows_than_workgroups(gpu, dtype):
    """Each workgroup walks several rows (the next row's chunks load into this row's registers)."""
    rows, vocab = 5003, 517
    z, y = inputs.xent_inputs(3, rows, vocab, dtype=dtype, ignore_every=50)
    loss, lse, dz = B.bs_softmax_xent(z.cuda(), y.cuda(), -100, 1.0)
    check_row_results("many", loss, lse, dz, z, y.numpy(), 1.0, -100, dtype == torch.bfloat16)


# (chunks of a row at most, rows): every register-resident form with more rows than the workgroups
# that a chip of 256 CUs holds (8 per CU up to 2,048 chunks, 4 to 4,096, 2 to 8,192, then 1; loss
# alone beyond 8,192: 2)
FORMS = [(300, 4200), (2047, 2100), (4000, 1100), (8191, 600), (8750, 600), (16383, 300), (17500, 300)]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("chunks,rows", FORMS)
def test_second_rows_of_every_form(gpu, dtype, chunks, rows):
    """A workgroup's second row (its chunks, label and the entries outside the chunks replace the
    first one's while that is written): odd row lengths, so that heads and chunk counts differ from
    row to row, ignored and out-of-range labels among ordinary ones; out of place, loss only, in
    place.  Sampled rows, most of them beyond the first ones of the workgroups, against the
    oracle."""
    per = 8 if dtype == torch.bfloat16 else 4
    vocab, g, bf16 = chunks * per + per - 3, 0.25, dtype == torch.bfloat16
    zg, _ = inputs.xent_inputs(chunks, rows, vocab, dtype=dtype, device=gpu)
    rng = np.random.default_rng(chunks)
    y = rng.integers(0, vocab, rows)
    y[rng.random(rows) < 0.2] = -100
    y[rng.random(rows) < 0.1] = vocab + 5
    y[-1], y[-2], y[-3], y[-4] = vocab - 1, 0, -100, vocab
    yg = torch.from_numpy(y).cuda()
    grid = {300: 2048, 2047: 2048, 4000: 1024, 8191: 512, 8750: 256}.get(chunks, 256)
    pick = np.unique(np.concatenate([rng.integers(0, rows, 6), rng.integers(grid, rows, 18),
                                     np.arange(rows - 4, rows)]))
    at = torch.from_numpy(pick).cuda()
    z, yp = zg[at].cpu(), y[pick]
    out_of_range = yp >= vocab
    want = np.where(out_of_range, 0, yp)
    l_ref, s_ref, d_ref = softmax_xent(z, want, -100, g)
    d_ref[out_of_range, 0] += g  # no one-hot term

    def check(name, loss, lse, dz):
        loss = f64(loss[at])
        assert np.isnan(loss[out_of_range]).all()
        check_close(name + " loss", loss[~out_of_range], l_ref[~out_of_range], LSE_TOL)
        check_close(name + " lse", f64(lse[at]), s_ref, LSE_TOL)
        if dz is not None:
            check_close(name + " dlogits", f64(dz[at]), d_ref, g * 1e-4, bf16)

    loss, lse, dz = B.bs_softmax_xent(zg, yg, -100, g)
    check("out of place", loss, lse, dz)
    l2, s2, _ = B.bs_softmax_xent(zg, yg, -100, g, with_grad=False)
    check("loss only", l2, s2, None)
    if chunks <= 8192:
        assert torch.equal(l2.view(torch.int32), loss.view(torch.int32)) and torch.equal(s2, lse)
    l3, s3, d3 = B.bs_softmax_xent(zg, yg, -100, g, dlogits=zg)  # in place
    assert torch.equal(l3.view(torch.int32), loss.view(torch.int32)) and torch.equal(s3, lse)
    assert torch.equal(d3, dz)
