"""Cross-entropy rows that start anywhere: head and tail entries around the 16-byte chunks, the
edges of every register-resident form (chunks of a row: 512, 2048, 4096, 8192, 16384, beyond),
logits and gradients that lie differently modulo 16 bytes, more rows than workgroups.  Bounds of
tests/test_gpu_xent.py."""
import pytest
import torch

from paper_2502_21231_amd import bs_attn as B
from paper_2502_21231_amd import inputs
from tests.test_gpu_xent import check_row_results

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
