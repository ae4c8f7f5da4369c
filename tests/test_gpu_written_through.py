"""Stores that are written through, in every launch that has them (through_shapes.py): chunks that begin on a 128-byte line and off one, ragged
last vectors, records that keep, forward and only forward, buffers that lie across a multiple of 2 GiB; nothing beside the chunks is written."""
import numpy as np
import pytest
import torch

import paper_2504_17307_amd as uccl
import through_shapes

pytestmark = pytest.mark.gpu
DESC = np.dtype([("src_off", "<u8"), ("dst_off", "<u8"), ("out_off", "<u8"), ("len", "<u4"), ("seq", "<u4")])
GATHER_DESC = np.dtype([("dst_off", "<u8"), ("out_off", "<u8"), ("len", "<u4"), ("seq", "<u4"), ("n_src", "<u4"), ("reserved", "<u4"),
                        ("src_off", "<u8", (uccl.UCCL_MAX_SOURCES,))])
FORWARD_ONLY = np.uint64(1 << 63)
TYPES = {"i32": (uccl.UCCL_I32, torch.int32), "bf16": (uccl.UCCL_BF16, torch.bfloat16)}


def _on_gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.uint8).reshape(-1)).cuda()


def _values(n_bytes, dtype, at=None):
    n = n_bytes // dtype.itemsize
    v = torch.randint(-1000, 1000, (n,), device="cuda", dtype=dtype) if dtype == torch.int32 else torch.randn(n, device="cuda", dtype=dtype)
    return v if at is None else at[:n * dtype.itemsize].view(dtype).copy_(v)


def _places(d, i, chunk, off_line):
    """A gap after every chunk; of five records one is kept, one relayed, the others are kept and forwarded; of three one is shorter."""
    at = i * np.uint64(chunk + 256) + np.uint64(off_line)
    d["dst_off"], d["out_off"], d["seq"] = at, at, i
    d["out_off"][i % 5 == 0] = uccl.UCCL_NO_FORWARD
    d["out_off"][i % 5 == 1] |= FORWARD_ONLY
    d["len"] = chunk - 4 * np.random.default_rng(chunk).integers(0, 600, len(i)) * (i % 3 == 0)


def _expect(d, acc, out, recv, combine):
    """The records one by one; combine(a, j, m): record j's value where the accumulator holds a, m elements."""
    es = acc.element_size()
    for j, x in enumerate(d):
        at, m, forward = int(x["dst_off"]) // es, int(x["len"]) // es, int(x["out_off"])
        t = combine(acc[at:at + m], j, m)
        if forward != uccl.UCCL_NO_FORWARD:
            to = (forward & ~(1 << 63)) // es
            out[to:to + m] = t
        if forward == uccl.UCCL_NO_FORWARD or not forward >> 63:
            acc[at:at + m] = t


def _same(a, b, what):
    assert torch.equal(a.view(torch.uint8).cpu(), b.view(torch.uint8)), what


def _apply(n, chunk, stated, op, dtype, off_line, acc, out, what):
    code, tt = TYPES[dtype]
    recv = _values(n * chunk, tt)
    d = np.zeros(n, dtype=DESC)
    _places(d, np.random.default_rng(n + chunk).permutation(n).astype(np.uint64), chunk, off_line)
    d["src_off"] = np.arange(n) * chunk
    want_acc, want_out, r = acc.cpu(), out.cpu(), recv.cpu()
    per = chunk // tt.itemsize
    _expect(d, want_acc, want_out, r, lambda a, j, m: a + r[j * per:j * per + m] if op == "sum" else r[j * per:j * per + m])
    bitmap = torch.zeros((n + 31) // 32, dtype=torch.int32, device="cuda")
    rec, opts = _on_gpu(d), (chunk, 0) if stated else (0, 0)
    uccl.uccl_chunk_apply_opts(acc, out, recv, rec, n, bitmap, code, uccl.UCCL_SUM if op == "sum" else uccl.UCCL_COPY, opts=opts)
    uccl.uccl_chunk_apply_opts(acc, out, recv, rec, n, bitmap, code, uccl.UCCL_SUM, opts=opts)   # all twice: nothing
    _same(acc, want_acc, what)
    _same(out, want_out, what)


@pytest.mark.parametrize("off_line", [0, 16])
@pytest.mark.parametrize("op,dtype", [("sum", "i32"), ("sum", "bf16"), ("copy", "i32")])
@pytest.mark.parametrize("n,chunk,stated,what", [s[:4] for s in through_shapes.APPLY])
def test_apply(n, chunk, stated, what, op, dtype, off_line):
    size = n * (chunk + 256) + 512
    _apply(n, chunk, stated, op, dtype, off_line, _values(size, TYPES[dtype][1]), _values(size, TYPES[dtype][1]), what)


@pytest.mark.parametrize("n,chunk,stated,what", [s[:4] for s in through_shapes.APPLY if s[0] * s[1] <= 100 << 20])
def test_buffers_across_a_multiple_of_2_gib(n, chunk, stated, what):
    """Bit 31 of the address is set in one half of each written buffer and clear in the other."""
    size = n * (chunk + 256) + 512
    room = torch.empty((1 << 32) + 2 * size, dtype=torch.uint8, device="cuda")
    first = -(-(room.data_ptr() + size) // (1 << 31)) * (1 << 31) - room.data_ptr()   # the boundary, as an offset
    acc, out = (_values(size, torch.int32, room[b - size // 2 // 128 * 128:]) for b in (first, first + (1 << 31)))
    for v in (acc, out):
        assert (v.data_ptr() >> 31) + 1 == (v.data_ptr() + size - 1) >> 31
    _apply(n, chunk, stated, "sum", "i32", 0, acc, out, what)


@pytest.mark.parametrize("off_line", [0, 16])
@pytest.mark.parametrize("dtype", ["i32", "bf16"])
@pytest.mark.parametrize("n,chunk,what", [s[:3] for s in through_shapes.FOLD])
def test_fold(n, chunk, what, dtype, off_line):
    code, tt = TYPES[dtype]
    size = n * (chunk + 256) + 512
    acc, out, recv = _values(size, tt), _values(size, tt), _values(2 * n * chunk, tt)
    d = np.zeros(n, dtype=GATHER_DESC)
    _places(d, np.random.default_rng(n + chunk).permutation(n).astype(np.uint64), chunk, off_line)
    d["n_src"], d["src_off"][:, 0], d["src_off"][:, 1] = 2, np.arange(n) * chunk, (np.arange(n) + n) * chunk
    want_acc, want_out, r = acc.cpu(), out.cpu(), recv.cpu()
    per = chunk // tt.itemsize

    def folded(a, j, m):   # in binary32, rounded once
        wide = torch.int32 if tt == torch.int32 else torch.float32
        return (a.to(wide) + r[j * per:j * per + m].to(wide) + r[(n + j) * per:(n + j) * per + m].to(wide)).to(tt)

    _expect(d, want_acc, want_out, r, folded)
    bitmap = torch.zeros((n + 31) // 32, dtype=torch.int32, device="cuda")
    uccl.uccl_chunk_reduce_gather(acc, out, recv, _on_gpu(d), n, bitmap, code, uccl.UCCL_SUM, opts=(chunk, 0))
    _same(acc, want_acc, what)
    _same(out, want_out, what)
