"""Stores that are written through: every launch that has them, chunks that begin on a 128-byte line and off one, ragged last vectors,
several buffers' places (bit 31 of an address set and clear); nothing beside the chunks is written."""
import numpy as np
import pytest
import torch

import paper_2504_17307_amd as uccl

pytestmark = pytest.mark.gpu
DESC = np.dtype([("src_off", "<u8"), ("dst_off", "<u8"), ("out_off", "<u8"), ("len", "<u4"), ("seq", "<u4")])
GATHER_DESC = np.dtype([("dst_off", "<u8"), ("out_off", "<u8"), ("len", "<u4"), ("seq", "<u4"), ("n_src", "<u4"), ("reserved", "<u4"),
                        ("src_off", "<u8", (uccl.UCCL_MAX_SOURCES,))])
# records, chunk bytes, and the launch they are meant for
SHAPES = [(57, 65536, "parts"), (300, 32768, "one each"), (200, 16384, "half"), (700, 4096, "group of one vector"), (400, 8192, "group of two"),
          (300, 65536, "group of four"), (3200, 4096, "tiles"), (3200, 8192, "tiles of four"), (800, 131072, "ordered"), (2100, 40960, "one record a tile")]


def _on_gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.uint8).reshape(-1)).cuda()


@pytest.mark.parametrize("off_line", [0, 16])
@pytest.mark.parametrize("op", ["sum", "copy"])
@pytest.mark.parametrize("n,chunk,what", SHAPES)
def test_apply(n, chunk, what, op, off_line):
    g = np.random.default_rng(n + chunk)
    pitch = chunk + 256   # a gap after every chunk
    acc = torch.randint(-1000, 1000, ((n * pitch + 512) // 4,), device="cuda", dtype=torch.int32)
    out = torch.randint(-1000, 1000, ((n * pitch + 512) // 4,), device="cuda", dtype=torch.int32)
    recv = torch.randint(-1000, 1000, (n * chunk // 4,), device="cuda", dtype=torch.int32)
    d = np.zeros(n, dtype=DESC)
    i = g.permutation(n).astype(np.uint64)
    d["src_off"], d["seq"] = np.arange(n) * chunk, i
    d["dst_off"] = i * np.uint64(pitch) + np.uint64(off_line)
    d["out_off"] = i * np.uint64(pitch) + np.uint64(off_line)
    d["out_off"][i % 5 == 0] = uccl.UCCL_NO_FORWARD
    d["len"] = chunk - 4 * g.integers(0, 600, n) * (i % 3 == 0)
    want_acc, want_out = acc.cpu().numpy().copy(), out.cpu().numpy().copy()
    r = recv.cpu().numpy()
    for x in d:
        at, m, s = int(x["dst_off"]) // 4, int(x["len"]) // 4, int(x["src_off"]) // 4
        want_acc[at:at + m] = r[s:s + m] + (want_acc[at:at + m] if op == "sum" else 0)
        if x["out_off"] != uccl.UCCL_NO_FORWARD:
            want_out[at:at + m] = want_acc[at:at + m]
    bitmap = torch.zeros((n + 31) // 32, dtype=torch.int32, device="cuda")
    rec = _on_gpu(d)
    uccl.uccl_chunk_apply_opts(acc, out, recv, rec, n, bitmap, uccl.UCCL_I32, uccl.UCCL_SUM if op == "sum" else uccl.UCCL_COPY, opts=(chunk, 0))
    uccl.uccl_chunk_apply_opts(acc, out, recv, rec, n, bitmap, uccl.UCCL_I32, uccl.UCCL_SUM, opts=(chunk, 0))   # all twice: nothing
    assert np.array_equal(acc.cpu().numpy(), want_acc), what
    assert np.array_equal(out.cpu().numpy(), want_out), what


@pytest.mark.parametrize("off_line", [0, 16])
@pytest.mark.parametrize("n,chunk,what", [(400, 4096, "group"), (3100, 4096, "tiles"), (600, 65536, "one record a tile"), (800, 131072, "ordered")])
def test_fold(n, chunk, what, off_line):
    g = np.random.default_rng(n + chunk)
    pitch = chunk + 256
    acc = torch.randint(-1000, 1000, ((n * pitch + 512) // 4,), device="cuda", dtype=torch.int32)
    recv = torch.randint(-1000, 1000, (2 * n * chunk // 4,), device="cuda", dtype=torch.int32)
    d = np.zeros(n, dtype=GATHER_DESC)
    i = g.permutation(n).astype(np.uint64)
    d["dst_off"], d["out_off"], d["seq"], d["n_src"] = i * np.uint64(pitch) + np.uint64(off_line), uccl.UCCL_NO_FORWARD, i, 2
    d["len"] = chunk - 4 * g.integers(0, 600, n) * (i % 3 == 0)
    d["src_off"][:, 0], d["src_off"][:, 1] = np.arange(n) * chunk, (np.arange(n) + n) * chunk
    want, r = acc.cpu().numpy().copy(), recv.cpu().numpy()
    for x in d:
        at, m = int(x["dst_off"]) // 4, int(x["len"]) // 4
        for s in x["src_off"][:2] // 4:
            want[at:at + m] += r[int(s):int(s) + m]
    bitmap = torch.zeros((n + 31) // 32, dtype=torch.int32, device="cuda")
    uccl.uccl_chunk_reduce_gather(acc, None, recv, _on_gpu(d), n, bitmap, uccl.UCCL_I32, uccl.UCCL_SUM, opts=(chunk, 0))
    assert np.array_equal(acc.cpu().numpy(), want), what
