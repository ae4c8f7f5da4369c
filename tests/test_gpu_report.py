"""The acknowledgement report at the edges of its segments (32768 bits, one workgroup each): by many workgroups, by one
(calls without scratch words: captured ones here), and with every workgroup counting the others' segments itself."""
import ctypes as C

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
SEG = 32768


def patterns(n, g):
    yield "none", np.zeros(n, dtype=np.uint8)
    yield "all", np.ones(n, dtype=np.uint8)
    yield "every other", (np.arange(n) % 2).astype(np.uint8)                 # as many runs as there can be
    yield "every other from 0", (np.arange(n) % 2 == 0).astype(np.uint8)
    b = np.ones(n, dtype=np.uint8)
    b[[i for i in (SEG - 1, 2 * SEG, 64 * SEG, 65 * SEG - 1, 256 * SEG, n - 1) if i < n]] = 0   # runs that end and begin at segment edges
    yield "edges", b
    b = np.zeros(n, dtype=np.uint8)
    b[n // 3: n - n // 5] = 1                                                # one run over several segments, most of them without an edge
    yield "one run", b
    yield "random", (g.random(n, dtype=np.float32) < 0.97).astype(np.uint8)
    yield "few holes", (g.random(n, dtype=np.float32) < 0.9995).astype(np.uint8)


def many_workgroups(lib, dev, n_bits, rep, room):
    lib.uccl_dedup_report(dev, n_bits, rep, room)


def one_workgroup(lib, dev, n_bits, rep, room):
    """Under capture there are no scratch words."""
    import torch
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        lib.uccl_dedup_report(dev, n_bits, rep, room)
    graph.replay()
    torch.cuda.synchronize()


def recount(lib, dev, n_bits, rep, room):
    import torch
    from paper_2504_17307_amd.build import PROBE_LIB
    f = C.CDLL(PROBE_LIB).uccl_probe_report
    f.restype, f.argtypes = C.c_int, [C.c_void_p, C.c_uint64, C.c_void_p, C.c_uint32, C.c_void_p, C.c_void_p]
    words = torch.zeros(4 * (n_bits // SEG + 1), dtype=torch.int64, device="cuda")
    assert f(dev.data_ptr(), n_bits, rep.data_ptr(), room, words.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()


SMALL = [SEG - 1, SEG, SEG + 1, 2 * SEG, 2 * SEG + 33, 5 * SEG - 31, 48 * SEG + 7]
LARGE = [65 * SEG, 257 * SEG - 5, 600 * SEG + 1]          # segments before one's own: over one wavefront's lanes, over 256, more than twice that
# what a wavefront of the one workgroup walks: one step of 256 words, several, a second and a third batch of 12
WALKS = [SEG + 1, 3 * SEG + 5, 1 << 21, 4_000_037, 65 * SEG, 5_500_000]


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("how,n_bits", [(many_workgroups, n) for n in SMALL + LARGE] + [(one_workgroup, n) for n in WALKS]
                         + [(recount, n) for n in SMALL[2:] + LARGE[:2]])
def test_report(gpu_lib, how, n_bits, shift):
    """`shift`: the bitmap begins that many words off a 16-byte boundary."""
    import torch
    for name, bits in patterns(n_bits, np.random.default_rng(n_bits)):
        b = np.ones((n_bits + 31) // 32 * 32 + 64, dtype=np.uint8)           # bits past the end must be ignored
        b[:n_bits] = bits
        words = np.packbits(b, bitorder="little").view(np.uint32)
        dev = torch.from_numpy(np.concatenate([np.full(4, 0xFFFFFFFF, dtype=np.uint32)[:shift], words]).view(np.int32)).cuda()[shift:]
        assert dev.data_ptr() % 16 == 4 * shift
        for room in (0, 5, 700, 70000):                                      # 700: cuts in the middle of a walk
            ca, na, nr, rg = oracle.ack_report(words, n_bits, room)
            rep = torch.full((32 + 16 * room + 16,), 0xCD, dtype=torch.uint8, device="cuda")
            print(how.__name__, n_bits, shift, name, room, flush=True)
            torch.cuda.synchronize()
            how(gpu_lib, dev, n_bits, rep, room)
            raw = rep.cpu().numpy()
            assert [int(x) for x in raw[:16].view(np.uint64)] == [ca, na]
            assert [int(x) for x in raw[16:24].view(np.uint32)] == [nr, int(na == n_bits)]
            listed = min(nr, room)
            assert np.array_equal(raw[32:32 + 16 * listed].view(np.uint64).reshape(-1, 2), rg)
            assert np.all(raw[32 + 16 * listed:] == 0xCD), "wrote past the ranges there are"


def test_report_under_capture(gpu_lib):
    """A captured report has no scratch words and is one workgroup's work; replayed after the bitmap has changed,
    it gives what the eager call gives."""
    import torch
    n_bits, g = 3 * SEG + 5, np.random.default_rng(3)
    bitmap = torch.zeros((n_bits + 31) // 32, dtype=torch.int32, device="cuda")
    captured, eager = (torch.zeros(4 + 2 * 600, dtype=torch.int64, device="cuda") for _ in range(2))
    gpu_lib.uccl_dedup_report(bitmap, n_bits, eager, 600)   # the region exists
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        gpu_lib.uccl_dedup_report(bitmap, n_bits, captured, 600)
    for trial in range(4):
        bits = (g.random(len(bitmap) * 32) < 0.99).astype(np.uint8)
        bitmap.copy_(torch.from_numpy(np.packbits(bits, bitorder="little").view(np.int32).copy()))
        captured.zero_(), eager.zero_()
        graph.replay()
        gpu_lib.uccl_dedup_report(bitmap, n_bits, eager, 600)
        torch.cuda.synchronize()
        assert torch.equal(captured, eager) and int(eager[2]) & 0xFFFFFFFF > 100, trial
