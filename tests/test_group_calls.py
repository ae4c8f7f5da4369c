"""Calls whose records are decided 64 at a time (chunk_group_kernel): the rule that picks them (CPU), and parity at
the edges of groups, parts, trips and record counts (GPU).  Results never depend on the stated chunk size, so small records
reach every branch."""
import ctypes as C

import numpy as np
import pytest

import oracle
import paper_2504_17307_amd as pkg
from randstream import random_stream
from synth.layout import DESC, GATHER_DESC, NO_FORWARD, FORWARD_ONLY, F32, BF16, F16, I32, SUM, MAX, MIN, COPY, PROD

KiB = 1024


def test_rule():
    grouped = pkg.uccl_launch_grouped
    assert [grouped(n, (4 * KiB, 0)) for n in (191, 192, 3000, 3001)] == [0, 1, 1, 0]
    assert [grouped(n) for n in (191, 192, 640, 641, 1500, 1501, 3000, 3001)] == [0, 4, 4, 3, 3, 2, 2, 0]     # some may be long
    assert [grouped(n, (16 * KiB, 0)) for n in (319, 320, 2560, 2561)] == [0, 1, 1, 0]     # 40 MiB
    assert [grouped(n, (32 * KiB, 0)) for n in (255, 256, 768, 769)] == [0, 2, 2, 0]        # 24 MiB
    assert [grouped(n, (64 * KiB, 0)) for n in (256, 257, 640, 641)] == [0, 4, 4, 0]        # from where they are not cut into parts
    assert grouped(1000, (4 * KiB, 1)) == 0 and grouped(1000, (0, 1)) == 0                   # parts stated
    fold = lambda n, c=None: grouped(n, None if c is None else (c, 0), gather=True)
    assert [fold(n, 4 * KiB) for n in (288, 289, 3000, 3001)] == [0, 1, 1, 0]
    assert [fold(n, 8 * KiB) for n in (288, 289, 640, 641, 1024, 1025)] == [0, 2, 2, 0, 0, 1]
    assert [fold(n, 16 * KiB) for n in (549, 550, 1280, 1281)] == [0, 2, 2, 0] and fold(700, 12 * KiB) == 0    # 20 MiB
    assert [fold(n, 32 * KiB) for n in (512, 513, 896, 897)] == [0, 4, 4, 0]                 # 28 MiB
    assert [fold(n, 128 * KiB) for n in (128, 129, 160, 161, 256, 257, 360, 361)] == [0, 16, 16, 0, 0, 16, 16, 0]
    assert [fold(1, c << 20) for c in (16, 17, 48, 49)] == [0, 2176, 4096, 0] and fold(2, 20 << 20) == 2048 and fold(16, 2 << 20) == 256   # few and large
    assert [fold(n) for n in (256, 257, 800, 801, 3000, 3001)] == [0, 6, 6, 4, 4, 0]         # some may be long
    assert grouped(1000, (4 * KiB, 1), gather=True) == 0
    for n in (1, 2, 7, 16, 60, 128, 160):
        for c in range(1 << 20, 52 << 20, 1 << 20):
            assert n * fold(n, c) <= 4096
    for n in (192, 700, 3000):
        for c in (0, 64, 4 * KiB, 8 * KiB, 9008, 32 * KiB, 128 * KiB, 1 << 20, 2 ** 32 - 1):
            assert not (grouped(n, (c, 0)) and pkg.uccl_launch_ordered(n, (c, 0)))
            assert n * grouped(n, (c, 0)) <= 6000                                           # workgroups without work are few
            assert not (fold(n, c) and pkg.uccl_launch_ordered(n, (c, 0), gather=True)) and n * fold(n, c) <= 12000


def run(w, opts, streams=1, entry=None):
    import torch
    from gpuhelp import to_dev
    acc, recv, descs = to_dev(w["acc"]), to_dev(w["recv"]), to_dev(w["descs"])
    out = torch.full((max(w["out_bytes"], 16),), 0xA5, dtype=torch.uint8, device="cuda")
    bitmap = torch.zeros((w["n_bits"] + 31) // 32, dtype=torch.int32, device="cuda")
    rejected = torch.zeros(1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    for s in [torch.cuda.Stream() for _ in range(streams)]:
        pkg.uccl_chunk_apply_opts(acc, out, recv, descs, len(w["descs"]), bitmap, w["dtype"], w["op"], n_rejected=rejected,
                                  n_bits=w["n_bits"], opts=opts, stream=s)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in (acc, out, bitmap, rejected)]


def expected(w, rejected=0):
    acc, out, seen = w["acc"].copy(), np.full(max(w["out_bytes"], 16), 0xA5, dtype=np.uint8), oracle.new_seen(w["n_bits"])
    oracle.apply(acc, out, w["recv"], w["descs"][w["descs"]["seq"] < w["n_bits"]], seen, w["dtype"], w["op"])
    return [acc.view(np.uint8), out, oracle.pack_bitmap(seen).view(np.int32), np.array([rejected], dtype=np.int32)]


def check(w, opts, rejected=0, streams=1):
    """Against the oracle, and the form it replaces against it too."""
    assert pkg.uccl_launch_grouped(len(w["descs"]), opts) > 0 and pkg.uccl_launch_grouped(len(w["descs"]), (opts[0], 1)) == 0
    exp = expected(w, rejected * streams)
    for how in (opts, (opts[0], 1)):
        for name, g, e in zip(("acc", "out", "bitmap", "rejected"), run(w, how, streams), exp):
            assert np.array_equal(g, e), (name, how)


def edges(n, seed, op=SUM, trip=16384, least=0):
    """n records in shuffled order with repeats, bad sequence numbers, keep / forward / relay; lengths 0 .. 48, around the
    trips of a part, and a few that are longer than all parts of a record."""
    g = np.random.default_rng(seed)
    unique = n - n // 16
    seq = np.concatenate([np.arange(unique), g.integers(0, unique, n - unique)])[g.permutation(n)]
    lens = g.integers(least, 13, unique) * 4
    for at in (1024, 4096, 8192, 16384, trip, 2 * trip, 4 * trip):
        lens[g.integers(0, unique, 8)] = at + np.array([-16, -4, 0, 4, 8, 12, 16, 20])
    at = np.concatenate([[0], np.cumsum((lens + 15) // 16 * 16)])
    d = np.zeros(n, dtype=DESC)
    d["src_off"], d["dst_off"], d["out_off"], d["len"], d["seq"] = at[seq], at[seq], at[seq], lens[seq], seq
    d["out_off"][seq % 3 == 0] = NO_FORWARD
    if op != COPY:
        d["out_off"][seq % 3 == 1] |= np.uint64(FORWARD_ONLY)
    bad = g.random(n) < 0.02
    d["seq"][bad] = unique + 7
    total = int(at[-1]) + 16
    return dict(descs=d, recv=g.random(total // 4, dtype=np.float32), acc=g.random(total // 4, dtype=np.float32), out_bytes=total,
                n_bits=unique, dtype=F32, op=op), int(bad.sum())


@pytest.mark.gpu
@pytest.mark.parametrize("n,chunk", [(192, 0), (193, 4096), (255, 8192), (256, 0), (257, 32768), (320, 16384), (640, 0), (641, 0), (300, 65536),
                                     (160 * 4, 65536), (1500, 0), (1501, 0), (3000, 0), (3000, 4096), (2945, 8192)])
def test_edges(gpu_lib, n, chunk):
    for op in (SUM, COPY):
        w, bad = edges(n, n, op, trip=16384 * pkg.uccl_launch_grouped(n, (chunk, 0)))   # of all parts
        print(n, chunk, op, flush=True)
        check(w, (chunk, 0), rejected=bad, streams=1 + (op == COPY))   # the second stream finds every bit set, or takes its share


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,op", [(F32, SUM), (BF16, SUM), (F16, MAX), (I32, PROD), (F32, MIN), (BF16, COPY)])
def test_random_streams(gpu_lib, dtype, op):
    for seed, chunk in enumerate((0, 4096, 8192, 20000, 140000)):
        w = random_stream(1200 + seed, dtype, op, max_chunks=500, max_len=20000)
        need = {20000: 256, 140000: 192}.get(chunk, 192)
        copies = need // len(w["descs"]) + 1
        w["descs"] = np.concatenate([w["descs"]] * copies)[:3000 if chunk < 9000 else 270]
        print(dtype, op, seed, len(w["descs"]), flush=True)
        check(w, (chunk, 0), streams=1 + seed % 2)


def fold_records(w, n, dtype):
    """The calls' records as folds: records, accumulator, slots, and which records are valid."""
    src, g, es = w["descs"], np.random.default_rng(n), {F32: 4, I32: 4}.get(dtype, 2)
    kind = {F32: np.float32, I32: np.int32, BF16: np.uint16, F16: np.float16}[dtype]
    total = w["out_bytes"]
    draw = {F32: lambda m: g.random(m, dtype=np.float32), I32: lambda m: g.integers(-9, 9, m).astype(np.int32), F16: lambda m: g.random(m).astype(np.float16),
            BF16: lambda m: (g.random(m, dtype=np.float32).view(np.uint32) >> 16).astype(np.uint16)}[dtype]
    acc, recv = draw(total // es).view(kind), draw(3 * total // es).view(kind)
    d = np.zeros(n, dtype=GATHER_DESC)
    for f in ("dst_off", "out_off", "len", "seq"):
        d[f] = src[f]
    many = int(src["seq"].max()) + 1
    d["n_src"] = g.integers(1, 17, many)[src["seq"]]
    d["src_off"] = (g.integers(0, total // 16, (many, 16)).astype(np.uint64) * np.uint64(16))[src["seq"]]
    wrong = g.random(many)[src["seq"]] < 0.05
    d["src_off"][wrong, d["n_src"][wrong] - 1] += 8                                              # the last one that is named
    d["src_off"][d["n_src"] < 16, 15] += 8                                                       # one that is not
    good = ~wrong & (d["seq"] < w["n_bits"])
    return d, acc, recv, good


@pytest.mark.gpu
@pytest.mark.parametrize("n,chunk,dtype,op", [(257, 0, F32, SUM), (800, 0, BF16, SUM), (289, 4096, F32, MAX), (320, 8192, BF16, SUM), (550, 16384, F16, MIN),
                                              (513, 32768, I32, PROD), (257, 65536, F32, SUM), (801, 0, BF16, MAX), (3000, 0, F32, SUM), (3000, 4096, F32, SUM),
                                              (1, 48 << 20, F32, SUM), (2, 20 << 20, F16, MAX), (16, 2 << 20, BF16, SUM), (63, 300 << 10, I32, SUM), (130, 200 << 10, F32, MIN)])
def test_folds(gpu_lib, n, chunk, dtype, op):
    """One to sixteen sources, repeats, keep / forward / relay, records with a bad source or sequence number; against the oracle,
    and the form it replaces against it too."""
    import torch
    from gpuhelp import to_dev
    w, _ = edges(n, n + 2, trip=4096 * pkg.uccl_launch_grouped(n, (chunk, 0), gather=True))      # of all parts
    d, acc, recv, good = fold_records(w, n, dtype)
    total = w["out_bytes"]
    e, o, seen = acc.copy(), np.full(total, 0xA5, dtype=np.uint8), oracle.new_seen(w["n_bits"])
    oracle.reduce_gather(e, o, recv, d[good], seen, dtype, op)
    assert pkg.uccl_launch_grouped(n, (chunk, 0), gather=True) > 0 and pkg.uccl_launch_grouped(n, (chunk, 1), gather=True) == 0
    for opts in ((chunk, 0), (chunk, 1)):
        print(n, chunk, dtype, op, opts, flush=True)
        da, do = to_dev(acc), torch.full((total,), 0xA5, dtype=torch.uint8, device="cuda")
        bitmap, rejected = torch.zeros((w["n_bits"] + 31) // 32, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
        for again in range(2):                                                                   # the second call finds every bit set
            pkg.uccl_chunk_reduce_gather(da, do, to_dev(recv), to_dev(d), n, bitmap, dtype, op, n_rejected=rejected, n_bits=w["n_bits"], opts=opts)
            torch.cuda.synchronize()
        assert np.array_equal(da.cpu().numpy(), e.view(np.uint8)) and np.array_equal(do.cpu().numpy(), o), opts
        assert np.array_equal(bitmap.cpu().numpy(), oracle.pack_bitmap(seen).view(np.int32)) and int(rejected) == 2 * int((~good).sum())


@pytest.mark.gpu
@pytest.mark.parametrize("n,parts", [(1, 1), (64, 3), (65, 1), (300, 4), (2048, 2)])
def test_late_decisions(gpu_lib, n, parts):
    """Nobody leads: every group is decided by whichever wavefront has waited long enough, once."""
    import torch
    from gpuhelp import to_dev
    from paper_2504_17307_amd.build import PROBE_LIB
    f = C.CDLL(PROBE_LIB).uccl_probe_group
    f.argtypes = [C.c_void_p] * 4 + [C.c_uint32, C.c_void_p, C.c_uint64, C.c_void_p, C.c_uint32, C.c_void_p, C.c_uint64, C.c_void_p]
    w, bad = edges(n, n + 1, trip=4096, least=1) if n > 1 else (dict(descs=np.array([(0, 0, NO_FORWARD, 32, 0)], dtype=DESC), recv=np.ones(8, np.float32),
                                                                     acc=np.ones(8, np.float32), out_bytes=16, n_bits=1, dtype=F32, op=SUM), 0)
    d = w["descs"]
    assert all((d["seq"][g:g + 64] < w["n_bits"]).any() for g in range(0, n, 64))               # a group of bad records alone has nobody waiting
    exp = expected(w, bad)
    words = torch.zeros(((n - 1) // 64 + 2) * 16, dtype=torch.int64, device="cuda")
    for tag in (1, 2, 3):                                                                        # stale words of earlier calls
        acc, recv, descs = to_dev(w["acc"]), to_dev(w["recv"]), to_dev(d)
        out = torch.full((max(w["out_bytes"], 16),), 0xA5, dtype=torch.uint8, device="cuda")
        bitmap, rejected = torch.zeros((w["n_bits"] + 31) // 32, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        s = torch.cuda.current_stream().cuda_stream
        print(n, parts, tag, flush=True)
        assert f(acc.data_ptr(), out.data_ptr(), recv.data_ptr(), descs.data_ptr(), n, bitmap.data_ptr(), w["n_bits"], rejected.data_ptr(),
                 parts, words.data_ptr(), tag, s) == 0
        torch.cuda.synchronize()
        for name, g, e in zip(("acc", "out", "bitmap", "rejected"), (acc, out, bitmap, rejected), exp):
            assert np.array_equal(g.cpu().numpy(), e), (name, tag)
        assert int(words[(n - 1) // 64 * 16 + 16]) == 0                                          # nobody gave up


@pytest.mark.gpu
@pytest.mark.parametrize("late", [False, True])
@pytest.mark.parametrize("what", ["one vector", "four vectors", "fold"])
@pytest.mark.parametrize("n,parts,major", [(64, 3, 0), (65, 16, 0), (300, 6, 1), (700, 4, 1), (1500, 2, 1)])
def test_late_decisions_of_every_form(gpu_lib, n, parts, major, what, late):
    """Nobody leads, or the leader begins when another wavefront has: one of them decides, for apply and fold, in either order of
    the parts.  `late`: the first group has bad records only, so nobody waits there and the leader decides after all."""
    import torch
    from gpuhelp import to_dev
    from paper_2504_17307_amd.build import PROBE_LIB
    lib, fold = C.CDLL(PROBE_LIB), what == "fold"
    f = getattr(lib, ("uccl_probe_group_fold" if fold else "uccl_probe_group_apply") + ("_late" if late else ""))
    f.argtypes = [C.c_void_p] * 4 + [C.c_uint32, C.c_void_p, C.c_uint64, C.c_void_p] + [C.c_uint32] * (2 if fold else 3) + [C.c_void_p, C.c_uint64, C.c_void_p]
    w, _ = edges(n, n + 3, trip=parts * (16384 if what == "four vectors" else 4096), least=1)
    if late:
        w["descs"]["seq"][:64] = w["n_bits"] + 3
    d, acc, recv = w["descs"], w["acc"], w["recv"]
    good = d["seq"] < w["n_bits"]
    if fold:
        d, acc, recv, good = fold_records(w, n, F32)
    assert late or all(good[g:g + 64].any() for g in range(0, n, 64))       # a group of bad records alone has nobody waiting
    e, o, seen = acc.copy(), np.full(w["out_bytes"], 0xA5, dtype=np.uint8), oracle.new_seen(w["n_bits"])
    (oracle.reduce_gather if fold else oracle.apply)(e, o, recv, d[good], seen, F32, SUM)
    exp = (e.view(np.uint8), o, oracle.pack_bitmap(seen).view(np.int32), np.array([(~good).sum()], dtype=np.int32))
    words = torch.zeros(((n - 1) // 64 + 2) * 16, dtype=torch.int64, device="cuda")
    for tag in (1, 2, 3):                                                    # stale words of earlier calls
        da, dr, dd = to_dev(acc), to_dev(recv), to_dev(d)
        out = torch.full((w["out_bytes"],), 0xA5, dtype=torch.uint8, device="cuda")
        bitmap, rejected = torch.zeros((w["n_bits"] + 31) // 32, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        print(n, parts, major, what, late, tag, flush=True)
        args = [parts, major] + ([] if fold else [4 if what == "four vectors" else 1])
        assert f(da.data_ptr(), out.data_ptr(), dr.data_ptr(), dd.data_ptr(), n, bitmap.data_ptr(), w["n_bits"], rejected.data_ptr(), *args,
                 words.data_ptr(), tag, torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        for name, g, x in zip(("acc", "out", "bitmap", "rejected"), (da, out, bitmap, rejected), exp):
            assert np.array_equal(g.cpu().numpy(), x), (name, tag)
        assert int(words[(n - 1) // 64 * 16 + 16]) == 0                      # nobody gave up


@pytest.mark.gpu
@pytest.mark.parametrize("n", [192, 641, 2048])
def test_no_allocation_calls(gpu_lib, n):
    """The no-allocation entry point has the same form, eager; captured the one without scratch words, each replay checked."""
    import torch
    from gpuhelp import to_dev
    w, _ = edges(n, n + 4, trip=16384 * pkg.uccl_launch_grouped(n))
    w["descs"] = np.ascontiguousarray(np.resize(w["descs"][w["descs"]["seq"] < w["n_bits"]], n))    # the call is not a checked one
    exp = expected(w)
    recv, descs, acc0 = to_dev(w["recv"]), to_dev(w["descs"]), to_dev(w["acc"])
    sets = [(acc0.clone(), torch.zeros(w["out_bytes"], dtype=torch.uint8, device="cuda"), torch.zeros((w["n_bits"] + 31) // 32, dtype=torch.int32, device="cuda"))
            for _ in range(2)]

    def issue(a, o, b):
        pkg.uccl_dedup_reset(b, w["n_bits"])
        pkg.uccl_chunk_apply_noalloc(a, o, recv, descs, n, b, F32, SUM)
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        issue(*sets[0])
    with torch.cuda.stream(side):
        for replay in range(3):
            for a, o, b in sets:
                a.copy_(acc0), o.fill_(0xA5)
            graph.replay()
            issue(*sets[1])
            side.synchronize()
            for got in sets:
                for name, t, x in zip(("acc", "out", "bitmap"), got, exp):
                    assert np.array_equal(t.cpu().numpy()[:len(x)], x[:len(t)]), (name, replay)
    assert pkg.uccl_claim_timeouts() == 0


@pytest.mark.gpu
def test_threads_that_share_a_stream(gpu_lib):
    """Calls of several threads on one stream share its words: every call has its own outcome."""
    import threading
    import torch
    from gpuhelp import to_dev
    stream, jobs = torch.cuda.Stream(), []
    for k in range(4):
        w, bad = edges(500, 50 + k)
        recv, descs = to_dev(w["recv"]), to_dev(w["descs"])
        sets = [(to_dev(w["acc"]), torch.full((w["out_bytes"],), 0xA5, dtype=torch.uint8, device="cuda"),
                 torch.zeros((w["n_bits"] + 31) // 32, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")) for _ in range(6)]
        jobs.append((w, expected(w, bad), recv, descs, sets))
    torch.cuda.synchronize()

    def work(job):
        w, _, recv, descs, sets = job
        for a, o, b, r in sets:
            pkg.uccl_chunk_apply_opts(a, o, recv, descs, 500, b, F32, SUM, n_rejected=r, n_bits=w["n_bits"], stream=stream)
    threads = [threading.Thread(target=work, args=(j,)) for j in jobs]
    [t.start() for t in threads], [t.join() for t in threads]
    torch.cuda.synchronize()
    for _, exp, _, _, sets in jobs:
        for got in sets:
            for name, t, x in zip(("acc", "out", "bitmap", "rejected"), got, exp):
                assert np.array_equal(t.cpu().numpy(), x), name


@pytest.mark.gpu
def test_captured_and_in_turn_with_calls_that_share_the_words(gpu_lib):
    """Captured: the form without scratch words, each replay checked, with an eager call of the same records, an ordered call
    and a report on the same stream in between."""
    import torch
    from gpuhelp import to_dev
    w, bad = edges(700, 3)
    n, exp = len(w["descs"]), expected(w, bad)
    recv, descs, acc0 = to_dev(w["recv"]), to_dev(w["descs"]), to_dev(w["acc"])
    big, big_bad = edges(4000, 4)
    big_exp = expected(big, big_bad)
    big_recv, big_descs, big_acc0 = to_dev(big["recv"]), to_dev(big["descs"]), to_dev(big["acc"])
    assert pkg.uccl_launch_grouped(n) and pkg.uccl_launch_ordered(4000)
    bufs = lambda x, a: (a.clone(), torch.full((x["out_bytes"],), 0xA5, dtype=torch.uint8, device="cuda"),
                         torch.zeros((x["n_bits"] + 31) // 32, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
    sets, large = [bufs(w, acc0) for _ in range(2)], bufs(big, big_acc0)
    report = torch.zeros(4 + 128, dtype=torch.int64, device="cuda")
    long = torch.full((4096,), -1, dtype=torch.int32, device="cuda")

    def issue(a, o, b, r):
        pkg.uccl_dedup_reset(b, w["n_bits"])
        pkg.uccl_chunk_apply_opts(a, o, recv, descs, n, b, F32, SUM, n_rejected=r, n_bits=w["n_bits"])
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        issue(*sets[0])
    with torch.cuda.stream(side):
        for replay in range(4):
            for a, o, b, r in sets:
                a.copy_(acc0), o.fill_(0xA5), r.zero_()
            a, o, b, r = large
            a.copy_(big_acc0), o.fill_(0xA5), r.zero_()
            graph.replay()
            issue(*sets[1])
            pkg.uccl_dedup_reset(b, big["n_bits"])
            pkg.uccl_chunk_apply_opts(a, o, big_recv, big_descs, 4000, b, F32, SUM, n_rejected=r, n_bits=big["n_bits"])
            pkg.uccl_dedup_report(long, 131072, report, 64)
            side.synchronize()
            for got, want in ((sets[0], exp), (sets[1], exp), (large, big_exp)):
                for name, t, e in zip(("acc", "out", "bitmap", "rejected"), got, want):
                    assert np.array_equal(t.cpu().numpy()[:len(e)], e[:len(t)]), (name, replay)
            assert report[:2].tolist() == [131072, 131072]
    assert pkg.uccl_claim_timeouts() == 0
