"""What the library asks of the HIP runtime, call by call: launches, allocations, scratch words.  The runtime is
tests/hip_stub.c, so nothing runs and no GPU is needed; each test's body runs in a process of its own, where
the stub is loaded first and serves the library by its soname."""
import ctypes as C
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import paper_2504_17307_amd as pkg  # noqa: E402

KiB, MiB = 1 << 10, 1 << 20
A, OUT, RECV, DESCS, BITS, REPORT = (0x100000 * k for k in range(1, 7))   # addresses; nothing is read from them


class Runtime:
    """The stub and the library on it.  `launches`: (kernel, grid, block, lds, stream, scratch), one per accepted
    launch; `calls`: the other runtime calls by name.  `answer[name]`: what a call returns (a number or a function
    of its subject); `refuse(kernel, stream, start, stop)`: the launches to turn down."""

    def __init__(self, stub):
        self.stub = C.CDLL(stub, mode=C.RTLD_GLOBAL)
        self.lib = C.CDLL(pkg.LIB_PATH)
        for name, (res, args) in pkg._SIGNATURES.items():
            fn = getattr(self.lib, name)
            fn.restype, fn.argtypes = res, args
        self.launches, self.calls, self.answer, self.refuse = [], [], {}, lambda *a: False
        self.symbols = []   # of the accepted launches, whole
        self.launching = False
        on_launch = C.CFUNCTYPE(C.c_int, C.c_char_p, C.c_uint, C.c_uint, C.c_uint, C.c_void_p, C.POINTER(C.c_void_p), C.c_void_p, C.c_void_p)
        on_call = C.CFUNCTYPE(C.c_int, C.c_char_p, C.c_void_p)
        self.keep = on_launch(self._launch), on_call(self._call)
        self.stub.stub_callbacks(*self.keep)

    def _launch(self, kernel, grid, block, lds, stream, args, start, stop):
        name = next((k for k in KERNELS if k.encode() in kernel), kernel.decode())
        self.launching = True
        if self.refuse(name, stream or 0, start, stop):
            return 1
        scratch = None
        if name in ("chunk_order_kernel", "chunk_ordered_kernel", "gather_order_kernel", "gather_ordered_kernel"):
            words = C.cast(args[1], C.POINTER(C.c_uint64))           # OrderArgs: words, tag
            scratch = words[0], words[1]
        elif name in ("chunk_group_kernel", "gather_group_kernel"):
            words = C.cast(args[0] + 80, C.POINTER(C.c_uint64))       # ClaimArgs, after ten words of Buffers: claims, parts : 16 | tag : 48
            scratch = words[0], words[1] >> 16
        elif name == "ack_segments_kernel":
            scratch = C.cast(args[5], C.POINTER(C.c_uint64))[0], C.cast(args[6], C.POINTER(C.c_uint64))[0]
        self.launches.append((name, grid, block, lds, stream or 0, scratch))
        self.symbols.append(kernel.decode())
        return 0

    def _call(self, name, subject):
        name = name.decode()
        self.calls.append(name)
        a = self.answer.get(name, 0)
        return a(subject or 0) if callable(a) else a

    def apply(self, n, chunk=None, stream=0, op=0, parts=0, dtype=0, out=OUT):
        if chunk is None:
            return self.lib.uccl_chunk_apply(A, out, RECV, DESCS, n, BITS, dtype, op, stream)
        return self.lib.uccl_chunk_apply_opts(A, out, RECV, DESCS, n, BITS, dtype, op, None, None, C.byref(pkg.uccl_launch_opts(chunk, parts)), stream)

    def fold(self, n, chunk, stream=0):
        return self.lib.uccl_chunk_reduce_gather(A, OUT, RECV, DESCS, n, BITS, 0, 0, None, None, C.byref(pkg.uccl_launch_opts(chunk, 0)), stream)

    def report(self, bits, stream=0):
        return self.lib.uccl_dedup_report(BITS, bits, REPORT, 4, stream)

    def kernels(self):
        return [l[0] for l in self.launches]


KERNELS = ("chunk_group_kernel", "gather_group_kernel", "chunk_order_kernel", "chunk_ordered_kernel", "gather_order_kernel", "gather_ordered_kernel", "chunk_flat_kernel", "chunk_few_kernel",
           "chunk_gather_parts_kernel", "chunk_gather_kernel", "ack_segments_kernel", "ack_report_kernel", "fill_words_kernel")


def in_process(scenario, tmp_path):
    stub = str(tmp_path / "libamdhip64.so.7")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-w", "-I/opt/rocm/include", "-Wl,-soname,libamdhip64.so.7",
                           os.path.join(ROOT, "tests", "hip_stub.c"), "-o", stub])
    r = subprocess.run([sys.executable, os.path.abspath(__file__), scenario, stub], cwd=ROOT, capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and "SCENARIO DONE" in r.stdout, r.stdout[-2000:] + r.stderr[-4000:]


def stores_of_cut_calls(rt):
    none, through, by_record = (f"chunk_few_kernelILi256ELi2ENS_5OpF32ILi0EEELNS_7ThroughE{k}ELb1ELb0" for k in (0, 1, 3))
    for n, chunk, parts, stores in ((57, 64 * KiB, 0, through), (254, 66000, 0, through), (254, 66000, 8, through), (255, 66000, 8, none), (1000, 66000, 8, none), (1000, 64 * KiB, 8, through), (1536, 64 * KiB, 8, through), (1537, 64 * KiB, 8, none),
                                    (2048, 128 * KiB + 16, 16, none), (300, 40016, 2, through), (64, None, 0, by_record), (128, None, 0, by_record), (500, 0, 8, by_record)):
        rt.symbols.clear()
        assert rt.apply(n, chunk, parts=parts) == pkg.UCCL_OK
        assert len(rt.symbols) == 1 and stores in rt.symbols[0], (n, chunk, parts, rt.symbols)


def test_cut_calls_write_through_where_they_are_small_or_in_whole_lines(tmp_path):
    """Large chunks that share lines lose by it, up to 1.2 times: stated, the host sees it; not stated, the kernel looks at each record."""
    in_process("stores_of_cut_calls", tmp_path)


def stores_of_the_shapes(rt):
    """The table of calls that are run on a GPU for their stores: each gets the kernel that it is there for."""
    import through_shapes as t
    for n, chunk, stated, name, of_sum, of_copy in t.APPLY:
        for op, kernel, mangled in ((pkg.UCCL_SUM, of_sum, "NS_5OpI32ILi0EEE"), (pkg.UCCL_SUM, of_sum, "NS_4Op16ILi0ENS_9WidenBF16EEE"), (pkg.UCCL_COPY, of_copy, "NS_4CopyE")):
            rt.symbols.clear()
            assert rt.apply(n, chunk if stated else None, op=op, dtype=pkg.UCCL_BF16 if "BF16" in mangled else pkg.UCCL_I32) == pkg.UCCL_OK
            assert kernel is None or kernel.format(op=mangled) in rt.symbols[-1], (name, rt.symbols)
    for n, chunk, name, kernel in t.FOLD:
        rt.symbols.clear()
        assert rt.fold(n, chunk) == pkg.UCCL_OK
        assert kernel.format(op="NS_5OpF32ILi0EEE") in rt.symbols[-1], (name, rt.symbols)


def test_calls_run_for_their_stores_get_the_kernels_they_are_for(tmp_path):
    in_process("stores_of_the_shapes", tmp_path)


def stores_of_large_copies(rt):
    import through_shapes as t
    for n, chunk, out, kernel in ((24576, 4 * KiB, None, t.flat(8, 2, t.BUT_COMBINED)), (24577, 4 * KiB, None, t.flat(8, 2, t.FORWARDED)), (12289, 8 * KiB, OUT, t.flat(4, 2, t.FORWARDED)),
                                  (8192, 12 * KiB + 128, None, t.flat(2, 2, t.FORWARDED)), (6144, 16 * KiB, None, t.few(1024, 1, t.ALL, False)), (6145, 16 * KiB, None, t.few(1024, 1, t.NONE, False)),
                                  (2561, 16 * KiB, OUT, t.few(1024, 1, t.NONE, False))):
        rt.symbols.clear()
        assert rt.apply(n, chunk, op=pkg.UCCL_COPY, out=out) == pkg.UCCL_OK
        assert kernel.format(op="NS_4CopyE") in rt.symbols[-1], (n, chunk, rt.symbols)


def test_large_copies_that_forward_nothing_keep_the_former_stores(tmp_path):
    """Above 96 MiB what lines are shared costs more than writing through gives, up to 1.16 times."""
    in_process("stores_of_large_copies", tmp_path)


def stores_of_large_sums(rt):
    import through_shapes as t
    for n, dtype, mangled, stores in ((24576, pkg.UCCL_F32, "NS_5OpF32ILi0EEE", t.BUT_COMBINED), (24577, pkg.UCCL_F32, "NS_5OpF32ILi0EEE", t.NONE), (24577, pkg.UCCL_I32, "NS_5OpI32ILi0EEE", t.NONE),
                                      (24577, pkg.UCCL_BF16, "NS_4Op16ILi0ENS_9WidenBF16EEE", t.BUT_COMBINED)):
        rt.symbols.clear()
        assert rt.apply(n, 4 * KiB, dtype=dtype) == pkg.UCCL_OK
        assert t.flat(8, 2, stores).format(op=mangled) in rt.symbols[-1], (n, rt.symbols)


def test_large_tiles_of_32_bit_sums_keep_the_former_stores(tmp_path):
    in_process("stores_of_large_sums", tmp_path)


def stores_of_folds_in_tiles(rt):
    for n, chunk, tile, stores in ((16384, 4 * KiB, 8, 17), (65536, 4 * KiB, 8, 17), (8381, 9008, 4, 17), (8382, 9008, 4, 0), (12583, 6000, 4, 0), (600, 66000, 1, 17), (8192, 0, 4, 17)):
        rt.symbols.clear()
        assert rt.fold(n, chunk) == pkg.UCCL_OK
        assert f"chunk_gather_kernelILi1024ELi{tile}ELi2ENS_5OpF32ILi0EEELNS_5StoreE{stores}EE" in rt.symbols[-1], (n, chunk, rt.symbols)


def test_large_folds_of_chunks_that_share_lines_keep_the_default_policy(tmp_path):
    in_process("stores_of_folds_in_tiles", tmp_path)


def refused_counts(rt):
    for n, chunk in ((2 ** 32 - 1, 32 * KiB), (2 ** 32 - 1, 16 * KiB), (2 ** 32 - 1, 128 * KiB), (1 << 23, 128 * KiB), ((1 << 22) + 1, 32 * KiB)):
        assert rt.apply(n, chunk) == pkg.UCCL_ELAUNCH and rt.fold(n, chunk) == pkg.UCCL_ELAUNCH, (n, chunk)
        assert not rt.launches
    assert rt.apply(2 ** 32 - 1) == pkg.UCCL_ELAUNCH and not rt.launches
    # the largest counts that one workgroup per record (or per two) can be launched for are still taken
    assert rt.apply((1 << 22) - 1, 32 * KiB) == pkg.UCCL_OK and set(rt.kernels()) == {"chunk_order_kernel", "chunk_ordered_kernel"}


def test_record_counts_beyond_one_launch_are_refused_and_nothing_is_enqueued(tmp_path):
    """A count that is no count of records (-1, say) comes back as an error also where the call would be streamed in
    destination order, whose launches of 16383 records each would all be accepted."""
    in_process("refused_counts", tmp_path)


def no_allocation(rt):
    rt.apply(57, 64 * KiB), rt.apply(100), rt.apply(5000), rt.apply(8000, 32 * KiB), rt.apply(8000, 128 * KiB, op=pkg.UCCL_COPY)
    rt.fold(8, 128 * KiB), rt.fold(65, 16 * KiB), rt.fold(1024, 128 * KiB)
    rt.report(32768), rt.report(32769), rt.report(1572200)
    rt.lib.uccl_chunk_apply_noalloc(A, OUT, RECV, DESCS, 57, BITS, 0, 0, 0)
    rt.lib.uccl_chunk_scatter(A, RECV, DESCS, 5000, BITS, 0)
    assert {"chunk_few_kernel", "chunk_order_kernel", "gather_order_kernel", "chunk_gather_parts_kernel", "ack_segments_kernel"} <= set(rt.kernels())
    assert not {"hipMalloc", "hipFree", "hipHostMalloc", "hipMemsetAsync", "hipStreamCreateWithFlags", "hipStreamSynchronize"} & set(rt.calls), rt.calls


def test_no_data_path_call_allocates_or_waits(tmp_path):
    """Also not the first one on a device, and not the calls that a caller of the no-allocation entry point makes
    beside it: calls of more records than that takes, and the acknowledgement report."""
    in_process("no_allocation", tmp_path)


def threads_one_after_another(rt):
    import threading
    per_thread = 2
    for _ in range(24):
        t = threading.Thread(target=rt.apply, args=(8000, 32 * KiB, per_thread))
        t.start()
        t.join()
    ordered = [l for l in rt.launches if l[0] == "chunk_order_kernel"]
    regions = [scratch[0] for *_, scratch in ordered]
    assert len(regions) == len(set(regions)) == 16, regions     # the work of an ended thread may still be running
    assert rt.kernels().count("chunk_flat_kernel") == 24 - 16   # the rest: the form that needs none
    assert rt.apply(8000, 32 * KiB, stream=0x7000) == pkg.UCCL_OK and rt.kernels()[-1] == "chunk_ordered_kernel"


def test_a_thread_never_gets_the_scratch_words_of_one_that_has_ended(tmp_path):
    in_process("threads_one_after_another", tmp_path)


def reports_on_many_streams(rt):
    for k in range(80):
        assert rt.report(1572200, stream=0x1000 + 16 * k) == pkg.UCCL_OK
    assert rt.kernels() == ["ack_segments_kernel"] * 64 + ["ack_report_kernel"] * 16
    for k in range(80):   # the streams that move the payload come later
        rt.launches.clear()
        assert rt.apply(57, 64 * KiB, stream=0x9000 + 16 * k) == pkg.UCCL_OK
        assert rt.launches[0][:3] == (("chunk_few_kernel", 57 * 8, 256) if k < 64 else ("chunk_few_kernel", 57, 1024)), k
    rt.launches.clear()
    assert rt.report(1572200, stream=0x1000) == pkg.UCCL_OK and rt.fold(8, 128 * KiB, stream=0x9000) == pkg.UCCL_OK
    assert rt.kernels() == ["ack_segments_kernel", "chunk_gather_parts_kernel"]


def test_streams_that_only_report_leave_cut_calls_their_regions(tmp_path):
    in_process("reports_on_many_streams", tmp_path)


def a_full_queue(rt):
    import threading
    full, other, done = 0x1000, 0x2000, threading.Event()
    waited = []
    rt.refuse = lambda kernel, stream, *_: bool(stream == full and not waited and waited.append(done.wait(10)))
    t = threading.Thread(target=rt.apply, args=(8000, 32 * KiB, full))
    t.start()
    while not rt.launching:
        pass
    assert rt.report(1572200, other) == 0 and rt.apply(8000, 128 * KiB, other) == 0 and rt.apply(57, 64 * KiB, other) == 0 and rt.fold(8, 128 * KiB, other) == 0
    done.set()
    t.join()
    assert waited == [True], "calls on another stream waited for the launch on the first"


def test_a_launch_that_waits_for_its_stream_does_not_hold_up_other_streams(tmp_path):
    in_process("a_full_queue", tmp_path)


def feed_hand_over(rt):
    import numpy as np
    n = 20000                                        # large enough to be copied to device memory before the launch
    d = np.zeros(n, dtype=[("off", "<u8", 3), ("len", "<u4"), ("seq", "<u4")])
    d["seq"], d["len"], d["len"][17] = np.arange(n), 4096, 256 * KiB
    feed = C.c_void_p()
    assert rt.lib.uccl_feed_create(C.byref(feed), A, OUT, RECV, BITS, 0, 0, 3, n, 2, None) == 0
    rt.refuse = lambda kernel, *_: len(rt.launches) > 0              # whatever comes after the first launch of the hand-over
    assert rt.lib.uccl_feed_push(feed, 0, d.ctypes.data, n) == 0
    assert rt.kernels() == ["chunk_flat_kernel"] and rt.launches[0][1] <= n


def test_a_feed_hand_over_is_one_launch_per_lane(tmp_path):
    """All of a hand-over is enqueued or nothing, whatever its size, since it is offered again after an error; and the one
    long record in it, whose length is the hand-over's chunk size, does not multiply the others' workgroups."""
    in_process("feed_hand_over", tmp_path)


def feed_of_hundreds(rt):
    import numpy as np
    rt.answer["hipPointerGetAttributes"] = 1
    d = np.zeros(300, dtype=[("off", "<u8", 3), ("len", "<u4"), ("seq", "<u4")])
    d["seq"], d["len"] = np.arange(300), 4096
    feed = C.c_void_p()
    assert rt.lib.uccl_feed_create(C.byref(feed), A, OUT, RECV, BITS, 0, 0, 3, 3000, 2, None) == 0
    assert rt.lib.uccl_feed_push(feed, 0, d.ctypes.data, 300) == 0 and rt.lib.uccl_feed_flush(feed) == 0
    assert rt.kernels() == ["chunk_flat_kernel"] and "hipPointerGetAttributes" not in rt.calls


def test_a_feed_does_not_ask_where_its_own_pinned_slots_are(tmp_path):
    in_process("feed_of_hundreds", tmp_path)


def unusable_event(rt):
    bad = 0x5000
    rt.refuse = lambda kernel, stream, start, stop: bad in (start, stop)
    for start, stop in ((0x6000, bad), (bad, None), (None, bad)):
        for call in (lambda: rt.apply(8000, 32 * KiB), lambda: rt.apply(40000, 32 * KiB), lambda: rt.fold(1024, 128 * KiB), lambda: rt.apply(5000)):
            rt.lib.uccl_time_next_launch(start, stop)
            assert call() == pkg.UCCL_ELAUNCH and not rt.launches
    rt.lib.uccl_time_next_launch(0x6000, 0x7000)
    events = []
    rt.refuse = lambda kernel, stream, start, stop: events.append((start, stop))
    assert rt.apply(40000, 32 * KiB) == 0 and len(events) == 6
    assert events[0][0] == 0x6000 and events[-1][1] == 0x7000 and not any(start for start, _ in events[1:])


def test_a_timing_event_that_hip_does_not_take_fails_the_call_before_anything_is_enqueued(tmp_path):
    in_process("unusable_event", tmp_path)


def callers_error(rt):
    noalloc = lambda: rt.lib.uccl_chunk_apply_noalloc(A, OUT, RECV, DESCS, 57, BITS, 0, 0, 0)
    rt.lib.uccl_init()
    for capturing, kernels in ((1, ["fill_words_kernel", "chunk_few_kernel"]), (0, ["chunk_few_kernel"])):
        rt.answer["hipStreamIsCapturing"] = capturing
        rt.launches.clear(), rt.calls.clear()
        assert noalloc() == 0 and rt.kernels() == kernels
        assert rt.apply(57, 64 * KiB) == 0 and rt.apply(8000, 32 * KiB) == 0 and rt.fold(8, 128 * KiB) == 0 and rt.report(1572200) == 0
        assert "hipGetLastError" not in rt.calls       # reading it clears it
    rt.answer["hipStreamIsCapturing"] = -1             # the library's own failed query: nothing of that is left behind
    rt.launches.clear(), rt.calls.clear()
    assert noalloc() == 0 and rt.kernels() == ["fill_words_kernel", "chunk_few_kernel"] and rt.calls.count("hipGetLastError") == 1


def test_an_error_that_the_caller_has_pending_is_left_alone(tmp_path):
    in_process("callers_error", tmp_path)


def records_in_host_memory(rt):
    for where in (1, -1):                              # pinned; not known to the runtime
        rt.answer["hipPointerGetAttributes"] = where
        rt.launches.clear()
        rt.apply(8000, 32 * KiB), rt.apply(5000), rt.apply(8000, 128 * KiB, op=pkg.UCCL_COPY), rt.fold(1024, 128 * KiB)
        assert rt.kernels() == ["chunk_flat_kernel"] * 3 + ["chunk_gather_kernel"]
    rt.answer["hipPointerGetAttributes"] = 0
    rt.launches.clear()
    rt.apply(8000, 32 * KiB), rt.fold(1024, 128 * KiB)
    assert rt.kernels() == ["chunk_order_kernel", "chunk_ordered_kernel", "gather_order_kernel", "gather_ordered_kernel"]
    asked = rt.calls.count("hipPointerGetAttributes")
    rt.apply(57, 64 * KiB), rt.apply(100), rt.fold(8, 128 * KiB)
    assert rt.calls.count("hipPointerGetAttributes") == asked       # small calls do not pay for the question


def test_records_outside_device_memory_are_read_once(tmp_path):
    in_process("records_in_host_memory", tmp_path)


def unknown_sizes(rt):
    for op in (0, pkg.UCCL_COPY):
        for n in (3072, 8191):
            rt.launches.clear()
            assert rt.apply(n, op=op) == 0
            assert [l[:3] for l in rt.launches] == [("chunk_order_kernel", -(-n // 256), 256), ("chunk_ordered_kernel", 4 * n, 256)]
        for n in (3071, 8192, 16383):      # from 8192 on: tiles of four records
            rt.launches.clear()
            assert rt.apply(n, op=op) == 0 and [l[:2] for l in rt.launches] == [("chunk_flat_kernel", n if n < 8192 else -(-n // 4))]


def test_calls_of_unknown_size_take_tiles_where_there_are_many_records(tmp_path):
    in_process("unknown_sizes", tmp_path)


def stated_sizes(rt):
    for chunk, parts in ((16 * KiB, 4), (20000, 5), (128 * KiB, 32), (256 * KiB, 32), (1 * MiB, 32), (2 ** 32 - 1, 32)):
        rt.launches.clear()
        assert rt.apply(7000, chunk) == 0 and rt.fold(7000, chunk) == 0
        assert [l[1] for l in rt.launches] == [28, 7000 * parts] * 2, chunk


def test_a_stated_size_far_above_the_records_does_not_multiply_workgroups_without_end(tmp_path):
    in_process("stated_sizes", tmp_path)


def test_calls_of_unknown_size_take_few_workgroups_and_do_not_depend_on_the_sequence_numbers(tmp_path):
    in_process("unknown_sizes", tmp_path)


def folds_of_one_part(rt):
    for capturing in (0, 1):
        rt.answer["hipStreamIsCapturing"] = capturing
        rt.launches.clear(), rt.calls.clear()
        assert rt.fold(1, 4096) == 0 and rt.fold(288, 64) == 0
        assert [l[:3] for l in rt.launches] == [("chunk_gather_parts_kernel", 1, 256), ("chunk_gather_parts_kernel", 288, 256)]
        assert not rt.calls                            # no region is asked for
    assert rt.fold(8, 4112) == 0 and rt.kernels()[-1] == "chunk_gather_kernel"    # two parts: no words under capture


def test_a_fold_whose_records_have_one_part_needs_no_claim_words(tmp_path):
    in_process("folds_of_one_part", tmp_path)


def hundreds_on_many_streams(rt):
    import threading
    for k in range(80):
        assert rt.apply(300, stream=0x1000 + 16 * k) == pkg.UCCL_OK
    assert rt.kernels() == ["chunk_group_kernel"] * 64 + ["chunk_few_kernel"] * 16
    for k in range(64):   # the streams of the large calls and the reports come later
        rt.launches.clear()
        assert rt.apply(8000, 32 * KiB, stream=0x9000 + 16 * k) == 0 and rt.report(1572200, stream=0x9000 + 16 * k) == 0
        assert rt.kernels() == ["chunk_order_kernel", "chunk_ordered_kernel", "ack_segments_kernel"], k
    rt.launches.clear()
    per_thread = 2
    for call, times in ((lambda: rt.fold(300, 0, per_thread), 20), (lambda: rt.apply(8000, 32 * KiB, per_thread), 16)):
        for _ in range(times):
            t = threading.Thread(target=call)
            t.start()
            t.join()
    assert rt.kernels() == ["gather_group_kernel"] * 16 + ["chunk_gather_kernel"] * 4 + ["chunk_order_kernel", "chunk_ordered_kernel"] * 16


def test_streams_with_calls_of_hundreds_leave_the_others_their_regions(tmp_path):
    in_process("hundreds_on_many_streams", tmp_path)


def forms_of_hundreds(rt):
    import threading
    lib, group, opts = rt.lib, lambda wgs, k="chunk": [(k + "_group_kernel", wgs, 256)], lambda c: C.byref(pkg.uccl_launch_opts(c, 0))
    extents = C.byref(pkg.uccl_extents(MiB, MiB, MiB, 3000))
    calls = [   # (call, its launches, and the kernel of the form it has without scratch words or for records in host memory)
        (lambda s=0: rt.apply(300, 4 * KiB, s), group(300), "chunk_flat_kernel"), (lambda s=0: rt.apply(300, 8 * KiB, s), group(300), "chunk_flat_kernel"),
        (lambda s=0: rt.apply(320, 16 * KiB, s), group(320), "chunk_few_kernel"), (lambda s=0: rt.apply(256, 32 * KiB, s), group(512), "chunk_few_kernel"),
        (lambda s=0: rt.apply(257, 64 * KiB, s, op=pkg.UCCL_COPY), group(4 * 257), "chunk_few_kernel"), (lambda s=0: rt.apply(192, stream=s), group(4 * 192), "chunk_few_kernel"),
        (lambda s=0: lib.uccl_chunk_apply_checked(A, OUT, RECV, DESCS, 700, BITS, 0, 0, extents, None, s), group(3 * 700), "chunk_few_kernel"),
        (lambda s=0: lib.uccl_chunk_apply_noalloc(A, OUT, RECV, DESCS, 2048, BITS, 0, 0, s), group(2 * 2048), "chunk_flat_kernel"),
        (lambda s=0: lib.uccl_chunk_scatter(A, RECV, DESCS, 500, BITS, s), group(4 * 500), "chunk_few_kernel"),
        (lambda s=0: lib.uccl_chunk_scatter_opts(A, RECV, DESCS, 500, BITS, None, None, opts(8 * KiB), s), group(500), "chunk_flat_kernel"),
        (lambda s=0: rt.fold(289, 4 * KiB, s), group(289, "gather"), "chunk_gather_kernel"), (lambda s=0: rt.fold(320, 8 * KiB, s), group(640, "gather"), "chunk_gather_kernel"),
        (lambda s=0: rt.fold(257, 0, s), group(6 * 257, "gather"), "chunk_gather_kernel")]
    tags, words = [], set()
    for call, launches, other in calls:
        rt.launches.clear()
        assert call() == 0 and [l[:3] for l in rt.launches] == launches, (launches, rt.launches)
        at, tag = rt.launches[0][5]
        tags.append(tag), words.add(at)
        for name, what in (("hipPointerGetAttributes", 1), ("hipPointerGetAttributes", -1), ("hipStreamIsCapturing", 1), ("hipStreamIsCapturing", -1)):
            rt.answer[name] = what
            rt.launches.clear()
            assert call() == 0 and rt.kernels() == [other], (launches, name, what, rt.kernels())
            del rt.answer[name]
    assert tags == sorted(set(tags)) and len(words) == 1             # one stream: the same words, another tag each time
    rt.launches.clear()                                              # a count that the host does not know, and stated parts
    assert lib.uccl_chunk_apply_indirect(A, OUT, RECV, DESCS, BITS, 300, BITS, 0, 0, None, None, None, None) == 0 and rt.apply(300, 0, parts=1) == 0
    assert rt.kernels() == ["chunk_few_kernel"] * 2
    per_thread, own = 2, []
    for stream in (0x1000, 0x2000, per_thread):
        rt.launches.clear()
        assert rt.apply(300, stream=stream) == 0 and rt.fold(300, 0, stream) == 0
        own.append({l[5][0] for l in rt.launches})
    assert all(len(x) == 1 for x in own) and len(set().union(words, *own)) == 4
    rt.launches.clear()
    threads = [threading.Thread(target=lambda: [rt.apply(300, stream=0x1000) for _ in range(200)]) for _ in range(4)]
    [t.start() for t in threads], [t.join() for t in threads]
    order = [l[5][1] for l in rt.launches]
    assert len(order) == 800 and order == sorted(set(order))         # tags grow in the order of the launches


def test_calls_of_hundreds_are_launched_in_their_form_and_in_the_other_without_scratch_words(tmp_path):
    in_process("forms_of_hundreds", tmp_path)


def unknown_sizes_of_hundreds(rt):
    for op in (0, pkg.UCCL_COPY):
        for n, parts in ((192, 4), (640, 4), (641, 3), (1500, 3), (1501, 2), (3000, 2)):
            rt.launches.clear()
            assert rt.apply(n, op=op) == 0 and [l[:3] for l in rt.launches] == [("chunk_group_kernel", parts * n, 256)], (n, op)
    for n, parts in ((257, 6), (800, 6), (801, 4), (3000, 4)):
        rt.launches.clear()
        assert rt.fold(n, 0) == 0 and [l[:3] for l in rt.launches] == [("gather_group_kernel", parts * n, 256)], n


def few_large_folds(rt):
    for n, chunk, parts in ((1, 48 * MiB, 4096), (1, 17 * MiB, 2176), (2, 20 * MiB, 2048), (16, 3 * MiB, 256), (60, 512 * KiB, 64), (129, 300 * KiB, 31), (128, 128 * KiB, None)):
        rt.launches.clear()
        assert rt.fold(n, chunk) == 0
        assert [l[:3] for l in rt.launches] == ([("gather_group_kernel", n * parts, 256)] if parts else [("chunk_gather_parts_kernel", 2048, 256)]), (n, chunk)


def test_few_large_folds_take_a_bounded_number_of_workgroups(tmp_path):
    """All of them wait for one line of scratch words, and the stated size may be far above the records'."""
    in_process("few_large_folds", tmp_path)


def test_a_long_record_of_unknown_size_has_several_workgroups(tmp_path):
    """A call of hundreds of records of different lengths does not wait for one small workgroup to walk each of the long ones."""
    in_process("unknown_sizes_of_hundreds", tmp_path)


if __name__ == "__main__":
    globals()[sys.argv[1]](Runtime(sys.argv[2]))
    print("SCENARIO DONE")
