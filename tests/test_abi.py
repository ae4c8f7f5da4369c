"""The C-ABI library: loads without a GPU, exports what the header declares, and its
host-side argument checks return the documented codes before anything is enqueued."""
import ctypes as C
import os
import re
import subprocess

import pytest

import paper_2504_17307_amd as pkg


def declared_functions():
    text = open(pkg.HEADER_PATH).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(uccl_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = pkg.load()
    names = declared_functions()
    assert {"uccl_chunk_apply", "uccl_chunk_scatter", "uccl_dedup_reset", "uccl_strerror",
            "uccl_version", "uccl_chunk_apply_checked", "uccl_chunk_apply_indirect", "uccl_chunk_scatter_checked",
            "uccl_chunk_apply_opts", "uccl_chunk_scatter_opts", "uccl_init", "uccl_dedup_report",
            "uccl_time_next_launch", "uccl_last_error_detail"} <= set(names)
    assert not [n for n in names if n.startswith("uccl_set_")], "no process-wide tuning knob in the ABI"
    for n in names:
        assert hasattr(lib, n), n
    assert set(names) == set(pkg._SIGNATURES), "binding and header list the same entry points"
    assert lib.uccl_version() == 2


def test_record_layout_matches_generators():
    from synth.layout import DESC, NO_FORWARD
    assert DESC.itemsize == pkg.DESC_BYTES == 32
    assert [DESC.fields[n][1] for n in ("src_off", "dst_off", "out_off", "len", "seq")] == [0, 8, 16, 24, 28]
    assert int(NO_FORWARD) == pkg.UCCL_NO_FORWARD
    text = open(pkg.HEADER_PATH).read()
    order = [text.index(f" {n};") for n in ("src_off", "dst_off", "out_off", "len", "seq")]
    assert order == sorted(order)


def test_host_side_error_codes_enqueue_nothing():
    lib = pkg.load()
    A, B, D, M = 0x10000, 0x20000, 0x30000, 0x40000  # never dereferenced: every call fails on the host
    f = lib.uccl_chunk_apply
    assert f(None, None, B, D, 1, M, 0, 0, None) == pkg.UCCL_EINVAL
    assert f(A, None, None, D, 1, M, 0, 0, None) == pkg.UCCL_EINVAL
    assert f(A, None, B, None, 1, M, 0, 0, None) == pkg.UCCL_EINVAL
    assert f(A, None, B, D, 1, None, 0, 0, None) == pkg.UCCL_EINVAL
    assert f(A, None, B, D, 1, M, 4, 0, None) == pkg.UCCL_EINVAL   # dtype
    assert f(A, None, B, D, 1, M, -1, 0, None) == pkg.UCCL_EINVAL
    assert f(A, None, B, D, 1, M, 0, 5, None) == pkg.UCCL_EINVAL   # op
    assert f(A, None, B, D, 1, M, 0, -1, None) == pkg.UCCL_EINVAL
    assert f(A + 8, None, B, D, 1, M, 0, 0, None) == pkg.UCCL_EALIGN
    assert f(A, A + 4, B, D, 1, M, 0, 0, None) == pkg.UCCL_EALIGN
    assert f(A, None, B + 2, D, 1, M, 0, 0, None) == pkg.UCCL_EALIGN
    assert f(A, None, B, D + 8, 1, M, 0, 0, None) == pkg.UCCL_EALIGN
    assert f(A, None, B, D, 1, M + 2, 0, 0, None) == pkg.UCCL_EALIGN
    assert f(None, None, None, None, 0, None, 0, 0, None) == pkg.UCCL_OK  # empty call is a no-op
    g = lib.uccl_chunk_apply_checked
    assert g(A, None, B, D, 1, M, 0, 0, None, None, None) == pkg.UCCL_EINVAL  # extents required
    e = pkg.uccl_extents(0x20000, 0, 0x1000, 8)  # acc extent runs into recv_stage
    assert g(A, None, B, D, 1, M, 0, 0, C.byref(e), None, None) == pkg.UCCL_EINVAL
    e = pkg.uccl_extents(0x1000, 0, 0x1000, 8)
    assert g(A, None, B, D, 1, M, 0, 0, C.byref(e), 0x50002, None) == pkg.UCCL_EALIGN
    i = lib.uccl_chunk_apply_indirect
    assert i(A, None, B, D, None, 4, M, 0, 0, None, None, None, None) == pkg.UCCL_EINVAL   # count pointer required
    assert i(A, None, B, D, 0x60002, 4, M, 0, 0, None, None, None, None) == pkg.UCCL_EALIGN
    assert i(None, None, None, None, None, 0, None, 0, 0, None, None, None, None) == pkg.UCCL_OK
    o = lib.uccl_chunk_apply_opts
    assert o(None, None, None, None, 0, None, 0, 0, None, None, None, None) == pkg.UCCL_OK
    assert o(A, None, B, D, 1, M, 0, 0, None, None, C.byref(pkg.uccl_launch_opts(4096, 17)), None) == pkg.UCCL_EINVAL
    bad = pkg.uccl_launch_opts(4096, 2)
    bad.reserved[1] = 1
    assert o(A, None, B, D, 1, M, 0, 0, None, None, C.byref(bad), None) == pkg.UCCL_EINVAL
    assert o(A + 8, None, B, D, 1, M, 0, 0, None, None, C.byref(pkg.uccl_launch_opts(4096, 2)), None) == pkg.UCCL_EALIGN
    assert lib.uccl_chunk_scatter_opts(A, B, D, 1, M, None, None, C.byref(pkg.uccl_launch_opts(0, 99)), None) == pkg.UCCL_EINVAL
    assert lib.uccl_chunk_reduce_gather(A, None, B, D, 1, M, 0, 0, None, None, C.byref(pkg.uccl_launch_opts(0, 99)), None) == pkg.UCCL_EINVAL
    assert lib.uccl_claim_timeouts(None) == pkg.UCCL_EINVAL
    sg = lib.uccl_chunk_segment
    assert sg(A, B, 0, 4096, 0, 0, 64, None, 0, 0, 0, None) == pkg.UCCL_EINVAL        # chunk size 0
    assert sg(A, B, 0, 4096, 24, 0, 64, None, 0, 0, 0, None) == pkg.UCCL_EALIGN
    assert sg(A, B, 8, 4096, 64, 0, 64, None, 0, 0, 0, None) == pkg.UCCL_EALIGN
    assert sg(A, B, 0, 4096, 64, 4, 64, None, 0, 0, 0, None) == pkg.UCCL_EALIGN
    assert sg(A, B, 0, 4096, 64, 0, 32, None, 0, 0, 0, None) == pkg.UCCL_EINVAL        # slots would overlap
    assert sg(A, B, 0, 4096, 64, 0, 64, None, 256, 0, 0, None) == pkg.UCCL_EINVAL      # connection id is 8 bits
    assert sg(A, B, 0, 4096, 64, 0, 64, None, 0, 128, 0, None) == pkg.UCCL_EINVAL      # message id is 7 bits
    assert sg(None, None, 0, 0, 64, 0, 64, None, 0, 0, 0, None) == pkg.UCCL_OK         # nothing to cut
    assert sg(None, B, 0, 64, 64, 0, 64, None, 0, 0, 0, None) == pkg.UCCL_EINVAL
    assert sg(A, B, 0, 64, 64, 0, 64, 0x70004, 0, 0, 0, None) == pkg.UCCL_EALIGN
    na = lib.uccl_chunk_apply_noalloc
    assert na(A, None, B, D, pkg.UCCL_NOALLOC_MAX_DESCS + 1, M, 0, 0, None) == pkg.UCCL_ETOOBIG   # before any GPU call
    assert na(A, None, B, D, 1, M, 7, 0, None) == pkg.UCCL_EINVAL
    assert na(None, None, None, None, 0, None, 0, 0, None) == pkg.UCCL_OK
    assert "UCCL_NOALLOC_MAX_DESCS %d" % pkg.UCCL_NOALLOC_MAX_DESCS in open(pkg.HEADER_PATH).read()
    s = lib.uccl_chunk_scatter
    assert s(None, B, D, 1, M, None) == pkg.UCCL_EINVAL
    assert s(A + 1, B, D, 1, M, None) == pkg.UCCL_EALIGN
    assert s(None, None, None, 0, None, None) == pkg.UCCL_OK
    assert lib.uccl_chunk_scatter_checked(A, B, D, 1, M, None, None, None) == pkg.UCCL_EINVAL
    r = lib.uccl_dedup_reset
    assert r(None, 8, None) == pkg.UCCL_EINVAL and r(M + 1, 8, None) == pkg.UCCL_EALIGN
    assert r(None, 0, None) == pkg.UCCL_OK
    q = lib.uccl_dedup_report
    assert q(M, 64, None, 4, None) == pkg.UCCL_EINVAL and q(None, 64, A, 4, None) == pkg.UCCL_EINVAL
    assert q(M + 2, 64, A, 4, None) == pkg.UCCL_EALIGN and q(M, 64, A + 4, 4, None) == pkg.UCCL_EALIGN
    assert q(M, 1 << 40, A, 4, None) == pkg.UCCL_EINVAL
    ms = lib.uccl_message_status
    assert ms(M, M, 4, 0, A, 0, None) == pkg.UCCL_EINVAL and ms(M, M, 4, 48, A, 0, None) == pkg.UCCL_EINVAL
    assert ms(M, M, 4, 4096, A, 0, None) == pkg.UCCL_EINVAL and ms(None, M, 4, 256, A, 0, None) == pkg.UCCL_EINVAL
    assert ms(M, None, 4, 256, A, 0, None) == pkg.UCCL_EINVAL and ms(M, M, 4, 256, None, 0, None) == pkg.UCCL_EINVAL
    assert ms(M + 2, M, 4, 256, A, 0, None) == pkg.UCCL_EALIGN and ms(M, M, 4, 256, A + 8, 0, None) == pkg.UCCL_EALIGN
    assert ms(None, None, 0, 256, None, 0, None) == pkg.UCCL_OK
    assert ms(M, M, (1 << 24) + 1, 256, A, 0, None) == pkg.UCCL_EINVAL
    h = C.c_void_p()
    fc = lib.uccl_feed_create
    assert fc(None, A, None, B, M, 0, 0, 3, 64, 4, None) == pkg.UCCL_EINVAL
    assert fc(C.byref(h), None, None, B, M, 0, 0, 3, 64, 4, None) == pkg.UCCL_EINVAL
    assert fc(C.byref(h), A, None, B, M, 0, 0, 3, 0, 4, None) == pkg.UCCL_EINVAL     # capacity
    assert fc(C.byref(h), A, None, B, M, 0, 0, 3, 64, 1, None) == pkg.UCCL_EINVAL     # slots
    assert fc(C.byref(h), A, None, B, M, 0, 9, 3, 64, 4, None) == pkg.UCCL_EINVAL     # op
    assert fc(C.byref(h), A + 4, None, B, M, 0, 0, 3, 64, 4, None) == pkg.UCCL_EALIGN
    assert h.value is None
    for fn in (lib.uccl_feed_poll, lib.uccl_feed_flush, lib.uccl_feed_sync, lib.uccl_feed_destroy):
        assert fn(None) == pkg.UCCL_EINVAL
    assert lib.uccl_feed_push(None, 0, D, 1) == pkg.UCCL_EINVAL
    assert pkg.uccl_strerror(pkg.UCCL_EALIGN) == "misaligned pointer"
    with pytest.raises(pkg.UcclError) as err:
        pkg.uccl_chunk_apply(None, None, B, D, 1, M, 0, 0, stream=0)
    assert err.value.code == pkg.UCCL_EINVAL


def test_no_cpu_fallback_when_library_missing():
    with pytest.raises(RuntimeError):
        pkg.load(os.path.join(os.path.dirname(pkg.LIB_PATH), "no_such_library.so"))


def test_product_never_touches_the_oracle():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    for d, _, files in os.walk(os.path.join(root, "paper_2504_17307_amd")):
        for fn in files:
            if fn.endswith((".py", ".hip", ".h", ".cpp")):
                src = open(os.path.join(d, fn)).read()
                assert "oracle" not in src.replace("no CPU fallback", ""), fn
    for fn in os.listdir(os.path.join(root, "oracle")):
        if fn.endswith((".py", ".c", ".h")):
            src = open(os.path.join(root, "oracle", fn)).read()
            assert "paper_2504_17307_amd" not in src and "uccl_chunk.h" not in src, fn


def test_prepare_marshals_once_and_repeats_the_c_call():
    """Host logic of pkg.uccl_prepare on calls that return before anything is enqueued."""
    A, B, D, M = 0x10000, 0x20000, 0x30000, 0x40000
    empty = pkg.uccl_prepare(pkg.uccl_chunk_apply, A, None, B, D, 0, M, 0, 0, stream=0)   # no records: a no-op
    empty()
    empty()
    bad = pkg.uccl_prepare(pkg.uccl_chunk_apply_opts, A + 8, None, B, D, 1, M, 0, 0, opts=(4096, 0), stream=0)
    for _ in range(2):                       # the prepared call fails the same way every time it is made
        with pytest.raises(pkg.UcclError) as e:
            bad()
        assert e.value.code == pkg.UCCL_EALIGN
    with pytest.raises(ValueError):          # a function that makes no C call cannot be prepared
        pkg.uccl_prepare(lambda: None)
    with pytest.raises(ValueError):          # nor one whose own marshalling fails; and neither leaves the
        pkg.uccl_prepare(pkg.uccl_chunk_apply_checked, A, None, B, D, 1, M, 0, 0, stream=0)   # binding capturing
    with pytest.raises(pkg.UcclError):       # an ordinary call is made, not captured
        pkg.uccl_chunk_apply(A + 8, None, B, D, 1, M, 0, 0, stream=0)


def test_prepared_calls_pass_every_argument():
    """One to thirteen whole numbers and pointers arrive as they were given, call after call, from several threads; the objects
    that the arguments point into are kept; no arguments are taken."""
    import ctypes as C
    import gc
    import threading
    import weakref
    from paper_2504_17307_amd import _prepared
    for n in range(14):
        got = []
        kind = C.CFUNCTYPE(C.c_int, *[(C.c_uint64, C.c_uint32, C.c_int, C.c_void_p)[i % 4] for i in range(n)])
        f = kind(lambda *a: got.append(a) or 0)
        values = [((1 << 63) + 12345, (1 << 32) - 7, -5, 0x7FFF12345678)[i % 4] + (i // 4) for i in range(n)]
        call = _prepared.Prepared(C.cast(f, C.c_void_p).value, tuple(values), print, None)
        threads = [threading.Thread(target=lambda: [call() for _ in range(50)]) for _ in range(3)]
        [t.start() for t in threads], [t.join() for t in threads]
        assert got == [tuple(values)] * 150, n
    codes = []
    fails = C.CFUNCTYPE(C.c_int)(lambda: -3)
    assert _prepared.Prepared(C.cast(fails, C.c_void_p).value, (), codes.append, None)() is None and codes == [-3]
    with pytest.raises(TypeError):
        call(1)
    with pytest.raises(ValueError):
        _prepared.Prepared(1, (0,) * 14, print, None)

    class Kept:
        pass
    k = Kept()
    call = _prepared.Prepared(C.cast(fails, C.c_void_p).value, (), codes.append, (k,))
    k.cycle, gone = call, weakref.ref(k)
    del k
    gc.collect()
    assert gone() is not None and call.keeps[0] is gone()
    del call
    gc.collect()
    assert gone() is None


def test_a_prepared_call_is_an_object_like_others():
    """It takes attributes and weak references, says which call it makes, and keeps what it was given; none of that leaks."""
    import gc
    import weakref

    class Kept(int):
        pass
    acc = Kept(0x10000)
    call = pkg.uccl_prepare(pkg.uccl_chunk_apply, acc, None, 0x20000, 0x30000, 0, 0x40000, 0, 0, stream=0)
    assert call.__name__ == "uccl_chunk_apply"
    args, kwargs = call.keeps
    assert args[0] is acc and kwargs == {"stream": 0}
    call.label, acc.cycle = ["of", "the", "caller"], call
    assert call.label[0] == "of" and vars(call) == {"label": call.label}
    gone = weakref.ref(call)
    assert gone() is call
    call()
    del call, acc, args, kwargs
    gc.collect()
    assert gone() is None


def test_the_extension_is_of_this_interpreter_and_of_the_present_source(monkeypatch, tmp_path):
    """It calls raw addresses and reads object layouts: what another interpreter or an older source built is not loaded."""
    import sysconfig
    from paper_2504_17307_amd import build
    assert build.PREPARED_LIB.endswith("_prepared" + sysconfig.get_config_var("EXT_SUFFIX"))
    monkeypatch.setattr(pkg, "_extension", None)
    assert pkg._load_extension().__file__ == build.PREPARED_LIB
    newer = tmp_path / "prepared_call.c"
    newer.write_text("")
    os.utime(newer, (os.path.getmtime(build.PREPARED_LIB) + 60,) * 2)
    monkeypatch.setattr(build, "PREPARED_SRC", str(newer))
    monkeypatch.setattr(pkg, "_extension", None)
    with pytest.raises(RuntimeError, match="older than its source"):
        pkg.uccl_prepare(pkg.uccl_chunk_apply, 0x10000, None, 0x20000, 0x30000, 0, 0x40000, 0, 0, stream=0)


@pytest.mark.parametrize("failure", [FileNotFoundError("gcc"), subprocess.CalledProcessError(1, "gcc")])
def test_calls_can_be_prepared_where_the_extension_cannot_be_built(monkeypatch, tmp_path, failure):
    """No compiler, no headers of the interpreter, another calling convention: the same calls, by ctypes."""
    from paper_2504_17307_amd import build

    def fails(verbose=False):
        raise failure
    monkeypatch.setattr(build, "PREPARED_LIB", str(tmp_path / "none.so"))
    monkeypatch.setattr(build, "build_prepared", fails)
    monkeypatch.setattr(pkg, "_extension", None)
    for _ in range(2):
        call = pkg.uccl_prepare(pkg.uccl_chunk_apply_opts, 0x10008, None, 0x20000, 0x30000, 1, 0x40000, 0, 0, opts=(4096, 0), stream=0)
        with pytest.raises(pkg.UcclError) as e:
            call()
        assert e.value.code == pkg.UCCL_EALIGN
    assert pkg.uccl_prepare(pkg.uccl_chunk_apply, 0x10000, None, 0x20000, 0x30000, 0, 0x40000, 0, 0, stream=0)() is None


def test_launch_plan_rules():
    """Host logic: which launch a call gets (uccl_launch_plan is the rule the data-path calls apply)."""
    plan = pkg.uccl_launch_plan
    KiB = 1024
    # the routing table of the design, one row each
    assert plan(7856, (32 * KiB, 0)) == dict(kernel="chunk_flat_kernel", records_per_group=1, parts=1, threads=1024,
                                             groups=7856, unit_bytes=1024)
    assert plan(7856, (32 * KiB, 0), reads_acc=False)["unit_bytes"] == 2048          # copies keep 2 KiB units
    assert plan(2047, (32 * KiB, 0))["kernel"] == "chunk_few_kernel" and plan(2048, (32 * KiB, 0))["kernel"] == "chunk_flat_kernel"
    assert plan(57, (64 * KiB, 0)) == dict(kernel="chunk_few_kernel", records_per_group=1, parts=8, threads=256,
                                           groups=456, unit_bytes=2048)
    assert plan(8, (128 * KiB, 0))["parts"] == 16 and plan(256, (128 * KiB, 0))["parts"] == 1   # 32 MiB: not cut
    assert plan(32, (32 * KiB, 0))["parts"] == 8 and plan(33, (32 * KiB, 0))["parts"] == 1
    assert plan(3620, (16 * KiB, 0)) == dict(kernel="chunk_few_kernel", records_per_group=1, parts=1, threads=1024,
                                             groups=3620, unit_bytes=1024)
    assert plan(8192, (16 * KiB, 0)) == dict(kernel="chunk_flat_kernel", records_per_group=2, parts=1, threads=1024,
                                             groups=4096, unit_bytes=2048)
    assert plan(128, (4 * KiB, 0))["threads"] == 256 and plan(128, (4 * KiB, 0))["unit_bytes"] == 1024
    assert plan(128, (8 * KiB, 0))["unit_bytes"] == 2048
    assert plan(129, (4 * KiB, 0)) == dict(kernel="chunk_flat_kernel", records_per_group=8, parts=1, threads=1024,
                                           groups=17, unit_bytes=2048)
    assert plan(1000, (1 * KiB, 0))["records_per_group"] == 32 and plan(1000, (64, 0))["records_per_group"] == 32
    # no chunk size given: by record count alone
    assert [plan(n)["parts"] for n in (1, 64, 65, 128, 129)] == [8, 8, 4, 4, 1]
    assert [plan(n)["records_per_group"] for n in (8191, 8192, 32768, 131072)] == [1, 4, 8, 16]
    # a stated number of parts is honoured where a workgroup takes one record and the call has at most 2048
    assert plan(57, (64 * KiB, 5))["parts"] == 5 and plan(2048, (64 * KiB, 2))["groups"] == 4096
    assert plan(2049, (64 * KiB, 2))["parts"] == 1 and plan(57, (4 * KiB, 5))["parts"] == 1
    assert plan(0, (32 * KiB, 0))["groups"] == 0
    # the multi-source fold
    assert plan(8, (128 * KiB, 0), gather=True) == dict(kernel="chunk_gather_parts_kernel", records_per_group=1, parts=16,
                                                        threads=256, groups=128, unit_bytes=2048)
    assert plan(128, (32 * KiB, 0), gather=True)["parts"] == 4 and plan(1024, (128 * KiB, 0), gather=True)["parts"] == 1
    assert plan(5000, (4 * KiB, 0), gather=True)["records_per_group"] == 8
    # invariants over a sweep: a cut launch stays within 2048 workgroups of at most 16 per record;
    # the grid covers every record
    for c in (0, 64, 4 * KiB, 8 * KiB, 12 * KiB, 16 * KiB, 24 * KiB, 32 * KiB, 48 * KiB, 64 * KiB, 128 * KiB, 1 << 20):
        for n in (1, 2, 31, 32, 33, 64, 127, 128, 129, 512, 2047, 2048, 2049, 8191, 8192, 100000, 2 ** 32 - 1):
            for g in (False, True):
                p = plan(n, (c, 0), gather=g)
                assert 1 <= p["parts"] <= 16 and 1 <= p["records_per_group"] <= 32
                assert p["parts"] == 1 or (p["records_per_group"] == 1 and n * p["parts"] <= 2048)
                assert p["groups"] * p["records_per_group"] >= n * p["parts"] and p["groups"] <= n * p["parts"]
                assert p["threads"] in (256, 1024) and p["unit_bytes"] in (1024, 2048, 4096)
    # what the data-path calls refuse, the plan refuses
    lib = pkg.load()
    out = pkg.uccl_plan()
    bad = pkg.uccl_launch_opts(4096, 17)
    assert lib.uccl_launch_plan(10, C.byref(bad), 0, 1, C.byref(out)) == pkg.UCCL_EINVAL
    assert lib.uccl_launch_plan(10, None, 0, 1, None) == pkg.UCCL_EINVAL
