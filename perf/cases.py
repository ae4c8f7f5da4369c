"""What this library is used for, as cases that can be timed and compared.

Every case is one rank's share of a collective, as its control path hands it to the GPU: receive slots in
arrival order (out of order within a window, some chunks twice), one record per arrival, and the calls that a
program makes for it.  The kinds:

  ring      ring allreduce (reduce phase, then copy phase) or ring reduce-scatter of one message
  batch     many small ring allreduces, all messages' records of a phase in one call
  alltoall  all-to-all dispatch: scatter-copy to per-source offsets
  direct    one-hop reduce-scatter: every destination chunk folds one chunk from each peer
  segment   sender side: a tensor range cut into staged chunks with send records
  feedback  receiver feedback: selective acknowledgement of a bitmap, status of a message window

Sums and selections of this library are defined to the bit (one operation in binary32 and one rounding, a fold
in the order the record lists), so every output is compared exactly.
"""
import math

import numpy as np
import torch

import paper_2504_17307_amd as uccl

DTYPES = {"f32": (torch.float32, uccl.UCCL_F32, 4), "bf16": (torch.bfloat16, uccl.UCCL_BF16, 2),
          "f16": (torch.float16, uccl.UCCL_F16, 2), "i32": (torch.int32, uccl.UCCL_I32, 4)}
OPS = {"sum": uccl.UCCL_SUM, "max": uccl.UCCL_MAX, "min": uccl.UCCL_MIN}
DESC = np.dtype([("src_off", "<u8"), ("dst_off", "<u8"), ("out_off", "<u8"), ("len", "<u4"), ("seq", "<u4")])
GATHER_DESC = np.dtype([("dst_off", "<u8"), ("out_off", "<u8"), ("len", "<u4"), ("seq", "<u4"), ("n_src", "<u4"),
                        ("reserved", "<u4"), ("src_off", "<u8", (uccl.UCCL_MAX_SOURCES,))])
NO_FORWARD = np.uint64(uccl.UCCL_NO_FORWARD)
FORWARD_ONLY = np.uint64(1 << 63)
NOALLOC_RECORDS = 1500  # a case of the no-allocation entry point stays below its limit, duplicates included


def listed():
    return [
        # the smallest message of the small-message regime, alone: three calls, all latency
        {"name": "ring-64K-f32", "kind": "ring", "bytes": 64 << 10, "ranks": 8, "chunk": 4096, "dtype": "f32", "op": "sum",
         "window": 0, "dup": 0.03, "gather_phase": True, "relay": False, "entry": "opts"},
        # a small message in the transport's default chunks, from a caller that may not allocate
        {"name": "ring-1M-f32-noalloc", "kind": "ring", "bytes": 1 << 20, "ranks": 8, "chunk": 32768, "dtype": "f32", "op": "sum",
         "window": 0, "dup": 0.01, "gather_phase": True, "relay": False, "entry": "noalloc"},
        # benchmark configuration: 4 MiB message, 64 KiB chunks
        {"name": "ring-4M-f32", "kind": "ring", "bytes": 4 << 20, "ranks": 8, "chunk": 65536, "dtype": "f32", "op": "sum",
         "window": 0, "dup": 0.01, "gather_phase": True, "relay": False, "entry": "opts"},
        # benchmark configuration: the 128 messages that one connection may have in flight, in one call per phase
        {"name": "batch-128-f32", "kind": "batch", "messages": 128, "sizes": 5, "ranks": 8, "chunk": 4096, "dtype": "f32",
         "dup": 0.03, "entry": "opts"},
        # an odd-sized tensor in the payloads of 9 KB datagrams, through the plain entry point (no chunk size given)
        {"name": "ring-64M-f16-packets", "kind": "ring", "bytes": (64 << 20) + 54, "ranks": 16, "chunk": 8944, "dtype": "f16",
         "op": "sum", "window": 1024, "dup": 0.02, "gather_phase": True, "relay": False, "entry": "plain"},
        # the headline benchmark configuration: gradient bucket in bf16, default chunks
        {"name": "ring-256M-bf16", "kind": "ring", "bytes": 256 << 20, "ranks": 16, "chunk": 32768, "dtype": "bf16", "op": "sum",
         "window": 1024, "dup": 0.02, "gather_phase": True, "relay": False, "entry": "opts"},
        # benchmark configuration, the largest call: 1 GiB reduce-scatter in transport-buffer-sized chunks
        {"name": "ring-rs-1G-f32", "kind": "ring", "bytes": 1 << 30, "ranks": 8, "chunk": 131072, "dtype": "f32", "op": "sum",
         "window": 256, "dup": 0.005, "gather_phase": False, "relay": False, "entry": "opts"},
        # benchmark configuration: mixture-of-experts dispatch, rows of 7168 bf16 elements from seven peers
        {"name": "alltoall-bf16", "kind": "alltoall", "sources": 7, "row": 14336, "most": 16 << 20, "sizes": 29, "chunk": 16384,
         "dup": 0.01, "entry": "opts"},
        # benchmark configuration: one-hop reduce-scatter of 1 GiB, seven peers' copies of a 128 MiB segment
        {"name": "direct-128M-f32", "kind": "direct", "bytes": 128 << 20, "sources": 7, "chunk": 131072, "dtype": "f32", "op": "sum",
         "dup": 0.005, "entry": "opts"},
        # the same step of a small bf16 message in the smallest chunks that reach line rate
        {"name": "direct-1M-bf16", "kind": "direct", "bytes": 1 << 20, "sources": 7, "chunk": 16384, "dtype": "bf16", "op": "sum",
         "dup": 0.01, "entry": "opts"},
        # benchmark configuration: the first hop of the headline ring, this rank's own segment
        {"name": "segment-16M", "kind": "segment", "bytes": 16 << 20, "chunk": 32768},
        # benchmark configuration: feedback for a long run of small chunks with holes, and for a full message window
        {"name": "feedback-1.5M-bits", "kind": "feedback", "bits": 1572200, "holes": 97, "ranges": 4096, "slots": 128},
    ]


def _log(rng, lo, hi):
    return lo * (hi / lo) ** rng.random()


def _chunk(rng, lo, hi):
    """A chunk size: a power of two or, as often, a payload size that is none (a multiple of 16: slots are 16-byte aligned)."""
    c = _log(rng, lo, hi)
    return 1 << round(math.log2(c)) if rng.random() < 0.5 else int(c) // 16 * 16


def draw(rng):
    kind = rng.choice(["ring"] * 6 + ["batch", "alltoall", "alltoall", "direct", "direct", "direct", "segment", "feedback"])
    if kind == "ring":
        ranks = rng.choice([2, 4, 8, 8, 16, 16])
        dtype = rng.choice(["f32", "bf16", "bf16", "f16", "i32"])
        size = int(_log(rng, 64 << 10, 256 << 20)) // 4 * 4
        chunk = _chunk(rng, max(4096, size // 100000), 131072)
        gather_phase = rng.random() < 0.75
        case = {"kind": kind, "bytes": size, "ranks": ranks, "chunk": chunk, "dtype": dtype, "op": rng.choice(["sum", "sum", "sum", "max", "min"]),
                "window": rng.choice([0, 256, 1024]) if size // chunk < 4096 else rng.choice([256, 1024]), "dup": rng.choice([0.0, 0.005, 0.02, 0.03]),
                "gather_phase": gather_phase, "relay": rng.random() < 0.15, "entry": rng.choice(["opts", "opts", "plain", "checked", "noalloc"])}
        if case["entry"] == "noalloc" and -(-size // ranks // chunk) * (ranks - 1) > NOALLOC_RECORDS:
            case["entry"] = "plain"
        return case
    if kind == "batch":
        return {"kind": kind, "messages": int(_log(rng, 2, 256)), "sizes": rng.randrange(1 << 20), "ranks": rng.choice([4, 8, 16]), "chunk": _chunk(rng, 4096, 16384),
                "dtype": rng.choice(["f32", "bf16"]), "dup": rng.choice([0.0, 0.03]), "entry": rng.choice(["opts", "plain"])}
    if kind == "alltoall":
        return {"kind": kind, "sources": rng.choice([3, 7, 15]), "row": rng.choice([4096, 8192, 14336]), "most": int(_log(rng, 64 << 10, 32 << 20)),
                "sizes": rng.randrange(1 << 20), "chunk": _chunk(rng, 4096, 65536), "dup": rng.choice([0.0, 0.01]), "entry": rng.choice(["opts", "opts", "plain", "checked"])}
    if kind == "direct":
        return {"kind": kind, "bytes": int(_log(rng, 16 << 10, 64 << 20)) // 4 * 4, "sources": rng.choice([1, 2, 3, 7, 15, 16]), "chunk": _chunk(rng, 4096, 131072),
                "dtype": rng.choice(["f32", "bf16", "f16", "i32"]), "op": rng.choice(["sum", "sum", "max"]), "dup": rng.choice([0.0, 0.01]),
                "entry": rng.choice(["opts", "opts", "plain"])}
    if kind == "segment":
        return {"kind": kind, "bytes": int(_log(rng, 64 << 10, 256 << 20)), "chunk": _chunk(rng, 4096, 131072)}
    return {"kind": kind, "bits": int(_log(rng, 4096, 2 << 20)), "holes": rng.choice([3, 31, 97, 1000, 0]), "ranges": rng.choice([64, 512, 4096]), "slots": rng.choice([1, 16, 128])}


# ---- inputs ------------------------------------------------------------------------------------

def _values(seed, stream, n, dtype):
    """What a tensor buffer or a payload holds: gradients in the floating types, small counts in the whole ones."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 64 + stream)
    if dtype == "i32":
        return torch.randint(-(1 << 20), 1 << 20, (n,), generator=g, device="cuda", dtype=torch.int32)
    if dtype == "f32":
        return torch.rand(n, generator=g, device="cuda") * 2 - 1
    return torch.randn(n, generator=g, device="cuda", dtype=torch.bfloat16 if dtype == "bf16" else torch.float16)


def _arrivals(g, n, window, dup):
    """Arrival order of chunks 0..n-1 sprayed over paths: a chunk is late by up to `window` chunks (0: by any number), a
    retransmitted one comes a second time, later."""
    w = float(window or n)
    at = np.arange(n) + g.random(n) * w
    twice = np.flatnonzero(g.random(n) < dup)
    when = np.concatenate([at, at[twice] + 1 + g.random(len(twice)) * w])
    order = np.argsort(when, kind="stable")
    return np.concatenate([np.arange(n), twice])[order], when[order]


def _on_gpu(records):
    return torch.from_numpy(np.ascontiguousarray(records).view(np.uint8).reshape(-1)).cuda()


def _bitmap(n_bits):
    return torch.zeros((n_bits + 31) // 32, dtype=torch.int32, device="cuda")


def _ring_plan(case, elements):
    """The chunks one rank (rank 0) receives: per phase (lists by step of segment and whether it forwards / only forwards)."""
    r, es = case["ranks"], DTYPES[case["dtype"]][2]
    seg = -(-elements // r)                          # elements of a segment
    pitch = -(-seg * es // 16) * 16 // es            # and where the next one starts: on 16 bytes
    per = case["chunk"] // es
    cps = -(-seg // per)
    again = case.get("gather_phase", True)
    reduce_ = [((-s - 1) % r, s < r - 2 or again, case.get("relay", False) and s < r - 2) for s in range(r - 1)]
    copy = [((-s) % r, s < r - 2, False) for s in range(r - 1)] if again else []
    return seg, pitch, per, cps, reduce_, copy


def _ring_records(case, elements, dst_base, out_base, seq_base):
    """Records of one message in sender order without source offsets, a list per phase, and its number of staging slots."""
    es = DTYPES[case["dtype"]][2]
    seg, pitch, per, cps, reduce_, copy = _ring_plan(case, elements)
    chunk, slots, seq, phases = case["chunk"], 0, seq_base, []
    c = np.arange(cps, dtype=np.uint64)
    for steps in (reduce_, copy):
        d = np.zeros((len(steps), cps), dtype=DESC)
        for s, (segment, forward, only) in enumerate(steps):
            d[s]["dst_off"] = np.uint64(dst_base + segment * pitch * es) + c * np.uint64(chunk)
            d[s]["len"] = np.minimum(per, seg - c.astype(np.int64) * per) * es
            d[s]["seq"] = seq + c
            seq += cps
            d[s]["out_off"] = NO_FORWARD
            if forward:
                d[s]["out_off"] = np.uint64(out_base + slots * chunk) + c * np.uint64(chunk)
                slots += cps
                if only:
                    d[s]["out_off"] |= FORWARD_ONLY
        phases.append(d.reshape(-1))
    return phases, slots, seq


def _fill(sender_order, arrivals, slot0, chunk):
    d = sender_order[arrivals]
    d["src_off"] = (slot0 + np.arange(len(d), dtype=np.uint64)) * np.uint64(chunk)
    return d


def _apply(case, acc, out, recv, d, n, bitmap, op, n_bits, rejected):
    code = DTYPES[case["dtype"]][1]
    if case["entry"] == "opts":
        return uccl.uccl_prepare(uccl.uccl_chunk_apply_opts, acc, out, recv, d, n, bitmap, code, op, opts=(case["chunk"], 0))
    if case["entry"] == "checked":
        return uccl.uccl_prepare(uccl.uccl_chunk_apply_checked, acc, out, recv, d, n, bitmap, code, op, n_bits=n_bits, n_rejected=rejected)
    f = uccl.uccl_chunk_apply_noalloc if case["entry"] == "noalloc" else uccl.uccl_chunk_apply
    return uccl.uccl_prepare(f, acc, out, recv, d, n, bitmap, code, op)


def _message_elements(case):
    """Sizes of a batch's messages, in elements: log-uniform from 64 KiB to 1 MiB, part of the case and not of the seed."""
    u = np.random.default_rng(case["sizes"]).random(case["messages"])
    es = DTYPES[case["dtype"]][2]
    return [int(b) // 4 * 4 // es for b in (64 << 10) * 16.0 ** u]


def _ring_inputs(case, seed):
    """Accumulator, payloads in sender order (a matrix of chunks per phase) and records of a ring or batch case."""
    g = np.random.default_rng(seed)
    es = DTYPES[case["dtype"]][2]
    many = [case["bytes"] // es] if case["kind"] == "ring" else _message_elements(case)
    dst = out = seq = 0
    sender, arrive, when = ([], []), ([], []), ([], [])
    for k, elements in enumerate(many):
        phases, slots, seq_end = _ring_records(case, elements, dst, out, seq)
        for p, d in enumerate(phases):
            a, at = _arrivals(g, len(d), case.get("window", 0), case["dup"])
            arrive[p].append(a + sum(len(x) for x in sender[p]))
            when[p].append(at / max(1, len(d)))  # the messages of a batch are in flight together
            sender[p].append(d)
        _, pitch, _, _, _, _ = _ring_plan(case, elements)
        dst, out, seq = dst + pitch * es * case["ranks"], out + slots * case["chunk"], seq_end
    payloads, records, slot0 = [], [], 0
    for p in range(2):
        d = np.concatenate(sender[p])
        order = np.argsort(np.concatenate(when[p]), kind="stable")
        a = np.concatenate(arrive[p])[order]
        records.append((_fill(d, a, slot0, case["chunk"]), a))
        slot0 += len(a)
        payloads.append(_values(seed, 1 + p, len(d) * (case["chunk"] // es), case["dtype"]).view(len(d), case["chunk"] // es))
    acc = _values(seed, 0, dst // es, case["dtype"])
    return acc, payloads, records, out // es, seq


def _prepare_ring(case, seed):
    tt = DTYPES[case["dtype"]][0]
    acc, payloads, records, out_elements, n_bits = _ring_inputs(case, seed)
    recv = torch.cat([u[torch.from_numpy(a).cuda()] for u, (_, a) in zip(payloads, records) if len(a)]).view(-1)
    out = torch.zeros(out_elements, dtype=tt, device="cuda")
    bitmap = _bitmap(n_bits)
    rejected = torch.zeros(1, dtype=torch.int32, device="cuda")
    calls = [uccl.uccl_prepare(uccl.uccl_dedup_reset, bitmap, n_bits)]
    for op, (d, _) in zip((OPS[case.get("op", "sum")], uccl.UCCL_COPY), records):
        if len(d):
            calls.append(_apply(case, acc, out, recv, _on_gpu(d), len(d), bitmap, op, n_bits, rejected))
    return {"calls": calls, "outputs": {"acc": acc, "out": out, "bitmap": bitmap, "rejected": rejected}}


def _alltoall_lengths(case):
    g = np.random.default_rng(case["sizes"])
    return case["row"] * g.integers(1, max(2, case["most"] // case["row"] + 1), case["sources"])


def _prepare_alltoall(case, seed):
    g = np.random.default_rng(seed)
    lengths, chunk = _alltoall_lengths(case), case["chunk"]
    base, sender, arrive, when, n = 0, [], [], [], 0
    for length in lengths:
        c = np.arange(-(-int(length) // chunk), dtype=np.int64)
        d = np.zeros(len(c), dtype=DESC)
        d["dst_off"], d["out_off"], d["seq"] = base + c * chunk, NO_FORWARD, n + c
        d["len"] = np.minimum(chunk, length - c * chunk)
        a, at = _arrivals(g, len(c), 0, case["dup"])
        arrive.append(a + n)
        when.append(at)
        sender.append(d)
        base, n = base + int(length), n + len(c)
    a = np.concatenate(arrive)[np.argsort(np.concatenate(when), kind="stable")]
    d = _fill(np.concatenate(sender), a, 0, chunk)
    payload = _values(seed, 1, n * (chunk // 2), "bf16").view(n, -1)
    recv = payload[torch.from_numpy(a).cuda()].view(-1)
    dst = torch.zeros(base // 2, dtype=torch.bfloat16, device="cuda")
    bitmap = _bitmap(n)
    rejected = torch.zeros(1, dtype=torch.int32, device="cuda")
    calls, rec = [uccl.uccl_prepare(uccl.uccl_dedup_reset, bitmap, n)], _on_gpu(d)
    if case["entry"] == "opts":
        calls.append(uccl.uccl_prepare(uccl.uccl_chunk_scatter_opts, dst, recv, rec, len(d), bitmap, opts=(chunk, 0)))
    elif case["entry"] == "checked":
        calls.append(uccl.uccl_prepare(uccl.uccl_chunk_scatter_checked, dst, recv, rec, len(d), bitmap, n_rejected=rejected, n_bits=n))
    else:
        calls.append(uccl.uccl_prepare(uccl.uccl_chunk_scatter, dst, recv, rec, len(d), bitmap))
    return {"calls": calls, "outputs": {"acc": dst, "bitmap": bitmap, "rejected": rejected}}


def _direct_inputs(case, seed):
    g = np.random.default_rng(seed)
    es, k, chunk = DTYPES[case["dtype"]][2], case["sources"], case["chunk"]
    elements, per = case["bytes"] // es, chunk // es
    n = -(-elements // per)
    streams = [_arrivals(g, n, 0, case["dup"]) for _ in range(k)]
    order = np.argsort(np.concatenate([at for _, at in streams]), kind="stable")
    chunk_of = np.concatenate([a for a, _ in streams])[order]
    source_of = np.concatenate([np.full(len(a), p) for p, (a, _) in enumerate(streams)])[order]
    first = np.full((k, n), len(order), dtype=np.int64)
    np.minimum.at(first, (source_of, chunk_of), np.arange(len(order)))
    ready = np.argsort(first.max(axis=0), kind="stable")       # a record is issued when its last source is in
    pos = np.concatenate([np.arange(n), np.flatnonzero(g.random(n) < 0.02)])
    seq = ready[pos[np.argsort(np.concatenate([np.arange(n), pos[n:] + 1 + g.random(len(pos) - n) * (n / 4)]), kind="stable")]]
    d = np.zeros(len(seq), dtype=GATHER_DESC)
    d["dst_off"], d["out_off"], d["seq"], d["n_src"] = seq * chunk, NO_FORWARD, seq, k
    d["len"] = np.minimum(per, elements - seq * per) * es
    d["src_off"][:, :k] = (first[:, seq] * chunk).T
    payload = _values(seed, 1, k * n * per, case["dtype"]).view(k, n, per)
    return _values(seed, 0, elements, case["dtype"]), payload, d, source_of, chunk_of


def _prepare_direct(case, seed):
    acc, payload, d, source_of, chunk_of = _direct_inputs(case, seed)
    n = payload.shape[1]
    recv = payload.view(-1, payload.shape[2])[torch.from_numpy(source_of * n + chunk_of).cuda()].view(-1)
    bitmap = _bitmap(n)
    opts = (case["chunk"], 0) if case["entry"] == "opts" else None
    calls = [uccl.uccl_prepare(uccl.uccl_dedup_reset, bitmap, n),
             uccl.uccl_prepare(uccl.uccl_chunk_reduce_gather, acc, None, recv, _on_gpu(d), len(d), bitmap, DTYPES[case["dtype"]][1],
                               OPS[case["op"]], opts=opts)]
    return {"calls": calls, "outputs": {"acc": acc, "bitmap": bitmap}}


def _prepare_segment(case, seed):
    n = -(-case["bytes"] // case["chunk"])
    tensor = _values(seed, 0, -(-case["bytes"] // 4), "f32")
    stage = torch.zeros(n * case["chunk"] // 4, dtype=torch.float32, device="cuda")
    send = torch.zeros(n * uccl.SEND_DESC_BYTES // 4, dtype=torch.int32, device="cuda")
    calls = [uccl.uccl_prepare(uccl.uccl_chunk_segment, stage, tensor, 0, case["bytes"], case["chunk"], send_descs=send, conn_id=seed % 256,
                               msg_id=seed % 128)]
    # compared as whole words: the last one may hold only part of a value
    return {"calls": calls, "keep": tensor, "outputs": {"stage": stage.view(torch.int32), "send": send}}


def _prepare_feedback(case, seed):
    g = np.random.default_rng(seed)

    def packed(bits):
        return torch.from_numpy(np.packbits(np.resize(bits, (len(bits) + 31) // 32 * 32), bitorder="little").view(np.int32).copy()).cuda()

    bits = np.ones(case["bits"], dtype=np.uint8)
    if case["holes"]:
        bits[np.flatnonzero(g.random(case["bits"]) < 1.0 / case["holes"])] = 0
        bits[case["bits"] // 3 + int(g.integers(0, case["bits"] // 3)):] &= (g.random(1) < 0.5).astype(np.uint8)  # or not all sent yet
    known = g.integers(0, 257, case["slots"])
    window = (np.arange(256)[None, :] < np.where(g.random(case["slots"]) < 0.5, known, g.integers(0, 257, case["slots"]))[:, None]).astype(np.uint8)
    bitmap, slots = packed(bits), packed(window.reshape(-1))
    count = torch.from_numpy(known.astype(np.int32)).cuda()
    report = torch.zeros((uccl.ACK_HEADER_BYTES + 16 * case["ranges"]) // 8, dtype=torch.int64, device="cuda")
    status = torch.zeros(4 * case["slots"], dtype=torch.int32, device="cuda")
    calls = [uccl.uccl_prepare(uccl.uccl_dedup_report, bitmap, case["bits"], report, case["ranges"]),
             uccl.uccl_prepare(uccl.uccl_message_status, slots, count, case["slots"], 256, status)]
    return {"calls": calls, "outputs": {"report": report, "status": status}}


def prepare(case, seed):
    """Buffers, records and the marshalled calls that a control path keeps for a connection."""
    return {"ring": _prepare_ring, "batch": _prepare_ring, "alltoall": _prepare_alltoall, "direct": _prepare_direct, "segment": _prepare_segment,
            "feedback": _prepare_feedback}[case["kind"]](case, seed)


def run(state):
    for call in state["calls"]:
        call()
    return state["outputs"]


# ---- what a pass needs, and what it gives ---------------------------------------------------------

def _records(n, dup, size=36):
    return size * n * (1 + dup)


def work(case):
    """Payload once from its slot, accumulator read where it is combined and written where it is kept, staging copy
    written; a record and a bitmap word per arrival."""
    if case["kind"] in ("ring", "batch"):
        es = DTYPES[case["dtype"]][2]
        total = flops = 0
        for elements in [case["bytes"] // es] if case["kind"] == "ring" else _message_elements(case):
            seg, _, _, cps, reduce_, copy = _ring_plan(case, elements)
            for _, forward, only in reduce_:
                total += seg * es * (2 + forward + (not only))
                flops += seg
            for _, forward, _ in copy:
                total += seg * es * (2 + forward)
            total += _records(cps * (len(reduce_) + len(copy)), case["dup"])
        return {"bytes": total, "flops": flops}
    if case["kind"] == "alltoall":
        lengths = _alltoall_lengths(case)
        return {"bytes": int(2 * lengths.sum()) + _records(int((-(-lengths // case["chunk"])).sum()), case["dup"]), "flops": 0}
    if case["kind"] == "direct":
        es = DTYPES[case["dtype"]][2]
        return {"bytes": case["bytes"] * (case["sources"] + 2) + _records(-(-case["bytes"] // case["chunk"]), 0.02, 164),
                "flops": case["bytes"] // es * case["sources"]}
    if case["kind"] == "segment":
        return {"bytes": 2 * case["bytes"] + 16 * -(-case["bytes"] // case["chunk"]), "flops": 0}
    ranges = min(case["ranges"], case["bits"] // case["holes"] if case["holes"] else 0)
    return {"bytes": case["bits"] // 8 + 32 + 16 * ranges + case["slots"] * (32 + 4 + 16), "flops": 0}


def tolerance(case):
    """One binary32 operation and one rounding per element, or a fold in a stated order: no freedom in the result."""
    return "exact"


def _combine(op, a, r):
    return a + r if op == "sum" else torch.maximum(a, r) if op == "max" else torch.minimum(a, r)


def exact(case, seed):
    """The sums and selections of a pass in 64 bits."""
    if case.get("dtype") == "i32" or case["kind"] not in ("ring", "batch", "direct"):
        return None  # whole numbers and copies
    es = DTYPES[case["dtype"]][2]
    if case["kind"] == "direct":
        acc, payload, _, _, _ = _direct_inputs(case, seed)
        t = acc.double()
        for p in range(case["sources"]):
            t = _combine(case["op"], t, payload[p].reshape(-1)[: len(t)].double())
        return {"acc": t, "bitmap": None}
    acc, payloads, _, out_elements, _ = _ring_inputs(case, seed)
    t, out = acc.double(), torch.zeros(out_elements, dtype=torch.float64, device="cuda")
    many = [case["bytes"] // es] if case["kind"] == "ring" else _message_elements(case)
    base, at, slot = 0, [0, 0], 0
    for elements in many:
        seg, pitch, per, cps, reduce_, copy = _ring_plan(case, elements)
        for p, steps in enumerate((reduce_, copy)):
            for segment, forward, only in steps:
                r = payloads[p][at[p]: at[p] + cps].reshape(-1)[:seg].double()
                at[p] += cps
                lo = base + segment * pitch
                v = r if p else _combine(case.get("op", "sum"), t[lo: lo + seg], r)
                if not only:
                    t[lo: lo + seg] = v
                if forward:
                    out[slot * per: slot * per + seg] = v
                    slot += cps
        base += pitch * case["ranks"]
    return {"acc": t, "out": out, "bitmap": None, "rejected": None}
