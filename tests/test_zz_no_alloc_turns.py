"""Calls of the no-allocation entry point share one array of claim words: eager and captured calls in turn (the
captured ones clear their words first), and calls that run in another order than they were made."""
import time

import pytest
import torch

from synth import workloads as wl
from synth.layout import BF16

from gpuhelp import DeviceRun, oracle_results, assert_same

pytestmark = pytest.mark.gpu


def test_eager_calls_between_replays(gpu_lib):
    captured, eager = wl.config1(seed=17), wl.ring_share("eager", 18, R=4, M=4 * (9 * 40960 + 528), C=40960, dtype=BF16, paths=3,
                                                         window=None, dup=0.2, dist="normal")
    want = {w.name: oracle_results(w) for w in (captured, eager)}

    def issue(run, w):
        gpu_lib.uccl_dedup_reset(run.bitmap, w.n_bits)
        for ph, d in zip(w.phases, run.descs):
            gpu_lib.uccl_chunk_apply_noalloc(run.acc, run.out, run.recv, d, len(ph.descs), run.bitmap, w.dtype, ph.op)

    def check(run, w, what):
        torch.cuda.synchronize()
        for got, exp, name in zip(run.results(), want[w.name], ("acc", "out_stage", "bitmap")):
            assert_same(got, exp, f"{w.name}, {what}: {name}")

    gpu_lib.uccl_init()
    run = DeviceRun(captured)
    acc0 = run.acc.clone()
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        issue(run, captured)
    for turn in range(4):
        for _ in range(turn):                      # none, then several eager calls between two replays
            mine = DeviceRun(eager)
            issue(mine, eager)
            check(mine, eager, f"turn {turn}")
        run.acc.copy_(acc0)
        graph.replay()
        check(run, captured, f"replay {turn}")
    assert gpu_lib.uccl_claim_timeouts() == 0


def test_calls_that_run_in_another_order_than_they_were_made(gpu_lib):
    """A call held back on its stream is overtaken by one that was made after it on another stream: both are applied
    whole, whichever of them the array's words remember."""
    held_back, overtaking = wl.config1(seed=19), wl.config1(seed=20)
    want = [oracle_results(w) for w in (held_back, overtaking)]
    runs = [DeviceRun(w) for w in (held_back, overtaking)]
    first, opened = torch.cuda.Stream(), torch.cuda.Event()
    a, x = torch.randn(8192, 8192, device="cuda"), torch.zeros(64, device="cuda")

    def issue(run, w, stream):
        for ph, d in zip(w.phases, run.descs):
            gpu_lib.uccl_chunk_apply_noalloc(run.acc, run.out, run.recv, d, len(ph.descs), run.bitmap, w.dtype, ph.op, stream=stream)

    def overtakes(stream):                          # streams share hardware queues: one that does not wait behind `first`
        done = torch.cuda.Event()
        with torch.cuda.stream(stream):
            x.add_(1.0)
            done.record()
        end = time.monotonic() + 0.02
        while not done.query() and time.monotonic() < end:
            pass
        return done.query()

    torch.mm(a, a)
    torch.cuda.synchronize()
    with torch.cuda.stream(first):
        for _ in range(60):                         # some hundred milliseconds of other work
            torch.mm(a, a)
        opened.record()
    issue(runs[0], held_back, first)
    second = next(s for s in (torch.cuda.Stream() for _ in range(8)) if overtakes(s))
    issue(runs[1], overtaking, second)
    second.synchronize()
    overtaken = not opened.query()
    torch.cuda.synchronize()
    assert overtaken, "the first call was not held back long enough: nothing shown"
    for run, w, expected in zip(runs, (held_back, overtaking), want):
        for got, exp, name in zip(run.results(), expected, ("acc", "out_stage", "bitmap")):
            assert_same(got, exp, f"{w.name}: {name}")
    assert gpu_lib.uccl_claim_timeouts() == 0
