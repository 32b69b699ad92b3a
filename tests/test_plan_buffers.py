"""Plans that come and go: the buffers of a destroyed plan serve the next one, also while another stream
still decodes with the destroyed plan's copy.  Making a plan waits for no stream and breaks no capture."""
import ctypes
import threading

import pytest
import torch

import paper_2511_22481_amd as oa
import parity
from workloads import make_custom


@pytest.mark.gpu
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_buffers_of_destroyed_plans_are_reused_safely(kv):
    problems = [parity.to_device(make_custom(b, 128, [L + 37 * i for i in range(b)], 64, w, seed=b, kv_dtype=kv, q_std=0.7, kv_std=0.7))
                for b, L, w in ((3, 700, 512), (40, 3000, 2048), (1, 90, 4096), (7, 2000, 100))]
    want = []
    for inp in problems:
        out, lse, plan = parity.run_gpu(inp)
        want.append((out, lse, plan))                 # kept alive: these plans own their buffers
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    got = []
    for rep in range(12):
        k = rep % len(problems)
        inp = problems[k]
        with torch.cuda.stream(streams[rep % 2]):
            plan = oa.omniattn_plan(inp.seq_lens_host, batch=inp.q.shape[0], num_heads=128, max_pages_per_seq=inp.page_table.shape[1],
                                    num_pages=inp.kv_cache.shape[0], sink=inp.sink, window=inp.window,
                                    softmax_scale=inp.softmax_scale, kv_dtype=oa.FP8_E4M3 if kv == "fp8" else oa.BF16)
            out, lse = torch.empty_like(want[k][0]), torch.empty_like(want[k][1])
            ws = torch.empty(max(plan.workspace_bytes, 1), dtype=torch.uint8, device="cuda")
            for _ in range(4):
                oa.omniattn_decode(plan, inp.q, inp.kv_cache, inp.kv_scales, inp.page_table, out, lse, ws)
            got.append((k, out, lse, ws))
            plan.destroy()                            # its kernels may still run
    torch.cuda.synchronize()
    for k, out, lse, _ in got:
        assert torch.equal(out, want[k][0]) and torch.equal(lse, want[k][1])


def _spare_buffers():
    """Leaves buffers of destroyed plans behind, for the next plan to take."""
    plans = [_small_plan(None) for _ in range(3)]
    for p in plans:
        p.destroy()
    torch.cuda.synchronize()


def _small_plan(stream):
    return oa.omniattn_plan([700, 900], stream=stream, batch=2, num_heads=64, max_pages_per_seq=8, num_pages=16, sink=16,
                            window=256, softmax_scale=0.1)


@pytest.mark.gpu
@pytest.mark.parametrize("mode, thread", [("thread_local", True), ("relaxed", True), ("relaxed", False)])
def test_a_plan_is_made_while_a_stream_captures(mode, thread):
    """The modes in which hipMalloc is allowed: a plan can be made (on a stream that does not capture) and
    destroyed, and the capture comes out whole."""
    _spare_buffers()
    side, other, x, made = torch.cuda.Stream(), torch.cuda.Stream(), torch.zeros(64, device="cuda"), []

    def make():
        for _ in range(2):
            made.append(_small_plan(other))
            made[-1].destroy()
        made.append(_small_plan(other))

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side, capture_error_mode=mode):
        x.add_(1)
        if thread:
            t = threading.Thread(target=make)
            t.start()
            t.join()
        else:
            make()
        x.add_(1)
    assert len(made) == 3 and made[-1].num_units > 0
    x.zero_()
    for rep in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert float(x[5]) == 2 * (rep + 1)


@pytest.mark.gpu
def test_making_a_plan_waits_for_no_stream():
    _spare_buffers()
    busy, done = torch.cuda.Stream(), torch.cuda.Event()
    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    with torch.cuda.stream(busy):
        a @ a
    torch.cuda.synchronize()
    with torch.cuda.stream(busy):
        for _ in range(60):                              # 1 ms each
            a @ a
        done.record()
    plan = _small_plan(torch.cuda.current_stream())
    still_running = not done.query()
    torch.cuda.synchronize()
    assert still_running and plan.num_units > 0


def _busy(stream, n=60):
    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    torch.cuda.synchronize()
    done = torch.cuda.Event()
    with torch.cuda.stream(stream):
        for _ in range(n):                               # 1 ms each
            a @ a
        done.record()
    return done


@pytest.mark.gpu
def test_a_one_call_decode_waits_for_nothing():
    """Its plan is gone when it returns, and with it went device memory whose release waits for all streams."""
    inp = parity.to_device(make_custom(3, 48, [700, 90, 2000], 64, 512, seed=1, q_std=0.7, kv_std=0.7))
    want = parity.run_gpu(inp)
    _spare_buffers()
    done = _busy(torch.cuda.Stream())
    args = (inp.q, inp.kv_cache, inp.kv_scales, inp.page_table, inp.seq_lens_host, inp.sink, inp.window, inp.softmax_scale)
    got = [oa.decode(*args)[:2] for _ in range(5)]
    still_running = not done.query()
    torch.cuda.synchronize()
    assert still_running
    for out, lse in got:
        assert torch.equal(out, want[0]) and torch.equal(lse, want[1])


@pytest.mark.gpu
@pytest.mark.parametrize("big", [False, True])
def test_plan_of_a_one_call_decode_on_another_stream(big):
    """The plan that the call returns is used on a second, busy stream and dropped at once: its device copy stays whole
    until that decode is done, whatever is allocated in the meantime.  (big: a plan that outgrows the wrapper's buffer.)"""
    n = 2000 if big else 5
    inp = parity.to_device(make_custom(n, 64, [1 + (37 * i) % 400 for i in range(n)], 16, 128, seed=2, q_std=0.7, kv_std=0.7))
    want, want_lse, keep = parity.run_gpu(inp)
    assert (keep.num_units * 48 + keep.num_segments * 32 > 1 << 16) == big
    args = (inp.q, inp.kv_cache, inp.kv_scales, inp.page_table)
    other, results = torch.cuda.Stream(), []
    ws = torch.empty(max(keep.workspace_bytes, 256), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    for rep in range(4):
        plan = oa.decode(*args, inp.seq_lens_host, inp.sink, inp.window, inp.softmax_scale)[2]
        torch.cuda.synchronize()
        _busy(other, 5)
        out, lse = torch.zeros_like(want), torch.zeros_like(want_lse)
        other.wait_stream(torch.cuda.current_stream())
        oa.omniattn_decode(plan, *args, out, lse, ws, stream=other)
        del plan
        junk = [torch.full((1 << 16,), 255, dtype=torch.uint8, device="cuda") for _ in range(8)]
        torch.cuda.synchronize()
        results.append((out, lse, len(junk)))
    for out, lse, _ in results:
        assert torch.equal(out, want) and torch.equal(lse, want_lse)


def _one_call(window=512):
    inp = parity.to_device(make_custom(3, 48, [700, 90, 2000], 64, window, seed=1, q_std=0.7, kv_std=0.7))
    return (inp.q, inp.kv_cache, inp.kv_scales, inp.page_table, inp.seq_lens_host, inp.sink, inp.window, inp.softmax_scale)


@pytest.mark.gpu
def test_dropping_several_one_call_plans_waits_for_nothing():
    """More of them than the three that leave their pinned buffers behind, as a program has that keeps what the call returns."""
    args = _one_call()
    want = oa.decode(*args)[:2]
    _spare_buffers()
    held = [oa.decode(*args) for _ in range(6)]
    torch.cuda.synchronize()
    done = _busy(torch.cuda.Stream())
    got = [r[:2] for r in held]
    del held
    still_running = not done.query()
    torch.cuda.synchronize()
    assert still_running
    for out, lse in got:
        assert torch.equal(out, want[0]) and torch.equal(lse, want[1])


@pytest.mark.gpu
def test_one_call_decodes_run_ahead_of_their_stream():
    args = _one_call()
    want = oa.decode(*args)[:2]
    _spare_buffers()
    done = _busy(torch.cuda.current_stream())
    got = [oa.decode(*args)[:2] for _ in range(12)]
    still_running = not done.query()
    torch.cuda.synchronize()
    assert still_running
    for out, lse in got:
        assert torch.equal(out, want[0]) and torch.equal(lse, want[1])


@pytest.mark.gpu
def test_more_plans_than_are_kept():
    """Made and dropped while their stream is busy, of two sizes, so that kept buffers give way to larger ones whose place
    they take, and are freed with their copies still under way."""
    big = parity.to_device(make_custom(1300, 16, [1 + (37 * i) % 400 for i in range(1300)], 16, 128, seed=2, q_std=0.7, kv_std=0.7))
    big_args = (big.q, big.kv_cache, big.kv_scales, big.page_table, big.seq_lens_host, big.sink, big.window, big.softmax_scale)
    args = _one_call()
    want, want_big = oa.decode(*args)[:2], oa.decode(*big_args)[:2]
    torch.cuda.synchronize()
    _busy(torch.cuda.current_stream(), 5)
    held = [oa.decode(*args) for _ in range(24)] + [oa.decode(*big_args) for _ in range(4)]
    got = [r[:2] for r in held]
    del held
    got += [oa.decode(*args)[:2] for _ in range(40)]
    torch.cuda.synchronize()
    for out, lse in got:
        w = want if out.shape == want[0].shape else want_big
        assert torch.equal(out, w[0]) and torch.equal(lse, w[1])


@pytest.mark.gpu
def test_update_of_a_one_call_plan_that_outgrows_its_buffer():
    """Pieces of one tile first, 24 KB of metadata in the wrapper's 64 KB; then eight pieces a sequence, in memory of the
    plan's own; then short sequences again."""
    n = 300
    short, long = [20 + i % 12 for i in range(n)], [400 + i % 100 for i in range(n)]
    inp = parity.to_device(make_custom(n, 64, long, 16, 1024, seed=2, q_std=0.7, kv_std=0.7))
    args = (inp.q, inp.kv_cache, inp.kv_scales, inp.page_table)
    rest = (inp.sink, inp.window, inp.softmax_scale)
    small, small_lse, plan = oa.decode(*args, short, *rest, num_splits_hint=8)
    want, want_lse, ref = oa.decode(*args, long, *rest, num_splits_hint=8)
    size = lambda p: p.num_units * 48 + p.num_segments * 32
    assert size(plan) < 1 << 16 < size(ref)
    for lens, w, w_lse in ((long, want, want_lse), (short, small, small_lse), (long, want, want_lse)):
        oa.omniattn_plan_update(plan, lens)
        ws = torch.empty(max(plan.workspace_bytes, 256), dtype=torch.uint8, device="cuda")
        out, lse = torch.zeros_like(want), torch.zeros_like(want_lse)
        oa.omniattn_decode(plan, *args, out, lse, ws)
        torch.cuda.synchronize()
        assert torch.equal(out, w) and torch.equal(lse, w_lse)


def _plan_in(buffer, size):
    prob = oa.binding._problem(batch=2, num_heads=64, max_pages_per_seq=8, num_pages=16, sink=16, window=256, softmax_scale=0.1)
    lens, address = oa.binding._lens_array([700, 900])
    h = ctypes.c_void_p()
    return oa.load_library().omniattn_plan_in(ctypes.byref(h), ctypes.byref(prob), address, buffer, size, None), h


@pytest.mark.parametrize("offset", [1, 4, 8, 15])
def test_a_misaligned_plan_buffer_is_refused(offset):
    rc, h = _plan_in(4096 + offset, 1 << 16)
    assert rc == -1 and not h.value


@pytest.mark.gpu
@pytest.mark.parametrize("size", [0, 15, 16, 1 << 16])
def test_plan_buffer_of_any_size(size):
    """One that does not hold the metadata is left alone: memory of the plan's own instead."""
    buffer = torch.full((1 << 16,), 77, dtype=torch.uint8, device="cuda")
    rc, h = _plan_in(buffer.data_ptr(), size)
    assert rc == 0 and h.value
    torch.cuda.synchronize()
    assert bool((buffer == 77).all()) == (size < 1 << 16)
    oa.load_library().omniattn_plan_destroy(h)
