"""The work partition's three shapes, and the merge of few and many partial rows per sequence
(up to 8 partials one wave takes a head row, from 9 on four waves share it)."""
import random
import time

import pytest
import torch

import paper_2511_22481_amd as oa
import parity
from test_abi_and_plan import check_plan
from test_multi_query import _run
from workloads import make_custom


def test_whole_sequences_when_they_fill_the_units_evenly():
    p = check_plan([40000] * 256, 128, 4096)
    assert p.num_units == 256 and p.num_partials == 0
    p = check_plan([40000] * 512, 128, 4096)
    assert p.num_units == 256 and p.num_partials == 0


def test_even_pieces_for_a_few_equal_sequences():
    p = oa.omniattn_plan_host([131072] * 32, batch=32, num_heads=128, max_pages_per_seq=1024, num_pages=1 << 15,
                              sink=128, window=8192, softmax_scale=0.1, kv_dtype=oa.FP8_E4M3)
    pieces = [s["tile_hi"] - s["tile_lo"] for s in p.segments()]
    assert p.num_segments == p.num_units == 256 and max(pieces) - min(pieces) <= 1


def test_filled_units_when_the_count_is_odd():
    p = check_plan([40000] * 300, 128, 4096)
    load = [0] * p.num_units
    for s in p.segments():
        load[s["unit"]] += s["tile_hi"] - s["tile_lo"]
    assert p.num_units <= 256 and max(load) < 2 * 133      # whole sequences would give some unit two


@pytest.mark.parametrize("out_dtype", [oa.BF16, oa.FP32])
def test_short_pieces_stay_inside_the_static_scratch(out_dtype):
    p = oa.omniattn_plan_host([20000] * 2, batch=2, num_heads=128, max_pages_per_seq=157, num_pages=314, sink=0,
                              window=4096, softmax_scale=0.1, out_dtype=out_dtype)
    assert 64 <= p.num_partials and p.workspace_bytes <= oa.omniattn_static_scratch_bytes()


@pytest.mark.parametrize("batch, length, heads, q_len, sink, window",
                         [(29, 8000, 48, 8, 64, 1212), (88, 13124, 33, 2, 0, 1369)])
def test_filled_units_stay_inside_the_static_scratch(batch, length, heads, q_len, sink, window):
    """With the measured cost of a segment the fill cuts these into 319 and 323 partials, 41.98 and 42.5 MB of
    partial rows; at a cost of one tile into 313 and 317, which the buffer holds."""
    p = oa.omniattn_plan_host([length] * batch, batch=batch, num_heads=heads, max_pages_per_seq=110, num_pages=1 << 14, sink=sink,
                              window=window, softmax_scale=0.1, q_len=q_len)
    assert 0 < p.workspace_bytes <= oa.omniattn_static_scratch_bytes()
    check_segments(p, batch)


@pytest.mark.parametrize("batch, heads, q_len, lo, hi, sink, window, seed",
                         [(9, 160, 4, 2845, 2845, 64, 16409, 284), (66, 48, 2, 14, 8379, 0, 8981, 3743),
                          (49, 128, 1, 366, 63163, 130, 6693, 1762), (53, 128, 1, 7337, 23298, 128, 5266, 515)])
def test_fp8_with_fp32_results_stays_inside_the_static_scratch(batch, heads, q_len, lo, hi, sink, window, seed):
    """The 128-row plans of these, cheapest by the estimate, need 59 to 76 MB of fp32 partial rows; 64-row plans fit."""
    rng = random.Random(seed)
    lens = [rng.randint(lo, hi) for _ in range(batch)]
    p = oa.omniattn_plan_host(lens, batch=batch, num_heads=heads, max_pages_per_seq=512, num_pages=1 << 16, sink=sink,
                              window=window, softmax_scale=0.1, kv_dtype=oa.FP8_E4M3, out_dtype=oa.FP32, q_len=q_len)
    assert 0 < p.workspace_bytes <= oa.omniattn_static_scratch_bytes() and p.num_units <= 256
    check_segments(p, batch)


def _planning_us(lens, **problem):
    def once():
        t = time.perf_counter()
        oa.omniattn_plan_host(lens, batch=len(lens), max_pages_per_seq=512, num_pages=1 << 18, softmax_scale=0.1, **problem)
        return time.perf_counter() - t
    return 1e6 * min(once() for _ in range(30))


@pytest.mark.parametrize("batch, q_len, sink, window, lo, hi", [
    (222, 3, 128, 3363, 953, 2421), (178, 3, 4, 787, 953, 2421), (189, 2, 4, 3707, 953, 4421), (513, 4, 130, 41716, 600, 60000),
    (256, 1, 0, 32768, 512, 32768), (300, 1, 0, 32768, 20000, 40000), (1000, 1, 0, 32768, 512, 32768)])
def test_planning_time_of_large_ragged_batches(batch, q_len, sink, window, lo, hi):
    """A serving loop plans before every decode step.  Finding the partition takes at most six times as long as
    writing one down that is given (1.5 to 2.6 times; with every capacity tried one by one it was 9 to 29 times)."""
    rng = random.Random(batch)
    lens = [rng.randint(lo, hi) for _ in range(batch)]
    prob = dict(num_heads=128, q_len=q_len, sink=sink, window=window, kv_dtype=oa.FP8_E4M3)
    found, given = _planning_us(lens, **prob), _planning_us(lens, num_splits_hint=1, **prob)
    assert found < 6 * given, (found, given)


def check_segments(p, batch):
    segs, ends = p.segments(), {}
    for s in segs:
        assert s["tile_lo"] == ends.get((s["b"], s["hb"]), 0) and s["tile_hi"] > s["tile_lo"] and s["unit"] < p.num_units
        ends[s["b"], s["hb"]] = s["tile_hi"]
    assert {b for b, _ in ends} == set(range(batch)) and all(ends[s["b"], s["hb"]] == s["ntiles"] for s in segs)


@pytest.mark.gpu
@pytest.mark.parametrize("out_dtype", [None, torch.float32])
@pytest.mark.parametrize("hint", [8, 9, 13, 1000])
def test_merge_of_many_partials(hint, out_dtype):
    inp = parity.to_device(make_custom(3, 48, [1500, 2100, 65], 64, 1024, seed=hint, q_std=1.0, kv_std=1.0))
    out, lse, plan = parity.run_gpu(inp, out_dtype=out_dtype, num_splits_hint=hint)
    assert plan.max_splits == min(hint, (64 + 1024) // plan.tile_tokens + 1)
    parity.assert_parity(inp, out, lse, row_rel_l2=1e-2, what=f"{plan.max_splits} partials")


def test_kernel_for_few_rows_or_few_sequences():
    # 32 rows or fewer: always blocks of 32; more rows: where the sequences are too few for long pieces
    assert check_plan([32768] * 64, 128, 2048, H=16).head_block == 32
    assert check_plan([32768] * 2, 128, 2048, H=33).head_block == 32
    assert check_plan([20011], 128, 2048).head_block == 32
    assert check_plan([20011] * 64, 128, 2048).head_block == 128


@pytest.mark.gpu
@pytest.mark.parametrize("out_dtype", [None, torch.float32])
@pytest.mark.parametrize("b", [9, 10, 11, 24])
def test_merge_of_many_rows(b, out_dtype):
    """13 partials save three round trips: up to 1350 rows (10 sequences of 128 heads) four waves share each row, more
    are left to a wave each."""
    inp = parity.to_device(make_custom(b, 128, [33 + 32 * (i % 13) for i in range(b - 1)] + [13 * 32], 0, 1024, seed=b, q_std=1.0, kv_std=1.0))
    out, lse, plan = parity.run_gpu(inp, out_dtype=out_dtype, num_splits_hint=13)
    assert plan.max_splits == 13
    parity.assert_parity(inp, out, lse, row_rel_l2=1e-2, what=f"{b} sequences of up to 13 partials")


def _nan_at(inp, b, position):
    inp.kv_cache[int(inp.page_table[b, position // 128]), position % 128, 100] = float("nan")


@pytest.mark.gpu
@pytest.mark.parametrize("out_dtype", [None, torch.float32])
@pytest.mark.parametrize("heads", [16, 64, 128])
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_a_nan_partial_reaches_the_merged_row(kv, heads, out_dtype):
    """Sequences cut into 2 .. 13 partials, one of them NaN, each in turn, beside ones without: the launch
    merges with four waves per row (13 partials), so in an item of up to 7 some wave holds the NaN partial alone."""
    tile = 64 if kv == "fp8" else 32
    cuts = [(k, slot) for k in (2, 3, 4, 5, 6, 7, 13) for slot in range(k)]
    lens = [k * tile for k, _ in cuts] + [2 * tile, 6 * tile, 13 * tile]
    inp = make_custom(len(lens), heads, lens, 0, 4096, seed=heads, kv_dtype=kv, q_std=0.7, kv_std=0.7)
    for b, (_, slot) in enumerate(cuts):
        _nan_at(inp, b, slot * tile + 5)
    inp = parity.to_device(inp)
    out, lse, plan = parity.run_gpu(inp, out_dtype=out_dtype, num_splits_hint=13)
    assert plan.max_splits == 13 and plan.num_partials == sum(lens) // tile * -(-heads // plan.head_block)
    nan = torch.isnan(out).flatten(1)
    missed = [c for b, c in enumerate(cuts) if not nan[b].all()]
    assert not missed, f"finite rows although partial `slot` of `k` is NaN: {missed}"
    assert not nan[len(cuts):].any()
    assert torch.equal(torch.isnan(lse), nan.all(dim=1, keepdim=True).expand_as(lse))


@pytest.mark.gpu
@pytest.mark.parametrize("pieces, nan_slots", [(2, (1,)), (13, (4, 8, 12))])
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_nan_beside_an_empty_partial(kv, pieces, nan_slots):
    """Two queries whose windows end one token apart: the later one keeps nothing of the first tile, so its
    first partial is empty (lse -inf), and the others of the wave that merges it are NaN."""
    tile = 64 if kv == "fp8" else 32
    inp = make_custom(2, 2 * 16, [16 * tile] * 2, 0, (pieces - 1) * tile, seed=3, kv_dtype=kv, q_std=0.7, kv_std=0.7)
    for slot in nan_slots:
        _nan_at(inp, 0, (16 - pieces + slot) * tile + 7)
    inp = parity.to_device(inp)
    out, lse, plan = _run(inp, 2, 16, num_splits_hint=1000)
    assert plan.max_splits == pieces
    assert torch.isnan(out[0]).all() and not torch.isnan(out[1]).any()
    assert torch.isnan(lse[0]).all() and not torch.isnan(lse[1]).any()


@pytest.mark.gpu
def test_a_row_of_nan_partials_only():
    inp = make_custom(2, 16, [300, 300], 0, 4096, seed=5, q_std=0.7, kv_std=0.7)
    inp.q[0, 3, 17] = float("nan")                        # the logits of every token
    inp = parity.to_device(inp)
    for hint in (2, 4, 1000):
        out, lse, plan = parity.run_gpu(inp, num_splits_hint=hint)
        nan = torch.isnan(out).all(dim=-1)
        assert nan[0, 3] and int(nan.sum()) == 1 and int(torch.isnan(out).sum()) == 512
        assert torch.equal(torch.isnan(lse), nan)
