"""The kernels for blocks of 32, 64 and 128 head rows on the same short, ragged problems: no
tile, one, two or three tiles (fewer than are requested ahead), ragged ends, windows that open inside a
tile, several queries per sequence, rows past the last head; one segment per unit first, then (as the planner
has them for large batches) several, in blocks that it chooses."""
import dataclasses
import random

import pytest
import torch

import paper_2511_22481_amd as oa
import parity
from test_multi_query import _check, _run
from workloads import make_custom, poison_unretained
from workloads.generate import quantize_fp8_per_token


def _problem(kv, heads, q_len, sink, window):
    lens = [q_len, 5 + q_len, 31, 64, 65, 127, 200, 333, 2047, 3000, 0]
    return parity.to_device(make_custom(len(lens), heads * q_len, lens, sink, window, seed=heads + window, kv_dtype=kv,
                                        q_std=0.7, kv_std=0.7))


@pytest.mark.gpu
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("heads, q_len", [(1, 1), (17, 1), (32, 1), (33, 1), (64, 1), (128, 1), (16, 2), (11, 3), (40, 2)])
def test_blocks_of_32_rows(kv, heads, q_len):
    for sink, window in ((3, 40), (64, 512), (0, 4096)):
        inp = _problem(kv, heads, q_len, sink, window)
        for out_dtype in (None, torch.float32):
            out, lse, plan = _run(inp, q_len, heads, out_dtype=out_dtype)
            assert plan.head_block == 32
            _check(inp, out, lse, q_len, f"{heads} heads, {sink}/{window}")


@pytest.mark.gpu
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("heads, q_len", [(33, 1), (64, 1), (65, 1), (128, 1), (20, 2), (13, 4), (40, 2)])
def test_larger_blocks(kv, heads, q_len):
    """One work unit per sequence and head block: 64 rows (fp8 cache, up to 64 rows) or 128."""
    for sink, window in ((3, 40), (64, 512), (0, 4096)):
        inp = _problem(kv, heads, q_len, sink, window)
        for out_dtype in (None, torch.float32):
            out, lse, plan = _run(inp, q_len, heads, num_splits_hint=1, out_dtype=out_dtype)
            assert plan.head_block == (64 if kv == "fp8" and heads * q_len <= 64 else 128)
            _check(inp, out, lse, q_len, f"{heads} heads, {sink}/{window}")


# (sequences, shortest, longest, sink, window)
SHORT, MIDDLE, LONG = (500, 1, 200, 16, 96), (150, 1, 1500, 16, 600), (90, 1, 4000, 64, 2048)


@pytest.mark.gpu
@pytest.mark.parametrize("kv, heads, q_len, lengths, block", [
    ("fp8", 33, 1, SHORT, 64), ("fp8", 64, 1, SHORT, 64), ("fp8", 16, 3, SHORT, 64),
    ("fp8", 65, 1, MIDDLE, 64), ("fp8", 80, 1, MIDDLE, 64), ("fp8", 96, 1, MIDDLE, 64), ("fp8", 128, 1, MIDDLE, 64),
    ("fp8", 40, 2, MIDDLE, 64), ("fp8", 37, 3, MIDDLE, 64), ("fp8", 160, 1, LONG, 64),
    ("fp8", 80, 1, SHORT, 128), ("fp8", 128, 1, SHORT, 128), ("fp8", 160, 1, SHORT, 128), ("fp8", 40, 2, SHORT, 128),
    ("bf16", 80, 1, SHORT, 128), ("bf16", 48, 3, SHORT, 128),
    ("fp8", 16, 1, SHORT, 32), ("bf16", 16, 1, SHORT, 32), ("bf16", 11, 2, SHORT, 32), ("fp8", 48, 1, MIDDLE, 32),
    ("fp8", 80, 1, LONG, 32)])
def test_several_segments_per_unit(kv, heads, q_len, lengths, block):
    """The planner's own choice of kernel, units that run two to four segments of none, one, two and more tiles, last
    blocks of a few rows (a second block of 1, 16, 32 of 64, a third of 32), queries that end inside a block."""
    n, lo, hi, sink, window = lengths
    rng = random.Random(n)
    lens = [0 if rng.random() < 0.05 else max(q_len, rng.randint(lo, hi)) for _ in range(n)]
    inp = parity.to_device(make_custom(n, heads * q_len, lens, sink, window, seed=heads + n, kv_dtype=kv, q_std=0.7, kv_std=0.7))
    exact, exact_lse, plan = _run(inp, q_len, heads, out_dtype=torch.float32)
    assert plan.head_block == block and plan.num_segments > plan.num_units
    assert {0, 1, 2, 3} <= {s["tile_hi"] - s["tile_lo"] for s in plan.segments()}
    _check(inp, exact, exact_lse, q_len, f"{heads} heads, {lengths}")
    # bf16 results: the same numbers rounded where no partial rows lie in between
    out, lse, plan = _run(inp, q_len, heads)
    assert plan.head_block == block and plan.num_segments > plan.num_units
    if plan.num_partials == 0:
        assert torch.equal(exact.to(torch.bfloat16), out) and torch.equal(exact_lse, lse)
    else:
        _check(inp, out, lse, q_len, f"{heads} heads, {lengths}, bf16 results")


@pytest.mark.gpu
@pytest.mark.parametrize("heads, q_len", [(128, 1), (60, 2)])
def test_filled_units_of_64_rows(heads, q_len):
    """Partial rows and whole ones from the same unit: sequences cut wherever a unit is full."""
    n, lo, hi, sink, window = LONG
    rng = random.Random(n)
    lens = [0 if rng.random() < 0.05 else rng.randint(q_len, hi) for _ in range(n)]
    inp = parity.to_device(make_custom(n, heads * q_len, lens, sink, window, seed=heads, kv_dtype="fp8", q_std=0.7, kv_std=0.7))
    out, lse, plan = _run(inp, q_len, heads)
    assert plan.head_block == 64 and plan.num_segments > plan.num_units and plan.num_segments > plan.num_partials > 256
    _check(inp, out, lse, q_len, f"{heads} heads")


@pytest.mark.gpu
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("heads", [16, 64, 128])
def test_poison_and_page_order_in_every_kernel(kv, heads):
    """One work unit per sequence and head block, as in test_larger_blocks: what is not kept, and where its pages lie,
    has no influence."""
    lens, sink, window = [1000, 77, 400, 2600], 40, 150
    inp = make_custom(4, heads, lens, sink, window, seed=8, kv_dtype=kv, q_std=1.0, kv_std=1.0, spare_pages=4)
    perm = torch.randperm(inp.num_pages, generator=torch.Generator().manual_seed(99))
    table = inp.page_table.clone()
    table[table >= 0] = perm[inp.page_table[inp.page_table >= 0].long()].to(torch.int32)
    moved = dataclasses.replace(inp, page_table=table, kv_cache=torch.empty_like(inp.kv_cache), kv_scales=None)
    moved.kv_cache[perm] = inp.kv_cache
    if kv == "fp8":
        moved.kv_scales = torch.empty_like(inp.kv_scales)
        moved.kv_scales[perm] = inp.kv_scales
    inp = parity.to_device(inp)
    out, lse, plan = parity.run_gpu(inp, num_splits_hint=1)
    assert plan.head_block == {16: 32, 64: 64 if kv == "fp8" else 128, 128: 128}[heads]
    parity.assert_parity(inp, out, lse, row_rel_l2=1e-2, what=f"{kv}, {heads} heads")
    keep = [[j < L and (j < sink or j >= L - window) for j in range(-(-L // 128) * 128)] for L in lens]
    for other in (inp, parity.to_device(moved)):
        poison_unretained(other, keep)
        out1, lse1, _ = parity.run_gpu(other, plan=plan)
        assert torch.equal(out, out1) and torch.equal(lse, lse1)


@pytest.mark.gpu
@pytest.mark.parametrize("heads", [16, 64, 128])
def test_a_large_product_costs_only_its_own_64_dims(heads):
    """fp8: the matrix instruction aligns the products of 64 dims to the largest, also the one of 128 dims in
    the kernel for 32 rows: dim 0 carries a logit of 115 (166 in log2 units), dims 64 .. 127 all that differs.
    Bound on lse: 18 sums of up to 2^8, each rounded to 2^-17: 1.4e-4 in log2 units, 1e-4 in natural ones (seen:
    1.2e-5; dims 1 .. 63 in their place lose 1.5e-3)."""
    inp = make_custom(2, heads, [1024, 987], 0, 4096, seed=7, kv_dtype="fp8", q_std=0.5, kv_std=1.0)
    inp.q[..., :64] = 0
    inp.q[..., 128:] = 0
    inp.q[..., 0] = 200.0
    rows = inp.kv_cache.float()
    rows[..., 0] = 448.0
    inp.kv_cache = rows.to(inp.kv_cache.dtype)
    inp.kv_scales[...] = 8.0 / 448.0
    inp = parity.to_device(inp)
    out, lse, plan = parity.run_gpu(inp, out_dtype=torch.float32, num_splits_hint=1)
    assert plan.head_block == {16: 32}.get(heads, heads)
    e = parity.assert_parity(inp, out, lse, row_rel_l2=2e-2, what=f"{heads} heads")
    assert e["lse_abs"] <= 1e-4, e


@pytest.mark.gpu
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("heads", [32, 64, 128])
def test_reference_retry_in_every_kernel(kv, heads):
    """Logits that climb far above the first tile's maximum (131 in log2 units, the bound is 64) make a
    segment run twice; the latent values are spread, so that no 64-dim block holds one huge product."""
    L = 640
    inp = make_custom(2, heads, [L, L], 0, 4096, seed=4, kv_dtype=kv, q_std=0.0, kv_std=0.0)
    inp.q.zero_()
    inp.q[:, :, 512:] = 1.0
    rows = torch.zeros(L, 576)
    rows[:, 512:] = torch.linspace(0.0, 20.0, L)[:, None]
    rows[:, :512] = 0.25 * (torch.arange(L) % 5)[:, None]
    if kv == "fp8":
        rows, scales = quantize_fp8_per_token(rows)
    for b in range(2):
        for pg in range(L // 128):
            phys = int(inp.page_table[b, pg])
            inp.kv_cache[phys] = rows[pg * 128:(pg + 1) * 128].to(inp.kv_cache.dtype)
            if kv == "fp8":
                inp.kv_scales[phys] = scales[pg * 128:(pg + 1) * 128]
    inp = parity.to_device(inp)
    out, lse, plan = parity.run_gpu(inp, out_dtype=torch.float32, num_splits_hint=1)
    assert plan.head_block == {32: 32, 64: 64 if kv == "fp8" else 128, 128: 128}[heads]
    assert torch.isfinite(out).all() and torch.isfinite(lse).all()
    parity.assert_parity(inp, out, lse, what=f"retry, {heads} heads")


def test_blocks_of_64_rows_are_planned_for_an_fp8_cache():
    def block(batch, heads, window, kv):
        return oa.omniattn_plan_host([32768] * batch, batch=batch, num_heads=heads, max_pages_per_seq=256, num_pages=1 << 16,
                                     sink=128, window=window, softmax_scale=0.1, kv_dtype=kv).head_block
    assert block(128, 64, 2048, oa.FP8_E4M3) == 64 and block(32, 128, 8192, oa.FP8_E4M3) == 64
    assert block(256, 128, 1024, oa.FP8_E4M3) == 128 and block(4, 128, 2048, oa.FP8_E4M3) == 32
    assert block(64, 128, 2048, oa.BF16) == 128


@pytest.mark.parametrize("batch", [65, 100, 129, 200, 300])
def test_smaller_blocks_never_cost_the_static_scratch(batch):
    """Partial rows of a chosen plan fit the built-in buffer, or those of blocks of 128 rows would not either."""
    for kv in (oa.BF16, oa.FP8_E4M3):
        for out in (oa.BF16, oa.FP32):
            for heads in (16, 33, 64, 128):
                p = oa.omniattn_plan_host([30000 + 777 * (i % 13) for i in range(batch)], batch=batch, num_heads=heads,
                                          max_pages_per_seq=320, num_pages=1 << 16, sink=100, window=4096, softmax_scale=0.1,
                                          kv_dtype=kv, out_dtype=out)
                assert p.head_block == 128 or p.workspace_bytes <= oa.omniattn_static_scratch_bytes()


# Batches for which the planner takes decode_mid_kernel on a bf16 cache: one group of 64 rows, or two that share a block.
TILE_EDGES = [1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 160, 161, 192, 250, 333, 500, 650]


@pytest.mark.gpu
@pytest.mark.parametrize("heads, q_len, groups", [(128, 1, 2), (100, 1, 2), (64, 2, 2), (110, 2, 2), (85, 3, 2), (64, 1, 1), (33, 1, 1), (20, 2, 1)])
def test_groups_of_64_rows_over_a_bf16_cache(heads, q_len, groups):
    """Every tile count from none to twenty (fewer than the four stages, each stage reused), windows that open inside a
    tile, a second group of a few rows, queries that end inside a group; what is not kept has no influence."""
    lens = [0] + [max(L, q_len) for L in TILE_EDGES] * (4 if groups == 2 else 10)
    inp = make_custom(len(lens), heads * q_len, lens, 40, 600, seed=heads, kv_dtype="bf16", q_std=0.7, kv_std=0.7)
    inp = parity.to_device(inp)
    out, lse, plan = _run(inp, q_len, heads, out_dtype=torch.float32)
    assert plan.unit_groups == groups and plan.head_block == 64 * groups
    _check(inp, out, lse, q_len, f"{heads} heads, {q_len} queries")
    keep = [[j < L and (j < 40 or j >= L - 600 - (q_len - 1)) for j in range(-(-L // 128) * 128)] for L in lens]
    poison_unretained(inp, keep)
    again, lse2, _ = _run(inp, q_len, heads, out_dtype=torch.float32)
    assert torch.equal(out, again) and torch.equal(lse, lse2)
    out16, lse16, plan16 = _run(inp, q_len, heads)
    assert plan16.unit_groups == groups and plan16.head_block == 64 * groups
    if plan.num_partials == plan16.num_partials == 0:
        assert torch.equal(out.to(torch.bfloat16), out16) and torch.equal(lse, lse16)
    else:
        _check(inp, out16, lse16, q_len, f"{heads} heads, {q_len} queries, bf16 results")


@pytest.mark.gpu
@pytest.mark.parametrize("heads", [64, 128])
def test_reference_retry_with_groups_of_64_rows(heads):
    """As test_reference_retry_in_every_kernel, in a batch that runs on decode_mid_kernel with a bf16 cache."""
    B, L = 81, 640
    inp = make_custom(B, heads, [L] * B, 0, 4096, seed=4, kv_dtype="bf16", q_std=0.0, kv_std=0.0)
    inp.q.zero_()
    inp.q[:, :, 512:] = 1.0
    rows = torch.zeros(L, 576)
    rows[:, 512:] = torch.linspace(0.0, 20.0, L)[:, None]
    rows[:, :512] = 0.25 * (torch.arange(L) % 5)[:, None]
    for b in range(0, B, 2):                               # (every other sequence runs twice)
        for pg in range(L // 128):
            inp.kv_cache[int(inp.page_table[b, pg])] = rows[pg * 128:(pg + 1) * 128].to(inp.kv_cache.dtype)
    inp = parity.to_device(inp)
    out, lse, plan = parity.run_gpu(inp, out_dtype=torch.float32)
    assert plan.head_block // plan.unit_groups == 64
    assert torch.isfinite(out).all() and torch.isfinite(lse).all()
    parity.assert_parity(inp, out, lse, what=f"retry, {heads} heads")


def test_two_groups_to_a_block_where_a_sequence_would_be_cut_more():
    def plan(batch, heads, window, q_len=1):
        return oa.omniattn_plan_host([32768] * batch, batch=batch, num_heads=heads, max_pages_per_seq=256, num_pages=1 << 16,
                                     sink=128, window=window, softmax_scale=0.1, q_len=q_len)
    assert [plan(64, h, 2048).unit_groups for h in (64, 96, 128)] == [1, 2, 2] and plan(64, 128, 2048, 2).unit_groups == 2
    assert plan(64, 128, 2048).num_units == 128 and plan(64, 128, 2048, 2).num_partials == 0
    assert plan(256, 128, 4096).unit_groups == 1 and plan(64, 128, 2048, 4).unit_groups == 1


def _long_problem(kv, heads, lens, seed):
    """Sequences of tens of thousands of tokens, all kept, whose pages are drawn from a pool that they share."""
    pool, longest = 700, max(lens)
    inp = make_custom(len(lens), heads, [1] * len(lens), 0, longest, seed=seed, kv_dtype=kv, q_std=0.25, kv_std=0.7,
                      spare_pages=pool - len(lens))
    g = torch.Generator().manual_seed(seed)
    table = torch.stack([torch.randperm(pool, generator=g)[:-(-longest // 128)] for _ in lens]).to(torch.int32)
    return parity.to_device(dataclasses.replace(inp, page_table=table, seq_lens_host=lens, seq_lens=torch.tensor(lens, dtype=torch.int32)))


@pytest.mark.gpu
def test_segments_of_a_thousand_tiles_over_a_bf16_cache():
    """Segments of 64 rows and up to 1024 tiles, as many as a segment may have: two rounds of page-table entries to a
    thread, and every wave has some.  (One tile from another page shifts a row by 4 %.)"""
    lens = [32768 - 37 * (i % 5) for i in range(256)]
    inp = _long_problem("bf16", 64, lens, 5)
    out, lse, plan = parity.run_gpu(inp, out_dtype=torch.float32)
    sizes = [s["tile_hi"] - s["tile_lo"] for s in plan.segments()]
    assert plan.head_block == 64 and plan.num_partials == 0 and set(sizes) == {1020, 1021, 1022, 1023, 1024}
    rng = random.Random(1)
    pairs = [(b, rng.randrange(64)) for b in (0, 255, *(rng.randrange(256) for _ in range(22)))]
    parity.assert_parity(inp, out, lse, pairs=pairs, row_rel_l2=1e-2, what="bf16")


@pytest.mark.gpu
@pytest.mark.parametrize("heads", [64, 128])
def test_segments_of_a_thousand_tiles_over_an_fp8_cache(heads):
    """Whole sequences of up to 1024 tiles, also against the same ones in 16 pieces.  Both round the same weights; a piece is
    normalised by the sum of its rounded ones, which is within 2^-4 / sqrt(its tokens) < 2e-3 of the exact sum by which it is
    merged (20,000 tokens: 1,250 to a piece)."""
    lens = [65536, 40001, 33333, 65501, 20000]
    inp = _long_problem("fp8", heads, lens, 6)
    out, lse, plan = parity.run_gpu(inp, out_dtype=torch.float32, num_splits_hint=1)
    assert plan.head_block == heads and plan.head_block // plan.unit_groups == 64 and plan.num_partials == 0
    assert sorted(s["tile_hi"] - s["tile_lo"] for s in plan.segments()) == [313, 521, 626, 1024, 1024]
    rng = random.Random(2)
    pairs = [(b, rng.randrange(heads)) for b in range(5) for _ in range(4)]
    parity.assert_parity(inp, out, lse, pairs=pairs, row_rel_l2=2e-2, what=f"fp8, {heads} heads")
    cut, cut_lse, plan = parity.run_gpu(inp, out_dtype=torch.float32, num_splits_hint=16)
    assert plan.head_block == heads and plan.max_splits == 16
    rows = (out - cut).norm(dim=-1) / cut.norm(dim=-1)
    assert float(rows.max()) <= 4e-3 and float((lse - cut_lse).abs().max()) <= 1e-4, (float(rows.max()), float((lse - cut_lse).abs().max()))


@pytest.mark.gpu
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_segments_of_a_thousand_tiles_of_32_rows(kv):
    """One round of page-table entries to a thread, or two to four, and waves without any in the last.  (As above: one tile from
    another page shifts a row by 4 %; the rounding of the weights is that of the tests above.)"""
    tile = 32 if kv == "bf16" else 64
    lens = [tile * t - cut for t, cut in ((1024, 0), (769, 5), (513, 0), (257, tile - 1), (256, 0), (65, 1), (64, 0))]
    inp = _long_problem(kv, 16, lens, 8)
    out, lse, plan = parity.run_gpu(inp, out_dtype=torch.float32, num_splits_hint=1)
    assert plan.head_block == 32 and plan.num_partials == 0
    assert sorted(s["tile_hi"] - s["tile_lo"] for s in plan.segments()) == [64, 65, 256, 257, 513, 769, 1024]
    pairs = [(b, h) for b in range(len(lens)) for h in (b, 15)]
    parity.assert_parity(inp, out, lse, pairs=pairs, row_rel_l2=1e-2 if kv == "bf16" else 2e-2, what=kv)


@pytest.mark.gpu
@pytest.mark.parametrize("heads", [16, 64, 128])
def test_zero_softmax_scale_with_tiny_queries_over_an_fp8_cache(heads):
    """The scale taken times a query row's power of two is below the smallest float: masked positions stay masked."""
    inp = make_custom(3, heads, [333, 70, 5], 3, 100, seed=9, kv_dtype="fp8", q_std=1.0, kv_std=0.7, softmax_scale=0.0)
    inp.q = (inp.q.float() * 2.0 ** -60).to(torch.bfloat16)
    inp = parity.to_device(inp)
    out, lse, plan = parity.run_gpu(inp, out_dtype=torch.float32, num_splits_hint=1)
    assert plan.head_block == {16: 32}.get(heads, heads)
    parity.assert_parity(inp, out, lse, row_rel_l2=1e-2, what=f"{heads} heads")


@pytest.mark.gpu
@pytest.mark.parametrize("heads", [16, 64, 128])
@pytest.mark.parametrize("exponent", [-100, -118, -119, -120, -122, -126, -130])
def test_tiny_queries_over_an_fp8_cache(heads, exponent):
    """The power of two of a query row is kept to a normal number, and so is its reciprocal; at 2^-130 all elements are subnormal.
    Softmax scales of about one leave logits of zero to single precision: lse is the logarithm of the kept tokens, the output
    the mean of their values.  Scales of 0.1 over the queries' size, of both signs, give the logits of ordinary queries."""
    for scale in (1.0, -0.5, 0.1 * 2.0 ** -exponent, -0.1 * 2.0 ** -exponent):
        inp = make_custom(3, heads, [333, 70, 5], 3, 100, seed=9, kv_dtype="fp8", q_std=1.0, kv_std=0.7, softmax_scale=scale)
        inp.q = (inp.q.float() * 2.0 ** exponent).to(torch.bfloat16)
        inp = parity.to_device(inp)
        out, lse, plan = parity.run_gpu(inp, out_dtype=torch.float32, num_splits_hint=1)
        assert plan.head_block == {16: 32}.get(heads, heads)
        parity.assert_parity(inp, out, lse, row_rel_l2=1e-2, what=f"{heads} heads, 2^{exponent}, scale {scale}")


@pytest.mark.gpu
@pytest.mark.parametrize("heads", [16, 64, 128])
@pytest.mark.parametrize("scale", [2.0 ** -124, -2.0 ** -124])
def test_tiny_softmax_scales_with_huge_rows_over_an_fp8_cache(heads, scale):
    """The softmax scale times a query row's power of two is subnormal, and raw products of up to 2^126 make logits of it."""
    inp = make_custom(3, heads, [333, 70, 5], 3, 100, seed=9, kv_dtype="fp8", q_std=1.0, kv_std=0.7, softmax_scale=scale)
    inp.kv_scales = inp.kv_scales * 2.0 ** 113
    inp = parity.to_device(inp)
    out, lse, plan = parity.run_gpu(inp, out_dtype=torch.float32, num_splits_hint=1)
    assert plan.head_block == {16: 32}.get(heads, heads)
    parity.assert_parity(inp, out, lse, row_rel_l2=1e-2, what=f"{heads} heads, scale {scale}")


def _rows_of_a_group(kv, heads):
    """Of the kernels that 81 sequences of 640 tokens run on, as the planner has it and one work unit per sequence."""
    return {("bf16", 64): {64, 128}, ("bf16", 128): {64, 128}, ("fp8", 64): {32, 64}, ("fp8", 128): {64}}.get((kv, heads), {32})


@pytest.mark.gpu
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("heads", [16, 64, 128])
def test_zero_softmax_scale_with_huge_rows(kv, heads):
    """All kept tokens weigh the same however large their products with the query are; masked positions stay masked."""
    lens = [333, 70, 5] + [640] * 78
    inp = make_custom(81, heads, lens, 3, 600, seed=9, kv_dtype=kv, q_std=1.0, kv_std=0.7, softmax_scale=0.0)
    if kv == "fp8":
        inp.kv_scales = inp.kv_scales * 2.0 ** 110
    else:
        inp.kv_cache = inp.kv_cache * 2.0 ** 110
    inp = parity.to_device(inp)
    rows = set()
    for hint in (0, 1):
        out, lse, plan = parity.run_gpu(inp, num_splits_hint=hint)
        rows.add(plan.head_block // plan.unit_groups)
        parity.assert_parity(inp, out, lse, row_rel_l2=1e-2, what=f"{kv}, {heads} heads, hint {hint}")
    assert rows == _rows_of_a_group(kv, heads)


@pytest.mark.gpu
@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("heads", [16, 64, 128])
def test_a_query_element_that_is_no_number(kv, heads):
    """NaN or an infinity in one element, the lower and the upper one of a word, of the value and the rope part, beside numbers:
    that row is NaN, all others are the same bits as without it.  (fp8 cache: the row's largest element passes over it.)"""
    lens = [333, 70, 200] + [640] * 78
    inp = parity.to_device(make_custom(81, heads, lens, 3, 600, seed=9, kv_dtype=kv, q_std=1.0, kv_std=0.7))
    q, bad, rows = inp.q, (1, heads // 2 + 1), set()
    for hint in (0, 1, 4):
        inp.q = q
        out0, lse0, plan = parity.run_gpu(inp, num_splits_hint=hint)
        rows.add(plan.head_block // plan.unit_groups)
        for value in (float("nan"), float("inf"), float("-inf")):
            for dim in (16, 17, 511, 512, 575):
                inp.q = q.clone()
                inp.q[bad + (dim,)] = value
                out, lse, _ = parity.run_gpu(inp, plan=plan)
                assert torch.isnan(out[bad]).all() and torch.isnan(lse[bad]), (hint, value, dim)
                out[bad], lse[bad] = out0[bad], lse0[bad]
                assert torch.equal(out, out0) and torch.equal(lse, lse0), (hint, value, dim)
    assert rows == _rows_of_a_group(kv, heads)
