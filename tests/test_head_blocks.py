"""The kernels for blocks of 32, 64 and 128 head rows on the same short, ragged problems: no
tile, one, two or three tiles (fewer than are requested ahead), ragged ends, windows that open inside a
tile, several segments per unit, several queries per sequence, rows past the last head."""
import pytest
import torch

import paper_2511_22481_amd as oa
import parity
from test_multi_query import _check, _run
from workloads import make_custom
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
