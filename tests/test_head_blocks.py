"""The kernels for blocks of 32 head rows and for full head blocks on the same short, ragged problems: no
tile, one, two or three tiles (fewer than are requested ahead), ragged ends, windows that open inside a
tile, several segments per unit, several queries per sequence, rows past the last head."""
import pytest
import torch

import parity
from test_multi_query import _check, _run
from workloads import make_custom


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
@pytest.mark.parametrize("heads, q_len", [(33, 1), (64, 1), (128, 1), (40, 2)])
def test_full_blocks(kv, heads, q_len):
    for sink, window in ((3, 40), (64, 512), (0, 4096)):
        inp = _problem(kv, heads, q_len, sink, window)
        out, lse, plan = _run(inp, q_len, heads, num_splits_hint=1)
        assert plan.head_block == 128
        _check(inp, out, lse, q_len, f"{heads} heads, {sink}/{window}")
