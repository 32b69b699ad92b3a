"""The work partition's three shapes, and the merge of few and many partial rows per sequence
(up to 8 partials one wave takes a head row, from 9 on four waves share it)."""
import pytest
import torch

import paper_2511_22481_amd as oa
import parity
from test_abi_and_plan import check_plan
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
