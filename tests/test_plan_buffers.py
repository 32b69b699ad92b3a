"""Plans that come and go: the buffers of a destroyed plan serve the next one, also while another stream
still decodes with the destroyed plan's copy."""
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
