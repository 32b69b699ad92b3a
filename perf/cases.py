"""Decode work that a user of this library has it do, for timing and for comparing results.

Shapes are the DeepSeek-R1 absorbed-MLA decode of `workloads/configs.py` (rows of 512 + 64
numbers, 128-token pages in shuffled order, sink / window pairs of 64/512 up to 128/8192) and
what surrounds it in a serving program: one rank of a head-sharded model, a single interactive
sequence, a whole decode step on the physically compressed ring cache, the one-call wrapper.

Kinds of call (`op`):
  decode   omniattn_decode with the plan, the workspace and the output buffers a serving loop keeps;
  step     one decode step of a serving loop on a ring cache: the lengths are set (a verification
           step that rejects drafts rolls them back), q_len tokens are appended, the plan is
           refreshed for the new lengths, decode;
  oneshot  the wrapper `decode`, which plans and allocates by itself.
"""
import random

import torch

import paper_2511_22481_amd as oa

PAGE, QK, V = 128, 576, 512
SCALE = 192.0 ** -0.5


def _case(op, batch, heads, len_lo, len_hi, sink, window, kv="bf16", out="bf16", q_len=1, **kw):
    return dict(kw, op=op, batch=batch, heads=heads, len_lo=len_lo, len_hi=len_hi, sink=sink, window=window,
                kv=kv, out=out, q_len=q_len)


def listed():
    return [
        # the smallest configuration: launches and latency
        _case("decode", 4, 16, 2048, 2048, 64, 512, name="tiny_b4_h16"),
        # one interactive sequence: a single user's latency, nothing to batch with
        _case("decode", 1, 128, 20011, 20011, 128, 2048, name="single_b1_20k"),
        # the headline decode
        _case("decode", 64, 128, 32768, 32768, 128, 2048, name="r1_b64_32k"),
        # mixed lengths of a large serving batch
        _case("decode", 256, 128, 1024, 65536, 128, 4096, name="mixed_b256"),
        # sequences still shorter than the window: everything is kept
        _case("decode", 32, 128, 4096, 4096, 128, 8192, name="dense_b32_4k"),
        # a layer that the pattern search leaves uncompressed
        _case("decode", 64, 128, 32768, 32768, 0, 32768, name="r1_b64_32k_dense"),
        # long context, fp8 cache
        _case("decode", 32, 128, 131072, 131072, 128, 8192, kv="fp8", name="fp8_b32_128k"),
        # fp8 cache, mixed lengths, odd batch
        _case("decode", 93, 128, 1024, 65536, 128, 4096, kv="fp8", name="fp8_mixed_b93"),
        # one of eight head-sharded ranks: 16 heads read the whole latent cache
        _case("decode", 128, 16, 1024, 32768, 128, 2048, name="tp8_b128_h16"),
        # a serving step on the ring cache with one draft token per sequence to verify (two queries)
        _case("step", 64, 128, 3000, 30000, 128, 2048, q_len=2, name="step_mtp_b64"),
        # a serving step on an fp8 ring cache, ragged lengths, some below the window
        _case("step", 40, 128, 700, 30000, 64, 1024, kv="fp8", name="step_fp8_b40"),
        # the one-call wrapper on a few ragged sequences, fp32 results (offline evaluation)
        _case("oneshot", 3, 48, 500, 6000, 100, 1000, out="fp32", name="oneshot_b3_h48"),
    ]


# kept tokens times query rows of a pass, and cached tokens of a state: no case is larger
_MOST_WORK = 64 * 32768 * 128
_MOST_CACHED = 8_600_000


def _log_int(rng, lo, hi):
    return min(hi, max(lo, round(lo * (hi / lo) ** rng.random())))


def draw(rng):
    op = rng.choice(["decode", "decode", "decode", "decode", "step", "step", "oneshot"])
    kv = rng.choice(["bf16", "bf16", "fp8"])
    if op == "decode":
        batch, heads = _log_int(rng, 1, 256), rng.choice([16, 32, 64, 128, 128, 128])
        sink = rng.choice([0, 4, 64, 128, 128, 130])
        window = _log_int(rng, 512, 32768)
        hi = _log_int(rng, 1024, 131072)
        lo = hi if rng.random() < 0.3 else _log_int(rng, 512, hi)
        q_len = rng.choice([1, 1, 1, 2, 4])
        out = rng.choice(["bf16", "bf16", "bf16", "fp32"])
    elif op == "step":
        batch, heads = _log_int(rng, 4, 256), rng.choice([16, 32, 64, 128, 128])
        sink, window = rng.choice([0, 4, 64, 128]), _log_int(rng, 512, 8192)
        hi = _log_int(rng, 2048, 65536)
        lo = _log_int(rng, 600, hi)
        q_len, out = rng.choice([1, 1, 2, 3]), "bf16"
    else:
        batch, heads = _log_int(rng, 1, 8), rng.choice([16, 48, 128])
        sink, window = rng.choice([0, 64, 100]), _log_int(rng, 128, 8192)
        hi = _log_int(rng, 600, 16384)
        lo = _log_int(rng, 300, hi)
        q_len, out = 1, rng.choice(["bf16", "fp32"])
    while True:
        case = _case(op, batch, heads, lo, hi, sink, window, kv=kv, out=out, q_len=q_len)
        lens = _lens(case)
        work = _kept(case, lens) * max(128, heads * q_len)  # few heads: the cache rows are what costs
        if batch == 1 or (work <= _MOST_WORK and sum(lens) <= _MOST_CACHED):
            return case
        batch = max(1, batch * 3 // 4)


def _lens(case):
    """Lengths that the decode sees; a matter of the case, not of the seed: the work is the same for every seed."""
    lo, hi = case["len_lo"], case["len_hi"]
    rng = random.Random(lo * 1_000_003 + hi * 101 + case["batch"])
    return [lo if lo == hi else rng.randint(lo, hi) for _ in range(case["batch"])]


def _kept(case, lens, q_len=None):
    """Kept positions of all sequences (several queries: of the union of their kept sets)."""
    w = case["window"] + (case["q_len"] if q_len is None else q_len) - 1
    return sum(min(L, case["sink"] + w) for L in lens)


def _fill(shape, fp8, device, gen):
    """Latent rows are RMS-normed by the model: unit variance.  fp8: one scale per row, its largest value at 448."""
    pages = shape[0]
    rows = torch.empty(shape, dtype=torch.float8_e4m3fn if fp8 else torch.bfloat16, device=device)
    scales = torch.empty(shape[:-1], dtype=torch.float32, device=device) if fp8 else None
    for a in range(0, pages, 4096):
        x = torch.randn((min(4096, pages - a),) + tuple(shape[1:]), device=device, generator=gen)
        if fp8:
            s = x.abs().amax(dim=-1) / 448.0
            x.div_(s.unsqueeze(-1))
            scales[a:a + 4096] = s
        rows[a:a + 4096] = x.to(rows.dtype)
    return rows, scales


def prepare(case, seed):
    device = torch.device("cuda")
    gen = torch.Generator(device=device).manual_seed(int(seed))
    B, H, T, S, W = case["batch"], case["heads"], case["q_len"], case["sink"], case["window"]
    fp8 = case["kv"] == "fp8"
    lens = _lens(case)
    most = max(-(-L // PAGE) for L in lens)
    st = dict(op=case["op"], sink=S, window=W, q_len=T, lens=lens)

    table = torch.full((B, most), -1, dtype=torch.int32)
    if case["op"] == "step":
        # every sequence owns the pages of its ring; the table maps the kept logical pages to them
        per = oa.omniattn_ring_pages(S, W, q_len=T)
        pages = B * per
        own = torch.randperm(pages, generator=gen, device=device).to(torch.int32).reshape(B, per)
        own_host = own.cpu()
        for b, L in enumerate(lens):
            last = -(-(L - T) // PAGE)  # pages opened before this step's tokens
            for lp in sorted(set(range(min(-(-S // PAGE), last))) | set(range(max(0, (L - T - W) // PAGE), last))):
                table[b, lp] = own_host[b, oa.omniattn_ring_slot(S, W, lp, q_len=T)]
        st["seq_pages"] = own
        st["lens_before"] = torch.tensor([L - T for L in lens], dtype=torch.int32, device=device)
        st["seq_lens"] = st["lens_before"].clone()
        st["new_rows"], st["new_scales"] = _fill((T, B, QK), fp8, device, gen)
    else:
        counts = [-(-L // PAGE) for L in lens]
        pages = sum(counts)
        order = torch.randperm(pages, generator=gen, device=device).to(torch.int32).cpu()
        at = 0
        for b, n in enumerate(counts):
            table[b, :n] = order[at:at + n]
            at += n
    st["kv"], st["scales"] = _fill((pages, PAGE, QK), fp8, device, gen)
    st["table"] = table.to(device)
    # unit-variance queries: logits of standard deviation 1.7
    st["q"] = torch.randn((B, T, H, QK) if T > 1 else (B, H, QK), device=device, generator=gen).to(torch.bfloat16)
    st["out_dtype"] = torch.float32 if case["out"] == "fp32" else torch.bfloat16
    if case["op"] == "oneshot":
        return st
    st["plan"] = oa.omniattn_plan(lens, batch=B, num_heads=H, max_pages_per_seq=most, num_pages=pages, sink=S,
                                  window=W, softmax_scale=SCALE, kv_dtype=oa.FP8_E4M3 if fp8 else oa.BF16,
                                  out_dtype=oa.FP32 if case["out"] == "fp32" else oa.BF16,
                                  q_len=T if T > 1 else 0)
    lead = tuple(st["q"].shape[:-1])
    st["out"] = torch.empty(lead + (V,), dtype=st["out_dtype"], device=device)
    st["lse"] = torch.empty(lead, dtype=torch.float32, device=device)
    need = st["plan"].workspace_bytes
    st["workspace"] = torch.empty(need, dtype=torch.uint8, device=device) if need else None
    return st


def run(st):
    if st["op"] == "oneshot":
        out, lse, _ = oa.decode(st["q"], st["kv"], st["scales"], st["table"], st["lens"], st["sink"], st["window"],
                                SCALE, out_dtype=st["out_dtype"])
        return {"out": out, "lse": lse}
    if st["op"] == "step":
        st["seq_lens"].copy_(st["lens_before"])
        for t in range(st["q_len"]):
            oa.omniattn_ring_append(st["seq_lens"], st["new_rows"][t],
                                    None if st["new_scales"] is None else st["new_scales"][t], st["seq_pages"],
                                    st["kv"], st["scales"], st["table"], sink=st["sink"], window=st["window"],
                                    q_len=st["q_len"])
        oa.omniattn_plan_update(st["plan"], st["lens"])
    oa.omniattn_decode(st["plan"], st["q"], st["kv"], st["scales"], st["table"], st["out"], st["lse"],
                       st["workspace"])
    r = {"out": st["out"], "lse": st["lse"]}
    if st["op"] == "step":
        r.update(seq_lens=st["seq_lens"], table=st["table"], kv=st["kv"])
        if st["scales"] is not None:
            r["scales"] = st["scales"]
    return r


def work(case):
    lens = _lens(case)
    B, H, T = case["batch"], case["heads"], case["q_len"]
    row = QK + 4 if case["kv"] == "fp8" else 2 * QK
    rows = B * T * H
    moved = _kept(case, lens) * row + rows * (2 * QK + V * (4 if case["out"] == "fp32" else 2) + 4)
    if case["op"] == "step":
        moved += 2 * B * T * row
    flops = sum(2 * (QK + V) * H * _kept(case, [L - (T - 1 - t) for L in lens], q_len=1) for t in range(T))
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    # Measured against 64-bit sums.  bf16 cache (weights and results rounded to bf16, 2^-9 each): 2.7e-3
    # over all values, 1.7e-2 of the root mean square for the worst value.  fp8 cache (weights rounded
    # to e4m3, at most 2^-4 each): 1.8e-2 over all values, 0.21 for the worst; two correct results
    # that round differently are apart by 1.4 times that.
    return {"rel": 0.03, "max": 0.5} if case["kv"] == "fp8" else {"rel": 0.01, "max": 0.08}
