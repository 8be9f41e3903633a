"""The calls whose speed is followed: paged decode and speculative-verify
attention, lossless acceptance and a whole speculative step, each through the
package's ctypes binding as a rollout replica calls it.

A case is a dict of plain values.  Context lengths and draft lengths are part
of the case (drawn from its ``len_seed``), so its work is known without a GPU;
the values of q, K, V and the probabilities, the page permutation, the drafts
and the uniforms come from the seed of ``prepare``.
"""
import math
import random

import torch

from paper_2608_22788_amd import binding

PAGE = 16
VOCAB = 151936              # the vocabulary of the package's step benchmark
MAX_KV_BYTES = 1.6e9        # of a drawn case: below the largest listed one at any head shape


def _attn(name, batch, q_len, q_heads, kv_heads, head_dim, lengths, lo=0, hi=0, ragged=False, len_seed=0):
    return dict(name=name, kind="attn", batch=batch, q_len=q_len, q_heads=q_heads, kv_heads=kv_heads,
                head_dim=head_dim, lengths=lengths, lo=lo, hi=hi, ragged=ragged, len_seed=len_seed)


def listed():
    step = _attn("spec_step_b8", 8, 4, 32, 8, 128, "pareto", len_seed=12)
    step.update(kind="step", drafts=3, vocab=VOCAB)
    return [
        # the last straggler of a rollout step, one token at a time: latency only
        _attn("decode_b1", 1, 1, 32, 8, 128, "pareto", len_seed=1),
        # a small tail pool verifying three drafts per sequence
        _attn("verify_b4_q4", 4, 4, 32, 8, 128, "pareto", len_seed=2),
        # a replica that is draining: fewer sequences than fill the chip well
        _attn("decode_b32", 32, 1, 32, 8, 128, "pareto", len_seed=3),
        # the bulk pool at full concurrency
        _attn("decode_bulk_b256", 256, 1, 32, 8, 128, "lognormal", len_seed=4),
        # the tail pool: long contexts, multi-token-prediction drafts
        _attn("verify_mtp_b8_q4", 8, 4, 32, 8, 128, "uniform", 16384, 65536, len_seed=5),
        # the tail pool with a block drafter of 15 drafts
        _attn("verify_block_b4_q16", 4, 16, 32, 8, 128, "uniform", 32768, 98304, len_seed=6),
        # one launch for sequences with different draft depths, some decoding plainly
        _attn("mixed_b64_q6", 64, 6, 32, 8, 128, "pareto", ragged=True, len_seed=7),
        # a model with eight query heads per KV head verifying at bulk concurrency
        _attn("verify_g8_b256_q4", 256, 4, 32, 4, 128, "lognormal", len_seed=8),
        # the small head shape (head_dim 64)
        _attn("decode_d64_b64", 64, 1, 8, 2, 64, "lognormal", len_seed=9),
        # acceptance after verify, tail pool and bulk pool
        dict(name="accept_b8", kind="accept", batch=8, drafts=3, vocab=VOCAB),
        dict(name="accept_b128", kind="accept", batch=128, drafts=3, vocab=VOCAB),
        # one speculative step of a small tail pool: append, verify, accept
        step,
    ]


def draw(rng):
    kind = rng.choice(["attn"] * 7 + ["accept"] * 2 + ["step"])
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
    if kind == "accept":
        return dict(kind=kind, batch=log(1, 128), drafts=rng.choice([1, 2, 3, 5, 7]),
                    vocab=rng.choice([VOCAB, log(32000, VOCAB), 4 * log(8000, 37000)]))
    q_heads, kv_heads, head_dim = rng.choice(
        [(32, 8, 128)] * 4 + [(16, 4, 128), (32, 4, 128), (64, 4, 128), (8, 2, 64), (16, 2, 64)])
    q_len = rng.choice([1, 1, 1, 2, 3, 4, 4, 5, 6, 16])
    q_len = min(q_len, 64 // (q_heads // kv_heads))
    lengths = rng.choice(["pareto", "pareto", "lognormal", "uniform"])
    lo = log(64, 40000)
    c = _attn("", log(1, 16 if lengths == "uniform" else 256), q_len, q_heads, kv_heads, head_dim, lengths, lo,
              lo * rng.choice([1, 2, 3]), q_len > 1 and rng.random() < 0.3, rng.randrange(1 << 30))
    del c["name"]
    if kind == "step":
        c.update(kind=kind, batch=min(c["batch"], 24), lengths="pareto", ragged=False, q_len=max(2, min(q_len, 6)))
        c.update(drafts=c["q_len"] - 1, vocab=VOCAB)
    while c["batch"] > 1 and _kv_bytes(c) > MAX_KV_BYTES:
        c["batch"] = c["batch"] * 3 // 4
    return c


# ---- shapes ---------------------------------------------------------------------

def _lens(case):
    """Context length (the new tokens included) and new tokens per sequence."""
    r = random.Random(case["len_seed"])
    ctx, ql = [], []
    for _ in range(case["batch"]):
        if case["lengths"] == "pareto":        # prompt plus a heavy-tailed response
            n = 512 + min(int(1024.0 * (1.0 - r.random()) ** (-1.0 / 1.5)), 65536)
        elif case["lengths"] == "lognormal":   # the bulk pool's snapshot
            n = r.randint(256, 1024) + min(int(round(2048.0 * math.exp(0.8 * r.gauss(0.0, 1.0)))), 16384)
        else:
            n = r.randint(case["lo"], case["hi"])
        ctx.append(n)
        ql.append(r.randint(1, case["q_len"]) if case["ragged"] else case["q_len"])
    return ctx, ql


def _kv_bytes(case):
    return sum(_lens(case)[0]) * case["kv_heads"] * case["head_dim"] * 4


def _attn_work(case):
    ctx, ql = _lens(case)
    row = case["q_heads"] * case["head_dim"]
    visible = sum(q * (n - q) + q * (q + 1) // 2 for n, q in zip(ctx, ql))
    return dict(bytes=_kv_bytes(case) + sum(ql) * row * 4 + sum((n + PAGE - 1) // PAGE for n in ctx) * 4 +
                8 * case["batch"],
                flops=4 * row * visible)


def _accept_work(case):
    # a rejection reads one row of the target and one of the drafter
    n = case["batch"] * case["vocab"]
    return dict(bytes=8 * n, flops=2 * n)


def work(case):
    if case["kind"] == "attn":
        return _attn_work(case)
    if case["kind"] == "accept":
        return _accept_work(case)
    a, b = _attn_work(case), _accept_work(case)
    new = case["batch"] * case["q_len"] * case["kv_heads"] * case["head_dim"] * 2 * 2   # K and V rows, bf16
    return dict(bytes=a["bytes"] + b["bytes"] + 2 * new, flops=a["flops"] + b["flops"])


# ---- inputs ---------------------------------------------------------------------

def _attn_inputs(case, gen):
    ctx, ql = _lens(case)
    B, Hkv, D = case["batch"], case["kv_heads"], case["head_dim"]
    npg = [(n + PAGE - 1) // PAGE for n in ctx]
    total = sum(npg)
    perm = torch.randperm(total, generator=gen, device="cuda").to(torch.int32)
    table = torch.zeros(B, max(npg), dtype=torch.int32, device="cuda")
    off = 0
    for b, n in enumerate(npg):
        table[b, :n] = perm[off:off + n]
        off += n
    normal = lambda *shape: torch.empty(*shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)  # noqa: E731
    i32 = lambda a: torch.tensor(a, dtype=torch.int32, device="cuda")  # noqa: E731
    return dict(q=normal(B, case["q_len"], case["q_heads"], D), k=normal(total, Hkv, PAGE, D),
                v=normal(total, Hkv, PAGE, D), table=table, ctx=i32(ctx), ql=i32(ql), max_ctx=max(ctx),
                scale=1.0 / math.sqrt(D))


def _accept_inputs(case, gen):
    """Target and drafter distributions over the vocabulary (the drafter's
    logits are the target's with noise), drafts drawn from the drafter."""
    B, G, V = case["batch"], case["drafts"], case["vocab"]
    logits = torch.empty(B, G + 1, V, dtype=torch.float32, device="cuda").normal_(generator=gen) * 2.0
    noise = torch.empty(B, G, V, dtype=torch.float32, device="cuda").normal_(generator=gen) * 0.7
    p = torch.softmax(logits, -1)
    q = torch.softmax(logits[:, :G] + noise, -1)
    race = noise.exponential_(generator=gen)
    drafts = (q / race).argmax(-1).to(torch.int32)
    uniform = lambda *shape: torch.rand(*shape, generator=gen, device="cuda")  # noqa: E731
    return dict(p=p, q_draft=q, drafts=drafts, num=torch.full((B,), G, dtype=torch.int32, device="cuda"),
                ua=uniform(B, G), us=uniform(B))


def _inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    s = {}
    if case["kind"] != "accept":
        s.update(_attn_inputs(case, gen))
    if case["kind"] == "step":
        shape = (case["batch"], case["q_len"], case["kv_heads"], case["head_dim"])
        s["k_new"], s["v_new"] = (torch.empty(*shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
                                  for _ in range(2))
    if case["kind"] != "attn":
        s.update(_accept_inputs(case, gen))
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["kind"] = case["kind"]
    if case["kind"] != "accept":
        s["out"] = torch.zeros_like(s["q"])
        shape = binding.shape_of(s["q"], s["k"], s["table"], s["max_ctx"])
        s["ws"] = binding.new_workspace(binding.workspace_size(shape))
    if case["kind"] != "attn":
        B = case["batch"]
        s["accepted"] = torch.zeros(B, dtype=torch.int32, device="cuda")
        s["token"] = torch.zeros(B, dtype=torch.int32, device="cuda")
        s["accept_ws"] = torch.empty(int(binding.lib.ts_spec_accept_workspace_size(B, case["vocab"])),
                                     dtype=torch.uint8, device="cuda")
    return s


def run(s):
    if s["kind"] == "step":
        binding.kv_append(s["k_new"], s["v_new"], s["k"], s["v"], s["table"], s["ctx"], s["ql"])
    if s["kind"] != "accept":
        binding.decode_attn(s["q"], s["k"], s["v"], s["table"], s["ctx"], s["ql"], s["out"], s["scale"],
                            workspace=s["ws"], max_ctx_len=s["max_ctx"])
    if s["kind"] == "attn":
        return s["out"]
    binding.spec_accept(s["p"], s["q_draft"], s["drafts"], s["num"], s["ua"], s["us"], s["accepted"], s["token"],
                        workspace=s["accept_ws"])
    if s["kind"] == "accept":
        return s["accepted"], s["token"]
    return s["k"], s["v"], s["out"], s["accepted"], s["token"]


# ---- expected results -----------------------------------------------------------

def tolerance(case):
    if case["kind"] == "accept":
        return "exact"      # the rule is evaluated without rounding
    # bf16 outputs from bf16 probabilities: two correct kernels differ by the
    # rounding of either; the present one is 2.1e-3 to 2.4e-3 from float64 over
    # the cases, 0.016 at the worst element
    return {"rel": 1e-2, "max": 0.07}


def exact(case, seed):
    if case["kind"] == "accept":
        return None         # whole numbers
    s = _inputs(case, seed)
    ctx, ql = _lens(case)
    Hkv, D = case["kv_heads"], case["head_dim"]
    G = case["q_heads"] // Hkv
    out = torch.zeros(s["q"].shape, dtype=torch.float64, device="cuda")
    if case["kind"] == "step":
        for b in range(case["batch"]):
            for i in range(ql[b]):
                t = ctx[b] - ql[b] + i
                page = int(s["table"][b, t // PAGE])
                s["k"][page, :, t % PAGE] = s["k_new"][b, i]
                s["v"][page, :, t % PAGE] = s["v_new"][b, i]
    for b, (n, Q) in enumerate(zip(ctx, ql)):
        pages = s["table"][b, :(n + PAGE - 1) // PAGE].long()
        rows = lambda x: x[pages].transpose(0, 1).reshape(Hkv, -1, D)[:, :n].double()  # noqa: E731
        q = s["q"][b, :Q].double().view(Q, Hkv, G, D).permute(1, 0, 2, 3).reshape(Hkv, Q * G, D)
        sc = torch.matmul(q, rows(s["k"]).transpose(1, 2).contiguous()) * s["scale"]
        pos = torch.arange(n, device="cuda")[None, :]
        last = (n - Q + torch.arange(Q, device="cuda")).repeat_interleave(G)[:, None]
        w = torch.softmax(sc.masked_fill(pos > last, -math.inf), -1)
        o = torch.matmul(w, rows(s["v"]).contiguous())
        out[b, :Q] = o.view(Hkv, Q, G, D).permute(1, 0, 2, 3).reshape(Q, Hkv * G, D)
    if case["kind"] == "attn":
        return out
    return s["k"].double(), s["v"].double(), out, None, None
