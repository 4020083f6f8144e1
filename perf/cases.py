"""The work that a serving program has this library do, as timed cases.

A program that decodes with entropic time owns the logits, the queries and the paged cache,
and calls the library once per decode step: ent_decode_step_append in its loop (no
diagnostics asked for), or ent_decode_step where it wants the scores, thresholds and
log-sum-exps too.  Around the steps it forms the block summaries of new prompts
(ent_block_summary), picks the next batch (ent_schedule), and for requests without a paged
cache only runs the controller and the sampler (ent_entropy_temperature, ent_sample).

Sizes are those of the benchmark's workloads (an 8B-shaped step, a 70B-shaped loop, long
contexts, a skewed batch, the fp32 `tiny` shape) and generic smaller and odd ones.  Context
lengths and logit scales of a case are fixed sets of values, dealt to the sequences in an
order that the seed draws, so a case's work does not depend on the seed.

Every pass of a step is the same step: the controller state and the lengths, which a step
updates in place, have a copy of their own for each of SLOTS passes.  An appended token is
written to the same cache slot each time.
"""
from __future__ import annotations

import math

import torch

from paper_2603_03310_amd import ent
from paper_2603_03310_amd.runner import make_config

SLOTS = 4096
ROOM = 64            # tokens of room that a loop's block tables have past the longest context
ETA, T_MIN, T_MAX, H_TARGET, KAPPA_MIN, B_MIN = -0.05, 0.05, 5.0, 2.5, 0.05, 4
T_CAL, RHO_T, DKAPPA, KAPPA_PREV = 1.0, 0.05, 0.05, 0.5   # the guards, where a case has them on
ZIPF = 1.2
PRM = (1.0, 0.25, 4.0, 16.0, 0.5, 1e-3, 0.25)   # scheduler: alpha, beta, gamma, slo, floors, rate

STEP = dict(kind="step", batch=64, q_heads=32, kv_heads=8, head_dim=128, dtype="bf16",
            vocab=128256, ctx="uniform", lo=2048, hi=8192, logits="normal", s_lo=0.5, s_hi=4.0,
            settled=False, estimator="exact", est_k=256, guards=False, scoring="meankey",
            keep_first=0, keep_last=0)


def listed():
    return [
        # The smallest step: fp32 caches, a small vocabulary, as in bring-up and debugging.
        dict(STEP, name="tiny_fp32", batch=4, q_heads=8, kv_heads=8, head_dim=64, dtype="f32",
             vocab=1024, lo=128, hi=512),
        # One interactive request: latency of the whole loop step.
        dict(STEP, name="single_request", kind="loop", batch=1, lo=2500, hi=2500, s_lo=2.0,
             s_hi=2.0, settled=True),
        # A few requests at a time, ragged and short.
        dict(STEP, name="small_batch", kind="loop", batch=9, lo=301, hi=4001, s_lo=0.3, s_hi=5.0,
             settled=True),
        # The 8B-shaped decode step, the first after prompts (temperature 1, most blocks kept).
        dict(STEP, name="step_8b"),
        # The 70B-shaped loop with the temperatures the controller settles at (about a
        # sixth of the blocks kept).
        dict(STEP, name="loop_70b", kind="loop", batch=128, q_heads=64, lo=4096, hi=16384,
             s_lo=0.3, s_hi=5.0, settled=True),
        # Long documents.
        dict(STEP, name="long_context", batch=16, lo=32768, hi=131072),
        # Many requests of very unequal lengths, peaked and flat next-token distributions.
        dict(STEP, name="skewed_batch", batch=256, ctx="lognormal", lo=64, hi=32768,
             logits="mixed", s_lo=0.3, s_hi=0.3),
        # The conservative mode: scores from every key, the first and last blocks kept.
        dict(STEP, name="exact_scoring", scoring="exact", keep_first=1, keep_last=2),
        # Controller on the tail-corrected estimate, with the rate guards on.
        dict(STEP, name="tail_estimate", estimator="tail", guards=True),
        # Block summaries of a batch of new prompts.
        dict(STEP, name="prompt_summaries", kind="summary"),
        # Controller and sampler alone; an odd vocabulary, so rows are not 16-byte aligned.
        dict(kind="sample", name="sampler_only", batch=64, vocab=50257, logits="normal",
             s_lo=0.5, s_hi=4.0, settled=False),
        # The next batch out of a full pool.
        dict(kind="schedule", name="schedule_pool", pool=8192, b_sel=64),
    ]


def _between(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "step", "loop", "loop", "step_f32", "exact", "estimate", "summary",
                       "sample", "schedule"])
    if kind == "schedule":
        n = _between(rng, 64, 8192)
        return dict(kind="schedule", pool=n, b_sel=_between(rng, 1, max(1, n // 4)))
    vocab = rng.choice([32000, 50257, 128256, _between(rng, 8000, 150000)])
    if kind == "sample":
        return dict(kind="sample", batch=_between(rng, 1, 256), vocab=vocab, logits="normal",
                    s_lo=0.5, s_hi=4.0, settled=rng.random() < 0.5)
    c = dict(STEP, vocab=vocab, kind=kind if kind in ("loop", "summary") else "step")
    c["q_heads"], c["kv_heads"], c["head_dim"] = rng.choice(
        [(32, 8, 128), (32, 8, 128), (64, 8, 128), (16, 4, 64), (8, 8, 128), (48, 6, 128)])
    c["batch"] = _between(rng, 1, 256)
    # Context lengths: as long as the batch leaves room for in the largest listed case.
    top = min(131072, 1000000 // c["batch"])
    c["hi"] = _between(rng, 128, max(256, top))
    c["lo"] = max(1, int(c["hi"] * rng.uniform(0.05, 1.0)))
    c["settled"] = kind == "loop"
    if rng.random() < 0.25 and kind in ("step", "loop"):
        c["logits"], c["s_lo"], c["s_hi"] = "mixed", 0.3, 0.3
    if kind == "step_f32":
        c.update(dtype="f32", q_heads=8, kv_heads=8, head_dim=64, batch=min(c["batch"], 32),
                 hi=min(c["hi"], 4096), lo=min(c["lo"], 4096))
    if kind == "exact":
        c.update(scoring="exact", keep_first=rng.randint(0, 2), keep_last=rng.randint(0, 2))
    if kind == "estimate":
        c.update(estimator=rng.choice(["topk", "tail"]), est_k=_between(rng, 16, 512),
                 guards=rng.random() < 0.5)
    return c


# --------------------------------------------------------------------------- inputs

def _quantiles(n):
    return [(i + 0.5) / n for i in range(n)]


def _lengths(c):
    """Context lengths of the case, in ascending order."""
    q = _quantiles(c["batch"])
    if c["ctx"] == "uniform":
        return [int(round(c["lo"] + (c["hi"] - c["lo"]) * x)) for x in q]
    z = torch.special.ndtri(torch.tensor(q, dtype=torch.float64))      # lognormal, median 1024
    return [min(c["hi"], max(c["lo"], int(round(1024.0 * math.exp(v))))) for v in z.tolist()]


def _scales(c):
    return [c["s_lo"] + (c["s_hi"] - c["s_lo"]) * x for x in _quantiles(c["batch"])]


def _deal(values, g):
    p = torch.randperm(len(values), generator=g).tolist()
    return [values[i] for i in p]


def _max_blocks(c):
    return -(-(c["hi"] + (ROOM if c["kind"] == "loop" else 0)) // 16)


def _config(c, blocks):
    step = c["kind"] != "sample"
    g = c.get("guards", False)
    est = dict(exact=0, topk=1, tail=2)[c.get("estimator", "exact")]
    return make_config(
        max_batch=c["batch"], num_q_heads=c["q_heads"] if step else 8,
        num_kv_heads=c["kv_heads"] if step else 8, head_dim=c["head_dim"] if step else 64,
        max_blocks_per_seq=_max_blocks(c) if step else 1, num_pool_blocks=max(1, blocks),
        vocab=c["vocab"], kv_dtype=int(c.get("dtype", "bf16") == "bf16"),
        scale=1.0 / math.sqrt(c["head_dim"] if step else 64), eta=ETA, h_target=H_TARGET,
        t_min=T_MIN, t_max=T_MAX, eps_h=0.5 if g else 0.0, h_min=H_TARGET, kappa_min=KAPPA_MIN,
        b_min=B_MIN, log_v=math.log(c["vocab"]), estimator=est, est_k=c.get("est_k", 256),
        t_cal=T_CAL, rho_t=RHO_T if g else math.inf, dkappa=DKAPPA if g else 1.0,
        scoring=int(c.get("scoring", "meankey") == "exact"), keep_first=c.get("keep_first", 0),
        keep_last=c.get("keep_last", 0))


class _Inputs:
    """Everything the seed draws, on the GPU."""


def _inputs(c, seed):
    x = _Inputs()
    dev = "cuda"
    g = torch.Generator()
    g.manual_seed(seed)
    gd = torch.Generator(device=dev)
    gd.manual_seed(seed)
    if c["kind"] == "schedule":
        n = c["pool"]

        def uniform(hi):
            return torch.rand(n, generator=gd, device=dev) * hi

        x.tau_last, x.gain = uniform(50.0), uniform(0.5)
        x.tau = x.tau_last + uniform(0.5)
        x.age = torch.randint(0, 40, (n,), generator=gd, device=dev, dtype=torch.int32)
        x.n_kept = torch.randint(0, 512, (n,), generator=gd, device=dev, dtype=torch.int32)
        x.ctx_lens = torch.randint(0, 32768, (n,), generator=gd, device=dev, dtype=torch.int32)
        return x
    B, V = c["batch"], c["vocab"]
    scales = _deal(_scales(c), g)
    # Settled temperatures: entropies at and a little above the target.
    temps = [1.0] * B
    if c["settled"] and c["logits"] == "normal":
        x_hi = math.sqrt(2.0 * math.log(V))
        temps = [min(T_MAX, max(T_MIN, s / (x_hi * (0.86 + 0.3 * u))))
                 for s, u in zip(scales, _deal(_quantiles(B), g))]
    f32 = dict(dtype=torch.float32, device=dev)
    if c["kind"] != "summary":
        x.logits = torch.randn(B, V, generator=gd, device=dev)
        x.logits *= torch.tensor(scales, **f32)[:, None]
        if c["logits"] == "mixed":          # every other row peaked, by a random rank of each token
            ranks = 1.0 + torch.arange(V, **f32)
            for b in range(0, B, 2):
                x.logits[b] = (-ZIPF * torch.log(ranks))[torch.randperm(V, generator=gd, device=dev)]
        x.temp = torch.tensor(temps, **f32)
        x.h_prev = torch.rand(B, generator=gd, device=dev) * math.log(V)
        x.uniforms = torch.rand(B, generator=gd, device=dev)
    if c["kind"] == "sample":
        return x
    Hq, Hkv, d = c["q_heads"], c["kv_heads"], c["head_dim"]
    edt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    x.lens = _deal(_lengths(c), g)
    grow = 1 if c["kind"] == "loop" else 0
    nbs = [-(-(n + grow) // 16) for n in x.lens]
    x.blocks, maxb = sum(nbs), _max_blocks(c)
    perm = torch.randperm(x.blocks, generator=gd, device=dev).to(torch.int32)
    x.rows = torch.full((B, maxb), -1, dtype=torch.int32)      # the block tables, on the host
    perm, at = perm.cpu(), 0
    for b, nb in enumerate(nbs):
        x.rows[b, :nb] = perm[at:at + nb]
        at += nb
    x.tables = x.rows.to(dev)
    x.k = torch.empty((x.blocks, Hkv, 16, d), dtype=edt, device=dev).normal_(generator=gd)
    x.v = torch.empty((x.blocks, Hkv, d, 16), dtype=edt, device=dev).normal_(generator=gd)
    x.ctx_lens = torch.tensor(x.lens, dtype=torch.int32, device=dev)
    if c["kind"] == "summary":
        return x
    x.q = torch.empty((B, Hq, d), dtype=edt, device=dev).normal_(generator=gd)
    if c["kind"] == "loop":
        x.k_new = torch.empty((B, Hkv, d), dtype=edt, device=dev).normal_(generator=gd)
        x.v_new = torch.empty((B, Hkv, d), dtype=edt, device=dev).normal_(generator=gd)
    if c["scoring"] == "meankey":
        x.ksum = _means(c, x)
    return x


def _valid(x):
    """Valid tokens of every pool block."""
    n = torch.full((x.blocks,), 16, dtype=torch.int64)
    for b, length in enumerate(x.lens):
        j = length // 16
        if j < x.rows.shape[1] and x.rows[b, j] >= 0:      # the partial block, or one still empty
            n[int(x.rows[b, j])] = length % 16
    return n.to("cuda")


def _means(c, x, dtype=torch.float32):
    """Mean key of every block, over its valid slots."""
    n = _valid(x)
    out = torch.empty((x.blocks, c["kv_heads"], c["head_dim"]), dtype=dtype, device="cuda")
    slot = torch.arange(16, device="cuda")
    for a in range(0, x.blocks, 8192):
        k = x.k[a:a + 8192].double()
        m = (slot[None, :] < n[a:a + 8192, None])[:, None, :, None]
        s = torch.where(m, k, torch.zeros((), dtype=torch.float64, device="cuda")).sum(2)
        out[a:a + 8192] = s / n[a:a + 8192].clamp(min=1)[:, None, None]
    return out


# --------------------------------------------------------------------------- the calls

class _State:
    """A program's buffers; owns its library context."""

    ctx = None

    def __del__(self):
        if self.ctx and ent is not None:      # None: the interpreter is ending
            ent.ent_destroy(self.ctx)


def prepare(case, seed):
    c, x = case, _inputs(case, seed)
    s = _State()
    s.kind, s.x, s.at = c["kind"], x, 0
    s.stream = torch.cuda.current_stream().cuda_stream
    f32, i32 = dict(dtype=torch.float32, device="cuda"), dict(dtype=torch.int32, device="cuda")
    if c["kind"] == "schedule":
        s.pool, s.b_sel, s.prm = c["pool"], c["b_sel"], ent.ent_sched_params(*PRM)
        s.selected, s.n_selected = torch.full((c["pool"],), -1, **i32), torch.zeros(1, **i32)
        s.priority = torch.zeros(c["pool"], **f32)
        s.ctx = ent.ent_init(make_config(max_batch=1, max_blocks_per_seq=1, num_pool_blocks=1))
        return s
    B = s.B = c["batch"]
    s.ctx = ent.ent_init(_config(c, getattr(x, "blocks", 1)))
    if c["kind"] == "summary":
        s.ksum = torch.zeros((x.blocks, c["kv_heads"], c["head_dim"]), **f32)
        return s

    def slots(v):
        return v.expand(SLOTS, B).contiguous().unbind(0)

    s.h_prev, s.tau, s.temp = slots(x.h_prev), slots(torch.zeros(B, **f32)), slots(x.temp)
    s.h, s.temp_used, s.tokens = torch.zeros(B, **f32), torch.zeros(B, **f32), torch.zeros(B, **i32)
    s.row_stats = torch.zeros((B, ent.ent_row_stats_chunks(c["vocab"]), 2), **f32)
    if c["kind"] == "sample":
        return s
    s.kappa = slots(torch.full((B,), KAPPA_PREV if c["guards"] else math.nan, **f32))
    s.lens = slots(x.ctx_lens) if c["kind"] == "loop" else None
    maxb = x.tables.shape[1]
    s.kept, s.n_kept = torch.full((B, maxb), -1, **i32), torch.zeros(B, **i32)
    s.out = torch.zeros((B, c["q_heads"], c["head_dim"]), **f32)
    s.ksum = getattr(x, "ksum", None)
    if c["kind"] == "step":
        s.lse = torch.zeros((B, c["q_heads"]), **f32)
        s.scores, s.theta = torch.zeros((B, maxb), **f32), torch.zeros(B, **f32)
    return s


def run(s):
    x, i = s.x, s.at % SLOTS
    s.at += 1
    if s.kind == "schedule":
        ent.ent_schedule(s.ctx, s.pool, s.prm, x.tau, x.n_kept, x.ctx_lens, x.tau_last, x.gain,
                         x.age, s.b_sel, s.selected, s.n_selected, s.priority, s.stream)
        return dict(selected=s.selected, n_selected=s.n_selected, priority=s.priority,
                    gain=x.gain, tau_last=x.tau_last, age=x.age)
    if s.kind == "summary":
        ent.ent_block_summary(s.ctx, s.B, x.k, x.tables, x.ctx_lens, s.ksum, s.stream)
        return dict(ksum=s.ksum)
    state = dict(h=s.h, temp_used=s.temp_used, tokens=s.tokens, h_prev=s.h_prev[i], tau=s.tau[i],
                 temp=s.temp[i])
    if s.kind == "sample":
        ent.ent_entropy_temperature(s.ctx, s.B, x.logits, x.logits.stride(0), s.h_prev[i],
                                    s.tau[i], s.temp[i], s.h, s.temp_used, s.row_stats, s.stream)
        ent.ent_sample(s.ctx, s.B, x.logits, x.logits.stride(0), s.row_stats, s.temp_used,
                       x.uniforms, s.tokens, s.stream)
        return state
    state.update(kept=s.kept, n_kept=s.n_kept, out=s.out, kappa=s.kappa[i])
    if s.kind == "loop":
        ent.ent_decode_step_append(s.ctx, s.B, x.logits, x.logits.stride(0), s.h_prev[i],
                                   s.tau[i], s.temp[i], x.q, x.k, x.v, s.ksum, x.tables,
                                   s.lens[i], x.uniforms, x.k_new, x.v_new, s.h, s.temp_used,
                                   s.kept, s.n_kept, s.out, s.tokens, s.row_stats,
                                   stream=s.stream, kappa=s.kappa[i])
        state.update(ctx_lens=s.lens[i], ksum=s.ksum, k_cache=x.k, v_cache=x.v)
        return state
    ent.ent_decode_step(s.ctx, s.B, x.logits, x.logits.stride(0), s.h_prev[i], s.tau[i],
                        s.temp[i], x.q, x.k, x.v, s.ksum, x.tables, x.ctx_lens, x.uniforms, s.h,
                        s.temp_used, s.kept, s.n_kept, s.out, s.tokens, s.row_stats, s.lse,
                        s.scores, s.theta, s.stream, s.kappa[i])
    state.update(lse=s.lse, scores=s.scores, theta=s.theta)
    return state


# --------------------------------------------------------------------------- what a pass needs

def _estimate(c, p):
    """The entropy, or the estimate of it that the case uses, of rows of probabilities."""
    est = c.get("estimator", "exact")
    if est == "exact" or c["est_k"] >= c["vocab"]:
        return torch.special.entr(p).sum(-1)
    top = torch.topk(p, c["est_k"], -1).values
    m = top.sum(-1)
    h = torch.special.entr(top / m[..., None]).sum(-1)
    if est == "tail":
        rest = torch.clamp(1.0 - m, min=0.0)
        h = h + torch.special.entr(m) + torch.special.entr(rest) + rest * math.log(c["vocab"] - c["est_k"])
    return h


def _kept_fraction(c):
    """Mean kept fraction, from the entropies of rows made of the distributions' quantiles."""
    V = c["vocab"]
    log_v, x_hi, total = math.log(V), math.sqrt(2.0 * math.log(V)), 0.0
    normal = torch.special.ndtri((torch.arange(V, dtype=torch.float64) + 0.5) / V)
    zipf = -ZIPF * torch.log(torch.arange(1, V + 1, dtype=torch.float64))
    for i, (s, u) in enumerate(zip(_scales(c), _quantiles(c["batch"]))):
        x = x_hi * (0.86 + 0.3 * u) if c["settled"] and c["logits"] == "normal" else s
        z = zipf if c["logits"] == "mixed" and i % 2 == 0 else x * normal
        h = float(_estimate(c, torch.softmax(z, 0))) + (0.5 if c["guards"] else 0.0)
        kappa = KAPPA_MIN + (1.0 - KAPPA_MIN) * min(1.0, max(0.0, (h - H_TARGET) / (log_v - H_TARGET)))
        total += max(kappa, KAPPA_PREV - DKAPPA if c["guards"] else 0.0)
    return total / c["batch"]


def work(case):
    c = case
    if c["kind"] == "schedule":
        return dict(bytes=c["pool"] * (24 + 12) + 4 * c["b_sel"], flops=10 * c["pool"])
    B, V = c["batch"], c["vocab"]
    logits = dict(bytes=4 * B * V, flops=6 * B * V)
    if c["kind"] == "sample":
        return logits
    tokens = sum(_lengths(c))
    blocks = sum(-(-n // 16) for n in _lengths(c))
    Hq, Hkv, d, e = c["q_heads"], c["kv_heads"], c["head_dim"], 2 if c["dtype"] == "bf16" else 4
    if c["kind"] == "summary":
        return dict(bytes=tokens * Hkv * d * e + blocks * Hkv * d * 4, flops=tokens * Hkv * d)
    f = _kept_fraction(c)
    exact = c["scoring"] == "exact"
    score = tokens * Hkv * d * e if exact else blocks * Hkv * d * 4
    keep = f * tokens * Hkv * d * e * (1 if exact else 2)    # every key was read already
    scored = tokens if exact else blocks
    return dict(bytes=logits["bytes"] + score + keep + B * Hq * d * (e + 4),
                flops=logits["flops"] + 2 * scored * Hq * d + 4 * f * tokens * Hq * d)


def tolerance(case):
    """Floats: 32-bit sums, and probabilities of about 16 bits in the bf16 attention.  Whole
    values are equal unless a score or a running sum lies within rounding of a threshold."""
    if case["kind"] == "schedule":
        return "exact"
    if case["kind"] in ("summary", "sample"):
        return dict(rel=2e-6, differ=0.005)
    return dict(rel=1e-5, differ=0.01)


# --------------------------------------------------------------------------- 64 bits

def _budget(c, x, h, nb, b):
    """Kept fraction and number of blocks, in the stated order of 32-bit operations."""
    f = lambda v: torch.tensor(v, dtype=torch.float32)  # noqa: E731
    log_v, h_min, k_min = f(math.log(c["vocab"])), f(H_TARGET), f(KAPPA_MIN)
    guarded = torch.maximum(f(float(h)) + f(0.5 if c["guards"] else 0.0), h_min)
    u = torch.clamp((guarded - h_min) / (log_v - h_min), 0.0, 1.0)
    kappa = k_min + (f(1.0) - k_min) * u
    if c["guards"]:
        kappa = torch.maximum(kappa, f(KAPPA_PREV) - f(DKAPPA))
    k = min(nb, max(min(B_MIN, nb), int(torch.ceil(kappa * f(float(nb))))))
    return float(kappa), k


def _sequence(c, x, h, b):
    """Scores, threshold, attention and log-sum-exp of one sequence."""
    N, Hq, Hkv, d = x.lens[b], c["q_heads"], c["kv_heads"], c["head_dim"]
    nb, G = -(-N // 16), Hq // Hkv
    scale = 1.0 / math.sqrt(d)
    pages = x.tables[b, :nb].long()
    counts = torch.full((nb,), 16.0, dtype=torch.float64, device="cuda")
    counts[-1] = N - 16 * (nb - 1)
    qt = x.q[b].double().view(Hkv, G, d).transpose(1, 2).contiguous()          # [Hkv, d, G]
    if c["scoring"] == "exact":
        keys = x.k[pages].double().permute(1, 0, 2, 3).reshape(Hkv, nb * 16, d)[:, :N].contiguous()
        a = torch.softmax(scale * torch.matmul(keys, qt), 1)
        t = torch.zeros((Hkv, nb * 16, G), dtype=torch.float64, device="cuda")
        t[:, :N] = torch.special.entr(a)
        score = t.view(Hkv, nb, 16, G).sum((0, 2, 3)) / Hq
    else:
        means = x.ksum[pages].double().permute(1, 0, 2).contiguous()           # [Hkv, nb, d]
        z = scale * torch.matmul(means, qt)
        big = torch.logsumexp(z + torch.log(counts)[None, :, None], 1, keepdim=True)
        score = (counts[None, :, None] * torch.exp(z - big) * (big - z)).sum((0, 2)) / Hq
    kappa, k = _budget(c, x, h, nb, b)
    forced = torch.zeros(nb, dtype=torch.bool, device="cuda")
    forced[:c["keep_first"]] = True
    if c["keep_last"]:
        forced[-c["keep_last"]:] = True
    k = max(k, int(forced.sum()))
    rank = torch.where(forced, math.inf, score)
    theta = torch.topk(rank, k).values[-1]
    kept = torch.nonzero(rank >= theta).flatten()
    n = min(N, 16 * int(kept.numel())) if int(kept[-1]) < nb - 1 else \
        16 * (int(kept.numel()) - 1) + N - 16 * (nb - 1)
    keys = x.k[pages[kept]].double().permute(1, 0, 2, 3).reshape(Hkv, -1, d)[:, :n].contiguous()
    vals = x.v[pages[kept]].double().permute(1, 2, 0, 3).reshape(Hkv, d, -1)[:, :, :n].contiguous()
    s = scale * torch.matmul(keys, qt)                                         # [Hkv, n, G]
    out = torch.matmul(vals, torch.softmax(s, 1)).transpose(1, 2).reshape(Hq, d)
    return kappa, score, theta, out, torch.logsumexp(s, 1).reshape(Hq)


def exact(case, seed):
    c, x = case, _inputs(case, seed)
    if c["kind"] == "schedule":
        al, be, ga, slo, slack, floor, rate = PRM
        ran = x.age == 0
        gain, tau, last = x.gain.double(), x.tau.double(), x.tau_last.double()
        gain = torch.where(ran, (1.0 - rate) * gain + rate * (tau - last), gain)
        cost = al * x.n_kept + be * ((x.ctx_lens + 15) // 16) \
            + ga * torch.clamp(slo - x.age.double(), min=slack)
        return dict(selected=None, n_selected=None, priority=torch.clamp(gain, min=floor) / cost,
                    gain=gain, tau_last=torch.where(ran, tau, last), age=None)
    if c["kind"] == "summary":
        return dict(ksum=_means(c, x, torch.float64))
    h = _estimate(c, torch.softmax(x.logits.double() / (T_CAL * x.temp.double()[:, None]), 1))
    step = ETA * (h - H_TARGET)
    if c.get("guards"):
        step = torch.clamp(step, -RHO_T, RHO_T)
    r = dict(h=h, temp_used=x.temp.double(), tokens=None, h_prev=h,
             tau=torch.clamp(x.h_prev.double() - h, min=0.0),
             temp=torch.clamp(x.temp.double() * torch.exp(step), T_MIN, T_MAX))
    if c["kind"] == "sample":
        return r
    seqs = [_sequence(c, x, h[b], b) for b in range(c["batch"])]
    f64 = dict(dtype=torch.float64, device="cuda")
    r.update(kept=None, n_kept=None, out=torch.stack([s[3] for s in seqs]),
             kappa=torch.tensor([s[0] for s in seqs], **f64))
    if c["kind"] == "loop":
        k = x.k
        for b, n in enumerate(x.lens):
            k[int(x.rows[b, n // 16]), :, n % 16] = x.k_new[b]
        x.lens = [n + 1 for n in x.lens]
        r.update(ctx_lens=None, ksum=_means(c, x, torch.float64), k_cache=None, v_cache=None)
        return r
    scores = torch.zeros((c["batch"], x.tables.shape[1]), **f64)
    for b, s in enumerate(seqs):
        scores[b, :s[1].numel()] = s[1]
    r.update(lse=torch.stack([s[4] for s in seqs]), scores=scores,
             theta=torch.stack([s[2] for s in seqs]))
    return r
