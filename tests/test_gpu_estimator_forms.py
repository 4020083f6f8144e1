"""The top-k estimators over rows that suit the binned selection and rows that
need the general one (top k spread over more than 64 doublings, few finite
logits; a row with a NaN runs, with no value promised), with ties of every kind
(equal, rounded, clipped, few threads above), at vocabularies around the limits of the
two (row ends off 16 bytes, maxima past the LDS stage, past the registers) and
at both ends of k.  The reference is the definition in float64."""
import math

import numpy as np
import pytest

from tests.test_gpu_parity import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

TOPK, TAIL = 1, 2


def _rows(torch, V):
    g = torch.Generator(device="cuda")
    g.manual_seed(V)
    n = torch.randn(V, generator=g, device="cuda")
    ranks = 1.0 + torch.randperm(V, generator=g, device="cuda").float()
    spike, masked, low, few = 2.0 * n, 2.0 * n, 2.0 * n, torch.full_like(n, -math.inf)
    spike = spike.clone()
    spike[V // 2] = 60.0
    masked[::2] = -math.inf
    low[V // 3:] = torch.finfo(torch.float32).min
    few[:: max(1, V // 40)] = 2.0 * n[:: max(1, V // 40)]
    clumped = n.clone()
    clumped[: V // 8] += 9.0
    stacked = torch.ones_like(n)       # ties, and above them many tokens of few threads
    for i in range(4):
        stacked[1024 * i: 1024 * i + 160] = 3.0 + 0.25 * n[1024 * i: 1024 * i + 160]
    return [n * 0.01, n * 0.5, n * 4.0, n * 60.0, -1.2 * torch.log(ranks), spike, masked, low, few,
            clumped, torch.zeros_like(n), torch.round(n), torch.round(40.0 * n) / 40.0,
            torch.clamp(2.0 * n, max=3.0), n.bfloat16().float(), stacked, -200.0 + 1e-2 * n]


@pytest.mark.parametrize("k", [1, 16, 256, 512])
@pytest.mark.parametrize("V", [300, 5000, 50257, 128256, 131073, 150001, 262145])
def test_estimate(torch_cuda, V, k):
    torch = torch_cuda
    from paper_2603_03310_amd import ent
    from paper_2603_03310_amd.runner import make_config
    print(f"[estimator] V={V} k={k}", flush=True)
    rows = _rows(torch, V)
    B = len(rows) + 1
    logits = torch.stack(rows + [rows[1].clone()])
    logits[-1, V // 2] = math.nan
    f32 = dict(dtype=torch.float32, device="cuda")
    z = logits.double()
    p = torch.softmax(z, 1)
    kk = min(k, V)
    top = torch.topk(p, kk, 1).values
    m = top.sum(1)
    want = {TOPK: torch.special.entr(top / m[:, None]).sum(1)}
    rest = torch.clamp(1.0 - m, min=0.0)
    want[TAIL] = want[TOPK] + torch.special.entr(m) + torch.special.entr(rest) \
        + rest * math.log(max(1, V - kk))
    for est in (TOPK, TAIL):
        ctx = ent.ent_init(make_config(max_batch=B, vocab=V, log_v=math.log(V), h_min=0.5,
                                       h_target=0.5, estimator=est, est_k=k))
        try:
            h, used = torch.zeros(B, **f32), torch.zeros(B, **f32)
            h_prev, tau, temp = torch.zeros(B, **f32), torch.zeros(B, **f32), torch.ones(B, **f32)
            ent.ent_entropy_temperature(ctx, B, logits, V, h_prev, tau, temp, h, used)
            torch.cuda.synchronize()
        finally:
            ent.ent_destroy(ctx)
        ref = want[est] if k < V else torch.special.entr(p).sum(1)
        # Scaled logits up to 400 carry 2^-24 of themselves into the exponent,
        # and -p ln p weighs that by at most ln V: 400 / 2^24 x 12.5 = 3e-4 at
        # the widest rows (x 60, and those around -200), under 1e-4 in the
        # others (|z| <= 60).
        tol = torch.full((B,), 1e-4, dtype=torch.float64, device="cuda")
        tol[3] = tol[B - 2] = 3e-4
        err = (h.double() - ref).abs()[:-1]
        assert bool((err <= tol[:-1]).all()), (est, err.tolist())


# The binned form counts maxima, and lists tokens, in bins of t = z log2(e) / T
# below the row's maximum.  Rows with a token whose exact t lies on one side of
# the list's edge and whose rounded t on the other: count, list and maxima must
# all go by the rounded one.

_LOG2E = np.float32(1.4426950408889634)
_BINS, _PER_UNIT = np.float32(2048), np.float32(32)


def _bin_pos(z, c2, M, fused):
    """Bin position of logits z, with t rounded or with t - M in one rounding."""
    if fused:
        d = (z.astype(np.float64) * np.float64(c2) - np.float64(M)).astype(np.float32)
    else:
        d = z * c2 - M
    return d * _PER_UNIT + _BINS


def _edge_row(rng, V, k, offset, T, planted):
    """A normal row around `offset` with `planted` tokens that straddle the edge
    at temperature T, beside the maxima of threads well above it."""
    chunks = -(-V // 4096)
    while True:
        z = (2.0 * rng.standard_normal(V) + offset).astype(np.float32)
        c2 = _LOG2E / np.float32(T)
        t = np.full(chunks * 4096, -np.inf, np.float32)
        t[:V] = z * c2
        maxima = t.reshape(chunks, 4, 256, 4).max(axis=(1, 3)).reshape(-1)
        M = maxima.max()
        edge = np.floor((np.sort(maxima)[-k] - M) * _PER_UNIT + _BINS)
        z0 = np.float32((M + (edge - _BINS) / _PER_UNIT) / c2)
        near = z0 + np.spacing(z0) * np.arange(-64, 65, dtype=np.float32)
        a, b = _bin_pos(near, c2, M, False) >= edge, _bin_pos(near, c2, M, True) >= edge
        if not (a != b).any():
            continue
        pick = near[a != b][0]
        room = []
        for j in np.argsort(maxima)[::-1][:6]:         # the threads of the largest maxima
            at = (j // 256) * 4096 + (j % 256) * 4 + 1024 * np.arange(4)[:, None] + np.arange(4)
            at = at.reshape(-1)
            at = at[at < V]
            room += [p for p in at if p != at[np.argmax(z[at])]]
        z[np.array(room[:planted])] = pick
        return z


@pytest.mark.parametrize("k", [16, 256])
@pytest.mark.parametrize("offset", [-100.0, 20.0, 300.0])
def test_estimate_of_rows_with_tokens_at_the_edge(torch_cuda, offset, k):
    torch = torch_cuda
    from paper_2603_03310_amd import ent
    from paper_2603_03310_amd.runner import make_config
    V, planted, per_t = 32000, 80, 16
    rng = np.random.default_rng(1320 + k)
    temps = np.repeat(np.array([0.3, 0.37, 0.61, 0.7, 1.0, 1.9], np.float32), per_t)
    print(f"[estimator edge] k={k} offset={offset} rows={len(temps)}", flush=True)
    rows = [_edge_row(rng, V, k, offset, T, planted) for T in temps]
    rows += [(2.0 * rng.standard_normal(V) + offset).astype(np.float32) for _ in range(160)]
    temps = np.concatenate([temps, rng.uniform(0.2, 2.0, 160).astype(np.float32)])
    B = len(rows)
    logits = torch.from_numpy(np.stack(rows)).cuda()
    T = torch.from_numpy(temps).cuda()
    p = torch.softmax(logits.double() / T.double()[:, None], 1)
    top = torch.topk(p, k, 1).values
    m = top.sum(1)
    ref = torch.special.entr(top / m[:, None]).sum(1)
    f32, i32 = dict(dtype=torch.float32, device="cuda"), dict(dtype=torch.int32, device="cuda")
    ctx = ent.ent_init(make_config(
        max_batch=B, num_q_heads=4, num_kv_heads=4, head_dim=64, max_blocks_per_seq=1,
        num_pool_blocks=1, vocab=V, log_v=math.log(V), estimator=TOPK, est_k=k, t_min=1e-3))
    try:
        got = []
        for form in ("staged", "staged", "step"):
            h, used = torch.zeros(B, **f32), torch.zeros(B, **f32)
            h_prev, tau, temp = torch.zeros(B, **f32), torch.zeros(B, **f32), T.clone()
            if form == "staged":
                ent.ent_entropy_temperature(ctx, B, logits, V, h_prev, tau, temp, h, used)
            else:
                zeros = lambda *s, **d: torch.zeros(*s, device="cuda", **d)  # noqa: E731
                bf = dict(dtype=torch.bfloat16)
                ent.ent_decode_step(
                    ctx, B, logits, V, h_prev, tau, temp, zeros(B, 4, 64, **bf),
                    zeros(1, 4, 16, 64, **bf), zeros(1, 4, 64, 16, **bf), zeros(1, 4, 64),
                    torch.zeros(B, 1, **i32), torch.ones(B, **i32), zeros(B), h, used,
                    torch.zeros(B, 1, **i32), torch.zeros(B, **i32), zeros(B, 4, 64),
                    torch.zeros(B, **i32))
            torch.cuda.synchronize()
            got.append(h.double())
    finally:
        ent.ent_destroy(ctx)
    # t rounds by 2^-24 |t|; -p ln p weighs that by at most ln k, and its log2
    # and exp2 sums add some 1e-6.
    tmax = (logits.abs().max(1).values / T).double() * 1.45
    tol = 3e-6 + tmax * 2.0 ** -24 * math.log(k)
    err = (got[0] - ref).abs()
    assert bool((err <= tol).all()), (float((err / tol).max()), int((err > tol).sum()))
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
