"""The top-k estimators over rows that suit the binned selection and rows that
need the general one (top k spread over more than 64 doublings, thousands of
equal logits, few finite ones; a row with a NaN runs, with no value promised), at vocabularies around the limits of the
two (row ends off 16 bytes, maxima past the LDS stage, past the registers) and
at both ends of k.  The reference is the definition in float64."""
import math

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
    return [n * 0.01, n * 0.5, n * 4.0, n * 60.0, -1.2 * torch.log(ranks), spike, masked, low, few,
            clumped, torch.zeros_like(n), torch.round(n), torch.round(40.0 * n) / 40.0]


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
        # the widest row (x 60), under 1e-4 in the others (|z| <= 60).
        tol = torch.full((B,), 1e-4, dtype=torch.float64, device="cuda")
        tol[3] = 3e-4
        err = (h.double() - ref).abs()[:-1]
        assert bool((err <= tol[:-1]).all()), (est, err.tolist())
