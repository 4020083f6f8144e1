"""The decode's split of its kept units over workgroups, at the counts where it
changes: fewer units than one range's minimum, one range more or less, the
second workgroup per CU, and segments cut into more pieces than the merge reads
at once.  Every block kept; the reference is plain float64 attention."""
import math

import pytest

from tests.test_gpu_parity import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

# Blocks per sequence; the kept units of the batch are their sum times KV heads.
CASES = [
    ("bf16", 1, 8, [1]), ("bf16", 1, 4, [7]), ("bf16", 1, 4, [8]), ("bf16", 1, 4, [9]),
    ("bf16", 2, 1, [3, 0, 6, 1]), ("bf16", 1, 8, [130]), ("bf16", 8, 4, [43]),
    ("bf16", 1, 8, [8191]), ("bf16", 1, 8, [8192]), ("bf16", 4, 16, [1500, 548, 1]),
    ("bf16", 8, 16, [40, 0] + [13] * 30), ("bf16", 2, 16, [700, 600]),
    ("f32", 1, 1, [1]), ("f32", 2, 4, [5, 0, 30]), ("f32", 1, 2, [2049]), ("f32", 2, 8, [70, 3]),
    ("f32", 1, 16, [300, 1]),
]


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("dtype,hkv,group,blocks", CASES)
def test_decode_over_ranges(torch_cuda, dtype, hkv, group, blocks, head_dim):
    torch = torch_cuda
    from paper_2603_03310_amd import ent
    from paper_2603_03310_amd.runner import make_config
    B, maxb, pool, d = len(blocks), max(blocks), 64, head_dim
    print(f"[ranges] {dtype} Hkv={hkv} G={group} d={d} blocks={blocks}", flush=True)
    edt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    normal = lambda *s: torch.randn(*s, generator=g, device="cuda").to(edt)  # noqa: E731
    q, k, v = normal(B, hkv * group, d), normal(pool, hkv, 16, d), normal(pool, hkv, d, 16)
    tables = torch.randint(0, pool, (B, maxb), generator=g, device="cuda", dtype=torch.int32)
    lens = [max(0, 16 * n - 3) for n in blocks]
    i32 = dict(dtype=torch.int32, device="cuda")
    ctx_lens, n_kept = torch.tensor(lens, **i32), torch.tensor(blocks, **i32)
    kept = torch.arange(maxb, **i32).expand(B, maxb).contiguous()
    out = torch.full((B, hkv * group, d), math.nan, device="cuda")
    lse = torch.full((B, hkv * group), math.nan, device="cuda")
    scale = 1.0 / math.sqrt(d)
    ctx = ent.ent_init(make_config(max_batch=B, num_q_heads=hkv * group, num_kv_heads=hkv, head_dim=d,
                                   max_blocks_per_seq=maxb, num_pool_blocks=pool, vocab=64,
                                   log_v=math.log(64), kv_dtype=int(dtype == "bf16"), scale=scale))
    try:
        ent.ent_sparse_paged_decode(ctx, B, q, k, v, tables, ctx_lens, kept, n_kept, out, lse)
        assert ent.ent_device_status(ctx) == 0
    finally:
        ent.ent_destroy(ctx)
    # P keeps 16 bits in the bf16 path (2^-17 of each weight, |v| <= 5), and
    # float32 sums; fp32: 32-bit sums only.
    tol = 4e-5 if dtype == "bf16" else 1e-5
    for b, n in enumerate(lens):
        if n == 0:
            assert not out[b].any() and bool((lse[b] == -math.inf).all())
            continue
        pages = tables[b, :blocks[b]].long()
        keys = k[pages].double().permute(1, 0, 2, 3).reshape(hkv, -1, d)[:, :n].contiguous()
        vals = v[pages].double().permute(1, 0, 3, 2).reshape(hkv, -1, d)[:, :n].contiguous()
        qt = q[b].double().view(hkv, group, d).transpose(1, 2).contiguous()
        s = scale * torch.matmul(keys, qt)                       # [Hkv, n, G]
        ref = torch.matmul(torch.softmax(s, 1).transpose(1, 2).contiguous(), vals).reshape(-1, d)
        assert float((out[b].double() - ref).abs().max()) <= tol
        want = torch.logsumexp(s, 1).reshape(-1)
        assert float((lse[b].double() - want).abs().max()) <= 1e-5 * max(1.0, float(want.abs().max()))
