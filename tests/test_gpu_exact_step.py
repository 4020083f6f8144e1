"""The exact scoring mode's whole step (its own launches) against the staged
calls, bit for bit, with the append and without: both cache types, a head count
off the powers of two, tables of one tile and of several, an estimator, forced
keeps, with and without summaries."""
import math

import pytest

from tests.test_gpu_parity import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

# dtype, KV heads, group, head_dim, block-table width, lengths, options
CASES = [
    ("bf16", 8, 4, 128, 100, [1, 17, 300, 1500], {}),
    ("bf16", 3, 4, 64, 20, [5, 0, 319], dict(keep_first=1, keep_last=2)),
    ("bf16", 4, 2, 128, 2500, [39000, 5, 4096], dict(estimator=2, est_k=64)),
    ("bf16", 1, 16, 128, 300, [4799, 256], dict(estimator=1, est_k=16, eps_h=0.5, dkappa=0.05)),
    ("f32", 8, 1, 64, 40, [1, 100, 639], {}),
    ("f32", 2, 8, 128, 600, [9000, 33], {}),
]


@pytest.mark.parametrize("summaries", [True, False], ids=["ksum", "no_ksum"])
@pytest.mark.parametrize("dtype,hkv,group,d,maxb,lens,opts", CASES)
def test_exact_step_equals_staged(torch_cuda, dtype, hkv, group, d, maxb, lens, opts, summaries):
    torch = torch_cuda
    from paper_2603_03310_amd import ent
    from paper_2603_03310_amd.runner import make_config
    print(f"[exact step] {dtype} Hkv={hkv} G={group} d={d} MAXB={maxb}", flush=True)
    B, V, hq = len(lens), 9001, hkv * group
    edt = torch.bfloat16 if dtype == "bf16" else torch.float32
    pool = sum(-(-(n + 1) // 16) for n in lens)

    def program(form):
        g = torch.Generator(device="cuda")
        g.manual_seed(11)
        normal = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
        f32, i32 = dict(dtype=torch.float32, device="cuda"), dict(dtype=torch.int32, device="cuda")
        logits, q = 2.0 * normal(B, V), normal(B, hq, d).to(edt)
        k, v = normal(pool, hkv, 16, d).to(edt), normal(pool, hkv, d, 16).to(edt)
        k_new, v_new = normal(B, hkv, d).to(edt), normal(B, hkv, d).to(edt)
        uniforms = torch.rand(B, generator=g, device="cuda")
        perm = torch.randperm(pool, generator=g, device="cuda").to(torch.int32)
        tables, at = torch.full((B, maxb), -1, **i32), 0
        for b, n in enumerate(lens):
            nb = -(-(n + 1) // 16)
            tables[b, :nb] = perm[at:at + nb]
            at += nb
        s = dict(ctx_lens=torch.tensor(lens, **i32), h_prev=torch.full((B,), 5.0, **f32),
                 tau=torch.zeros(B, **f32), temp=torch.ones(B, **f32),
                 kappa=torch.full((B,), 0.5, **f32), h=torch.zeros(B, **f32),
                 used=torch.zeros(B, **f32), kept=torch.full((B, maxb), -1, **i32),
                 n_kept=torch.zeros(B, **i32), out=torch.zeros(B, hq, d, **f32),
                 lse=torch.zeros(B, hq, **f32), scores=torch.zeros(B, maxb, **f32),
                 theta=torch.zeros(B, **f32), tokens=torch.zeros(B, **i32), k=k, v=v,
                 stats=torch.zeros(B, ent.ent_row_stats_chunks(V), 2, **f32),
                 ksum=torch.zeros(pool, hkv, d, **f32))
        ksum = s["ksum"] if summaries else None
        ctx = ent.ent_init(make_config(
            max_batch=B, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, max_blocks_per_seq=maxb,
            num_pool_blocks=pool, vocab=V, log_v=math.log(V), kv_dtype=int(dtype == "bf16"),
            scale=1.0 / math.sqrt(d), scoring=1, **opts))
        try:
            if form == "append":
                ent.ent_decode_step_append(
                    ctx, B, logits, V, s["h_prev"], s["tau"], s["temp"], q, k, v, ksum, tables,
                    s["ctx_lens"], uniforms, k_new, v_new, s["h"], s["used"], s["kept"], s["n_kept"],
                    s["out"], s["tokens"], s["stats"], s["lse"], s["scores"], s["theta"],
                    kappa=s["kappa"])
            else:
                if form == "step":
                    ent.ent_decode_step(
                        ctx, B, logits, V, s["h_prev"], s["tau"], s["temp"], q, k, v, ksum, tables,
                        s["ctx_lens"], uniforms, s["h"], s["used"], s["kept"], s["n_kept"], s["out"],
                        s["tokens"], s["stats"], s["lse"], s["scores"], s["theta"], None, s["kappa"])
                else:
                    ent.ent_entropy_temperature(ctx, B, logits, V, s["h_prev"], s["tau"], s["temp"],
                                                s["h"], s["used"], s["stats"])
                    ent.ent_block_select(ctx, B, q, ksum, tables, s["ctx_lens"], s["h"], s["kept"],
                                         s["n_kept"], s["scores"], s["theta"], None, s["kappa"], k)
                    ent.ent_sparse_paged_decode(ctx, B, q, k, v, tables, s["ctx_lens"], s["kept"],
                                                s["n_kept"], s["out"], s["lse"])
                    ent.ent_sample(ctx, B, logits, V, s["stats"], s["used"], uniforms, s["tokens"])
                ent.ent_kv_append(ctx, B, k_new, v_new, tables, s["ctx_lens"], k, v, ksum)
            assert ent.ent_device_status(ctx) == 0
        finally:
            ent.ent_destroy(ctx)
        return s

    staged = program("staged")
    for form in ("step", "append"):
        got = program(form)
        for name, want in staged.items():
            assert torch.equal(torch.nan_to_num(got[name].float(), nan=7.0),
                               torch.nan_to_num(want.float(), nan=7.0)), (form, name)
