"""Block summaries over the splits of a block's KV heads between waves (odd
head counts, a last wave with one tile), both head sizes and both cache types,
full, partial and missing blocks.  The reference is the slot-order float32 sum
divided by the count, which the kernel evaluates bit for bit."""
import numpy as np
import pytest

from tests.test_gpu_parity import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("hkv", [1, 2, 3, 5, 8])
def test_summary_bits(torch_cuda, hkv, dtype, head_dim):
    torch = torch_cuda
    from paper_2603_03310_amd import ent
    from paper_2603_03310_amd.runner import make_config
    lens, maxb, pool, d = [0, 1, 15, 16, 33, 111], 7, 40, head_dim
    print(f"[summary] {dtype} Hkv={hkv} d={d}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    k = torch.randn(pool, hkv, 16, d, generator=g, device="cuda")
    k = k.to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    perm = torch.randperm(pool, generator=g, device="cuda").to(torch.int32)
    nbs = [-(-n // 16) for n in lens]
    tables = torch.full((len(lens), maxb), -1, dtype=torch.int32, device="cuda")
    want = np.full((pool, hkv, d), 7.0, dtype=np.float32)     # (numpy divides; torch multiplies by 1 / n)
    keys = k.float().cpu().numpy()
    at = 0
    for b, nb in enumerate(nbs):
        tables[b, :nb] = perm[at:at + nb]
        for j in range(nb):
            p = int(perm[at + j])
            n = min(16, lens[b] - 16 * j)
            acc = np.zeros((hkv, d), dtype=np.float32)
            for slot in range(n):
                acc = acc + keys[p, :, slot]
            want[p] = acc / np.float32(n)
        at += nb
    ksum = torch.full((pool, hkv, d), 7.0, device="cuda")     # blocks of no sequence stay
    ctx = ent.ent_init(make_config(max_batch=len(lens), num_q_heads=hkv, num_kv_heads=hkv,
                                   head_dim=d, max_blocks_per_seq=maxb, num_pool_blocks=pool,
                                   kv_dtype=int(dtype == "bf16")))
    try:
        ent.ent_block_summary(ctx, len(lens), k, tables,
                              torch.tensor(lens, dtype=torch.int32, device="cuda"), ksum)
        assert ent.ent_device_status(ctx) == 0
    finally:
        ent.ent_destroy(ctx)
    assert np.array_equal(ksum.cpu().numpy(), want)
