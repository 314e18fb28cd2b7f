"""Lists of every length through the gather: shorter and longer than what one round of its workgroups copies, empty, and with
entries behind the count that are no positions. Bit copies, so every row is compared with the indexed one."""
import pytest
import torch

from paper_2602_08686_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 64), (torch.bfloat16, 128), (torch.float32, 64), (torch.float32, 128)])
@pytest.mark.parametrize("batch,kv,length,budget", [(1, 1, 70, 33), (2, 3, 517, 40), (1, 8, 9001, 512), (1, 32, 2048, 300), (3, 48, 900, 100)])
def test_lists_of_any_length(dtype, d, batch, kv, length, budget):
    window = 32
    g = torch.Generator(device="cuda")
    g.manual_seed(length * 31 + d)
    cap = min(length, budget * kv - (kv - 1) * window)
    k = torch.randn(batch, kv, length, d, generator=g, device="cuda").to(dtype)
    v = torch.randn(batch, kv, length, d, generator=g, device="cuda").to(dtype)
    count = torch.randint(0, cap + 1, (batch, kv), generator=g, device="cuda", dtype=torch.int32)
    count.view(-1)[0] = cap  # all of the budget in one head
    count.view(-1)[-1] = 0 if batch * kv > 1 else cap
    idx = torch.randint(0, length, (batch, kv, cap), generator=g, device="cuda", dtype=torch.int32)
    at = torch.arange(cap, device="cuda").expand(batch, kv, cap)
    idx = torch.where(at < count[..., None], idx, torch.full_like(idx, 1 << 30))  # never followed
    p = B.make_params(batch=batch, n_q_heads=kv, n_kv_heads=kv, head_dim=d, seq_len=length, window=window, dtype=dtype,
                      pool=B.POOL_NONE, pool_kernel=1, budget=budget, cap=cap)
    outs = [torch.full((batch, kv, cap, d), 7.0, dtype=dtype, device="cuda") for _ in range(2)]
    B.ckv_compact_kv(p, k, v, idx, count, *outs)
    safe = torch.where(at < count[..., None], idx, torch.zeros_like(idx)).long()[..., None].expand(-1, -1, -1, d)
    for src, out in zip((k, v), outs):
        want = torch.where(at[..., None] < count[..., None, None], src.gather(2, safe), torch.full_like(out, 7.0))
        assert torch.equal(out, want)
