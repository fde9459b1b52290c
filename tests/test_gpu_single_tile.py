"""The prefill with one query tile per workgroup: its tiles run last first from
max_seqlen, which may be longer than every sequence; short, empty and one-row
sequences, both masks, every head grouping, the fused cache write.  Against the
fp64 oracle."""
import pytest
import torch

from gpu_support import (MAX_ABS, assert_parity, cu_from_lens, oracle_prefill, prefill_inputs,
                         scale_for, to_dev_i32)
from paper_2412_10543_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,extra_k,over,hq,hkv,d,causal", [
    ([1], 0, 0, 4, 2, 64, True),
    ([65, 0, 1, 130], 0, 700, 8, 2, 128, True),
    ([300, 20], 0, 1, 4, 2, 64, True),
    ([257], 40, 300, 4, 4, 128, True),
    ([64, 63, 200], 5, 64, 16, 2, 128, False),
])
def test_single_tile_prefill(orc, lens, extra_k, over, hq, hkv, d, causal):
    lens_k = [n + extra_k if n else 0 for n in lens]
    q, k, v = prefill_inputs(lens, lens_k, hq, hkv, d, seed=sum(lens) + hq)
    o = torch.full_like(q, float("nan"))
    lse = torch.full((hq, q.shape[0]), float("nan"), device="cuda")
    binding.rag_attn_prefill_varlen(q, k, v, o, lse, to_dev_i32(cu_from_lens(lens)),
                                    to_dev_i32(cu_from_lens(lens_k)), max(lens) + over,
                                    max(lens_k) + over, scale_for(d), causal)
    torch.cuda.synchronize()
    want, want_lse = oracle_prefill(orc, q, k, v, lens, lens_k, scale_for(d), causal)
    assert_parity(o, want, str(lens))
    assert float((lse.double().cpu() - torch.from_numpy(want_lse)).abs().max()) <= MAX_ABS


def test_single_tile_prefill_writes_the_cache():
    lens, hq, hkv, d = [70, 0, 1, 129], 8, 2, 128
    q, k, v = prefill_inputs(lens, lens, hq, hkv, d, seed=4)
    t = sum(lens)
    g = torch.Generator().manual_seed(1)
    slots = torch.randperm(16 * 20, generator=g)[:t].to(torch.int32)
    slots[::7] = -1
    slots = slots.cuda()
    kc, vc = (torch.zeros((20, hkv, 16, d), dtype=torch.bfloat16, device="cuda") for _ in "kv")
    k2, v2 = torch.zeros_like(kc), torch.zeros_like(vc)
    o, o2 = torch.empty_like(q), torch.empty_like(q)
    cu = to_dev_i32(cu_from_lens(lens))
    binding.rag_attn_prefill_varlen_kvcache(q, k, v, o, None, cu, 500, scale_for(d), kc, vc, slots)
    binding.rag_attn_prefill_varlen(q, k, v, o2, None, cu, cu, 129, 129, scale_for(d))
    binding.rag_kv_cache_write(k, v, k2, v2, slots)
    torch.cuda.synchronize()
    for a, b in ((o, o2), (kc, k2), (vc, v2)):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
