"""The decode plan made on the GPU from the rows' lengths: row counts at the
edges of its 64-row chunks, whole and crossing pieces, one long row among short
ones (more units than a row may have pieces), tables wide enough for the plan
with more (row, kv head) pairs than CUs.  Against the fp64 oracle, and with the
same rows cut uniformly."""
import numpy as np
import pytest
import torch

from gpu_support import (assert_parity, gpu_paged, oracle_paged, scale_for, to_dev_i32,
                         workspace_for)
from paper_2412_10543_amd import binding
from paper_2412_10543_amd.workloads import normal_bf16, paged_pool

pytestmark = pytest.mark.gpu


def _lens(kind, rows):
    r = np.random.Generator(np.random.PCG64(rows))
    if kind == "equal":
        return [600] * rows
    if kind == "one_key":
        return [1] * rows
    if kind == "one_long":
        return [int(x) for x in r.integers(1, 40, size=rows - 1)] + [9000]
    return [int(x) for x in np.exp(r.uniform(np.log(100), np.log(6000), size=rows))]


@pytest.mark.parametrize("rows,hq,hkv,d,kind,max_blocks", [
    (1, 8, 1, 128, "one_long", None),     # 256 units, at most 64 pieces a row
    (2, 32, 8, 128, "one_long", None),
    (5, 4, 2, 64, "spread", None),
    (12, 8, 4, 128, "spread", None),      # crossing
    (20, 32, 8, 128, "equal", None),      # whole rows
    (30, 16, 8, 64, "one_long", None),
    (63, 8, 1, 128, "spread", None),
    (64, 8, 2, 64, "one_long", None),
    (65, 8, 2, 64, "spread", None),
    (129, 4, 1, 64, "one_key", None),
    (200, 8, 1, 64, "one_long", None),
    (40, 32, 8, 64, "spread", 400),       # more pairs than CUs: crossing
    (70, 8, 4, 64, "one_long", 600),      # ... whole rows, the long one cut
    (256, 4, 1, 64, "equal", 130),
    (256, 8, 2, 64, "one_long", None),
    (257, 4, 1, 64, "spread", None),      # past the plan: uniform
])
def test_balanced_plan(orc, rows, hq, hkv, d, kind, max_blocks):
    lens = _lens(kind, rows)
    pool = paged_pool(lens, hkv, d, 900 + rows, device="cuda", max_blocks=max_blocks)
    q = normal_bf16((rows, hq, d), 901 + rows, "cuda")
    scale = scale_for(d)
    got = gpu_paged(q, pool, hq, hkv, d, scale)
    want = oracle_paged(orc, q, pool, scale)
    assert_parity(got, want, f"{rows} rows {kind}")
    cut = gpu_paged(q, pool, hq, hkv, d, scale, num_splits=3)
    # two cuts of one sum: each bf16 output is within one rounding (2^-8 of its
    # size) plus the weights' own bf16 rounding (2^-9 of the largest value, 5) of
    # the other
    assert float((got.float() - cut.float()).abs().max()) <= 2e-2
    # a used workspace is left ready for the next call
    ws = workspace_for(rows, hq, hkv, d, pool.block_tables.shape[1])
    for _ in range(3):
        o = torch.full_like(q, float("nan"))
        binding.rag_attn_decode_paged(q, pool.k_cache, pool.v_cache, o, pool.block_tables,
                                      to_dev_i32(lens), scale, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(o.view(torch.int16), got.view(torch.int16))


@pytest.mark.parametrize("entry", ["no workspace", "small workspace", "scratch"])
def test_uniform_splits_where_the_plan_does_not_fit(orc, entry):
    """More pairs than CUs: a call without the memory for the balanced plan is
    cut uniformly (here: not at all), as one with num_splits=1."""
    lens = _lens("spread", 40)
    hq, hkv, d = 32, 8, 64
    pool = paged_pool(lens, hkv, d, 970, device="cuda", max_blocks=400)
    if entry == "scratch":                 # 256 rows x 64 heads x 8 slots: over the scratch
        lens, hq = [17] * 256, 64
        pool = paged_pool(lens, hkv, d, 971, device="cuda", max_blocks=200)
    q = normal_bf16((len(lens), hq, d), 972, "cuda")
    want = gpu_paged(q, pool, hq, hkv, d, scale_for(d), num_splits=1)
    o = torch.full_like(q, float("nan"))
    args = (q, pool.k_cache, pool.v_cache, o, pool.block_tables, to_dev_i32(lens), scale_for(d))
    if entry == "scratch":
        binding.rag_attn_decode_paged_noalloc(*args)
    else:
        ws = torch.zeros(256, dtype=torch.uint8, device="cuda") if entry[0] == "s" else None
        binding.rag_attn_decode_paged(*args, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(o.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("rows,hq,hkv,d,kind", [(20, 32, 8, 128, "equal"), (66, 8, 2, 64, "spread"),
                                                (3, 8, 1, 128, "one_long")])
def test_append_stores_after_the_pages(rows, hq, hkv, d, kind):
    """The appending step equals a cache write then a step, bit for bit."""
    lens = _lens(kind, rows)
    pool = paged_pool(lens, hkv, d, 950 + rows, device="cuda")
    q = normal_bf16((rows, hq, d), 951, "cuda")
    kn, vn = (normal_bf16((rows, hkv, d), s, "cuda") for s in (952, 953))
    kl, scale = to_dev_i32(lens), scale_for(d)
    ws = workspace_for(rows, hq, hkv, d, pool.block_tables.shape[1])
    k2, v2 = pool.k_cache.clone(), pool.v_cache.clone()
    last = [n - 1 for n in lens]
    slots = [int(pool.block_tables[i, p // 16]) * 16 + p % 16 for i, p in enumerate(last)]
    o, o2 = torch.empty_like(q), torch.empty_like(q)
    binding.rag_kv_cache_write(kn, vn, k2, v2, to_dev_i32(slots))
    binding.rag_attn_decode_paged(q, k2, v2, o2, pool.block_tables, kl, scale, workspace=ws)
    binding.rag_attn_decode_paged_append(q, kn, vn, pool.k_cache, pool.v_cache, o,
                                         pool.block_tables, kl, scale, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(o.view(torch.int16), o2.view(torch.int16))
    assert torch.equal(pool.k_cache.view(torch.int16), k2.view(torch.int16))
    assert torch.equal(pool.v_cache.view(torch.int16), v2.view(torch.int16))


def _mixed_lens(kind, rows):
    r = np.random.Generator(np.random.PCG64(7 * rows))
    if kind == "short":                    # nothing to even out
        return [int(x) for x in r.integers(1, 300, size=rows)]
    if kind == "alike":                    # long, but every row about the same
        return [int(x) for x in r.integers(4990, 5049, size=rows)]
    return [int(x) for x in r.integers(1, 60, size=rows - 1)] + [6000]     # one long


@pytest.mark.parametrize("append", [False, True])
@pytest.mark.parametrize("rows,hq,hkv,d", [
    (16, 16, 16, 128), (32, 32, 8, 128), (63, 8, 8, 64), (64, 16, 4, 64), (65, 8, 4, 128),
    (128, 32, 2, 128), (256, 4, 1, 64), (8, 32, 32, 128), (12, 24, 24, 64)])
@pytest.mark.parametrize("kind", ["short", "alike", "long"])
def test_rows_behind_a_wide_table(orc, kind, rows, hq, hkv, d, append):
    """As many (row, kv head) pairs as CUs and a table wide enough for the plan:
    rows that are short stay whole (the bits of num_splits=1), long ones that are
    alike too where they come to about a whole number per CU, and one row that is
    far longer than the rest is cut."""
    lens = _mixed_lens(kind, rows)
    mb = 400
    assert binding.rag_attn_decode_num_splits(rows, hkv, mb, 16) > 1
    pool = paged_pool(lens, hkv, d, 960 + rows, device="cuda", max_blocks=mb)
    q = normal_bf16((rows, hq, d), 961, "cuda")
    scale, kl = scale_for(d), to_dev_i32(lens)
    ws = workspace_for(rows, hq, hkv, d, mb)

    def call(**kw):
        o = torch.full_like(q, float("nan"))
        if append:
            kn, vn = (normal_bf16((rows, hkv, d), s, "cuda") for s in (962, 963))
            binding.rag_attn_decode_paged_append(q, kn, vn, pool.k_cache, pool.v_cache, o,
                                                 pool.block_tables, kl, scale, **kw)
        else:
            binding.rag_attn_decode_paged(q, pool.k_cache, pool.v_cache, o, pool.block_tables, kl,
                                          scale, **kw)
        torch.cuda.synchronize()
        return o

    got, again, whole = call(workspace=ws), call(workspace=ws), call(num_splits=1)
    assert torch.equal(got.view(torch.int16), again.view(torch.int16))
    uncut = kind == "short" or (kind == "alike" and -rows * hkv % 256 < 32)
    assert torch.equal(got.view(torch.int16), whole.view(torch.int16)) == uncut
    # (the appended rows are in the cache by now)
    assert_parity(got, oracle_paged(orc, q, pool, scale), f"{kind} {rows} rows")
