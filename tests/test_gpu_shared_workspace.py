"""Calls of different sizes following each other in one workspace that was
zero-filled once: what one call leaves behind the counters must never lie where
another counts.  Each result equals, bit for bit, that of a workspace of its own."""
import numpy as np
import pytest
import torch

from gpu_support import scale_for, to_dev_i32, workspace_for
from paper_2412_10543_amd import binding
from paper_2412_10543_amd.workloads import normal_bf16, paged_pool


def _up(x):
    return (x + 255) // 256 * 256


def test_decode_counters_keep_their_place():
    """The bytes in front of the partials are the same for every call, and
    enough for its counters."""
    hq, d = 32, 128
    front = set()
    for rows, hkv, mb, splits in [(1, 8, 400, 0), (31, 8, 400, 0), (32, 8, 400, 0), (40, 8, 400, 0),
                                  (256, 8, 400, 0), (20, 8, 40, 0), (3, 8, 188, 6), (300, 8, 40, 2),
                                  (1100, 1, 313, 4), (8192, 8, 313, 2), (200, 1, 563, 0)]:
        n = binding.rag_attn_decode_num_splits(rows, hkv, mb, 16, splits)
        assert n > 1
        size = binding.rag_attn_decode_workspace_size(rows, hq, hkv, d, mb, 16, splits)
        front.add(size - _up(rows * hq * n * d * 4) - _up(rows * hq * n * 4))
        assert min(front) >= 4 * rows * hkv
    assert len(front) == 1
    # more pairs than there are counters: not split
    assert binding.rag_attn_decode_num_splits(8193, 8, 313, 16, 2) == 1
    assert binding.rag_attn_decode_workspace_size(8193, hq, 8, d, 313, 16, 2) == 0


def _decode(q, pool, lens, hkv, table, ws, splits, cu, nd):
    o = torch.full_like(q, float("nan"))
    kw = {} if cu is None else dict(cu_seqlens_q=to_dev_i32(cu), num_decode_seqs=nd,
                                    max_seqlen_q=max(np.diff(cu)))
    binding.rag_attn_decode_paged(q, pool.k_cache, pool.v_cache, o, table, to_dev_i32(lens),
                                  scale_for(q.shape[2]), num_splits=splits, workspace=ws, **kw)
    torch.cuda.synchronize()
    return o


@pytest.mark.gpu
def test_decode_batches_grow_and_shrink_in_one_workspace():
    """Rows that differ from call to call, on both sides of 256 (row, kv head)
    pairs, automatic and explicit splits, and a mixed batch."""
    hq, hkv, d, mb = 32, 8, 64, 400
    r = np.random.Generator(np.random.PCG64(31))
    lens = [int(x) for x in r.integers(4500, 16 * mb, size=64)]
    pool = paged_pool(lens, hkv, d, 32, device="cuda", max_blocks=mb)
    calls = [(31, 0, 0), (40, 0, 0), (20, 0, 0), (64, 0, 0), (31, 0, 0), (7, 5, 0), (64, 3, 0),
             (30, 0, 2), (50, 2, 0), (33, 4, 3), (64, 0, 0)]
    size = max(binding.rag_attn_decode_workspace_size(n, hq, hkv, d, mb, 16, s) for n, s, _ in calls)
    ws = torch.zeros(size, dtype=torch.uint8, device="cuda")
    for i, (n, splits, pieces) in enumerate(calls):
        print(f"call {i}: {n} rows, splits {splits}, {pieces} pieces", flush=True)
        cu = None if pieces == 0 else list(range(n + 1)) + [n + 24 * (j + 1) for j in range(pieces)]
        s = n + pieces
        q = normal_bf16((n if cu is None else cu[-1], hq, d), 40 + i, "cuda")
        table = pool.block_tables[:s].contiguous()
        own = workspace_for(n, hq, hkv, d, mb, splits)
        want = _decode(q, pool, lens[:s], hkv, table, own, splits, cu, n)
        got = _decode(q, pool, lens[:s], hkv, table, ws, splits, cu, n)
        assert bool(torch.isfinite(got).all()), f"call {i}: rows left unwritten"
        assert torch.equal(got.view(torch.int16), want.view(torch.int16)), f"call {i}"


@pytest.mark.gpu
def test_more_rows_than_counters_are_not_split():
    rows, hq, hkv, d = 8200, 8, 8, 64
    lens = [1 + (7 * i) % 40 for i in range(rows)]
    pool = paged_pool(lens, hkv, d, 51, device="cuda")
    q = normal_bf16((rows, hq, d), 52, "cuda")
    one = _decode(q, pool, lens, hkv, pool.block_tables, None, 1, None, rows)
    two = _decode(q, pool, lens, hkv, pool.block_tables, None, 2, None, rows)
    assert torch.equal(one.view(torch.int16), two.view(torch.int16))
    assert bool(torch.isfinite(two).all())


def _linear(M, N, K, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    # every bit pattern is a valid packing of 4-bit codes
    qw = torch.randint(-2 ** 31, 2 ** 31 - 1, (K // 128, N, 16), generator=g, device="cuda",
                       dtype=torch.int32)
    sc = ((torch.rand((K // 128, N), generator=g, device="cuda") + 0.5) / (6.5 * K ** 0.5))
    z = torch.randint(0, 16, (K // 128, N), generator=g, device="cuda", dtype=torch.uint8)
    return torch.randn((M, K), generator=g, device="cuda").bfloat16(), qw, sc.bfloat16(), z


def _gemm(p, ws):
    y = torch.full((p[0].shape[0], p[1].shape[1]), float("nan"), dtype=torch.bfloat16, device="cuda")
    binding.rag_awq_gemm(*p, y, ws)
    torch.cuda.synchronize()
    return y


def _codes(qw, cols):
    """uint8 [K, len(cols)] of packed words (the layout of rag_awq_pack_weights)."""
    w = qw[:, cols].cpu().numpy().view(np.uint32)               # [G, cols, 16]
    out = np.zeros((w.shape[0], 128, len(cols)), dtype=np.uint8)
    for i in range(16):
        a, b, c = i >> 3, (i >> 2) & 1, i & 3
        for j in range(8):
            out[:, 8 * (4 * c + 2 * b + a) + j] = (w[:, :, i] >> (4 * (j // 2) + 16 * (j % 2))) & 15
    return out.reshape(-1, len(cols))


def _reference(p, cols):
    x, qw, sc, z = p
    g = np.arange(x.shape[1]) // 128
    w = (_codes(qw, cols).astype(np.float64) - z[:, cols].cpu().numpy()[g]) * \
        sc[:, cols].double().cpu().numpy()[g]
    return x.double().cpu().numpy() @ w


@pytest.mark.gpu
def test_layers_of_any_width_share_a_workspace():
    """Wide layers (hundreds of column blocks to count) and narrow split ones in
    turn: the linear layers of a 70B model at 16 rows, and row-tiled splits."""
    shapes = [(16, 10240, 8192), (16, 57344, 8192), (200, 1024, 2048), (16, 57344, 8192),
              (16, 8192, 28672), (40, 4096, 14336), (16, 57344, 8192), (16, 10240, 8192)]
    ws = torch.zeros(max(binding.rag_awq_workspace_size(*s) for s in shapes), dtype=torch.uint8,
                     device="cuda")
    for i, (M, N, K) in enumerate(shapes):
        print(f"call {i}: M={M} N={N} K={K}", flush=True)
        p = _linear(M, N, K, 60 + i)
        own = torch.zeros(max(binding.rag_awq_workspace_size(M, N, K), 256), dtype=torch.uint8,
                          device="cuda")
        want, got = _gemm(p, own), _gemm(p, ws)
        assert bool(torch.isfinite(got).all()), f"call {i}: columns left unwritten"
        assert torch.equal(got.view(torch.int16), want.view(torch.int16)), f"call {i}"
        cols = [0, 1, N // 2, N - 1]
        # outputs of order 1: bf16 rounding, and fp32 sums of 128-term groups
        assert np.abs(got[:, cols].double().cpu().numpy() - _reference(p, cols)).max() <= 2e-2


def test_more_column_blocks_than_counters():
    """A split small batch of more column blocks than counters is not split."""
    assert binding.rag_awq_workspace_size(4, 128 * 16384, 4224) > 0
    assert binding.rag_awq_workspace_size(4, 128 * 16385, 4224) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("M", [1, 5, 16])
def test_more_column_blocks_than_counters_on_the_gpu(M):
    N, K = 128 * 16385, 4224
    p = _linear(M, N, K, 80 + M)
    got = _gemm(p, torch.zeros(256, dtype=torch.uint8, device="cuda"))
    assert bool(torch.isfinite(got).all())
    cols = [0, 31, 32, 255, 256, N // 2 + 7, N - 1]
    assert np.abs(got[:, cols].double().cpu().numpy() - _reference(p, cols)).max() <= 2e-2


@pytest.mark.gpu
@pytest.mark.parametrize("N,K,batch,rows", [
    (4096, 14336, 64, [1, 9, 16, 17, 31, 32, 33, 37, 40, 48, 58, 63, 64]),   # 7B down
    (28672, 4096, 64, [7, 16, 17, 32, 33, 47, 58, 64]),                      # 7B gate_up
    (4096, 4096, 1024, [16, 40, 65, 96, 128, 200, 320, 511, 700, 1024]),     # 7B o
    (1024, 2048, 0, [17, 40, 64, 65, 200, 320])])                            # nothing to spare
def test_smaller_batches_fit_a_larger_ones_workspace(N, K, batch, rows):
    """A workspace sized for a layer's largest batch takes every smaller one
    (the split is then the best that fits it)."""
    size = binding.rag_awq_workspace_size(batch, N, K) if batch else 256
    ws = torch.zeros(max(size, 256), dtype=torch.uint8, device="cuda")
    cols = [0, 33, N // 2, N - 1]
    full = _linear(max(rows), N, K, 90 + N % 7)
    want = _reference(full, cols)
    for M in rows:
        print(f"M={M}", flush=True)
        got = _gemm((full[0][:M],) + full[1:], ws)
        assert bool(torch.isfinite(got).all())
        assert np.abs(got[:, cols].double().cpu().numpy() - want[:M]).max() <= 2e-2
