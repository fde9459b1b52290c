"""The int4 GEMM's row-tiled kernel at the edges of its tiles and of its rule:
row counts around each tile height (32 to 160) and around the hand-over from the
small-batch kernel, column counts that leave half a tile, one group, and splits
of the groups; calls of different shapes sharing one workspace.  Tolerance as in
test_gpu_awq.py (its arithmetic is the same: exact products, fp32 sums, one
rescale per group)."""
import dataclasses

import pytest
import torch

from paper_2412_10543_amd import binding
from paper_2412_10543_amd.workloads import awq_problem

import gpu_support as G_
from test_gpu_awq import _check, _device, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [65, 95, 96, 97, 127, 128, 129, 159, 160, 161, 191, 193, 257, 321,
                               479, 641])
def test_rows_around_the_tile_heights(M):
    N, K = 640, 896                       # half a column tile over; 7 groups: uneven splits
    p = awq_problem(M, N, K, seed=M, device="cuda")
    dev = _device(p)
    a = _run(p, *dev)
    _check(p, a)
    assert torch.equal(a.view(torch.int16), _run(p, *dev).view(torch.int16))


@pytest.mark.parametrize("M,N,K", [
    (17, 16512, 256), (31, 16512, 256), (32, 20480, 128),        # wide: one 32-row tile
    (33, 6144, 4096), (63, 6144, 4096), (64, 4608, 4096),        # tall enough: 32- or 64-row tiles
    (64, 4480, 4096), (32, 16384, 256),                          # just below: the small kernel
    (65, 128, 128), (300, 128, 128), (66, 256, 14336),           # one group; 112 groups
    (320, 28672, 256), (2304, 4096, 256), (1500, 10240, 128)])   # unsplit, many tiles
def test_rule_edges(M, N, K):
    p = awq_problem(M, N, K, seed=M + N + K, device="cuda")
    # A quarter of the scales' size: among millions of outputs with a spread near
    # 1 some exceed 8, where bf16 rounding alone (half an ulp, 2^-5) is more than
    # the 2e-2 that the checker also asks for; below 2 it is 2^-8.
    p.scales *= 0.25
    rows = list(range(0, M, 17)) + [M - 1] if M * N > 2 ** 22 else None
    _check(p, _run(p, *_device(p)), rows=rows)


@pytest.mark.parametrize("M", [40, 200])
def test_scales_off_the_plain_path(M):
    """Zero, subnormal, huge and negative scales in some columns and groups only
    (the others of their waves keep the plain ones)."""
    N, K = 6144, 4096
    p = awq_problem(M, N, K, seed=77, device="cuda")
    p.scales[3, 5::64] = 0.0
    p.scales[:, 70] = 0.0
    p.scales[7, 9::128] = 2.0 ** -130
    p.scales[11, 200] = 2.0 ** 12
    p.scales[12, 33::32] *= -1.0
    p.scales[0, 1::97] = 0.0
    y = _run(p, *_device(p))
    cols = list(range(0, 260)) + [N - 1]
    _check(p, y, rows=list(range(0, M, 13)) + [M - 1], cols=cols)
    assert bool((y[:, 70] == 0).all())


def test_one_workspace_for_every_shape():
    """Split and unsplit calls of both kernels in turn in one workspace,
    zero-filled once."""
    shapes = [(16, 4096, 14336), (320, 1024, 2048), (70, 512, 4096), (48, 6144, 4096),
              (1200, 256, 256), (16, 4096, 14336), (130, 2048, 1024)]
    ws = torch.zeros(max(binding.rag_awq_workspace_size(*s) for s in shapes), dtype=torch.uint8,
                     device="cuda")
    for i, (M, N, K) in enumerate(shapes):
        p = awq_problem(M, N, K, seed=500 + i, device="cuda")
        dev = _device(p)
        alone = _run(p, *dev)
        y = _run(p, *dev, ws=ws)
        assert torch.equal(y.view(torch.int16), alone.view(torch.int16)), (M, N, K)
        _check(p, y, rows=[0, M // 2, M - 1], cols=[0, 1, N // 2, N - 1])


def test_small_workspace_takes_the_small_batch_kernel():
    """32 rows of a layer that the row-tiled kernel would split: a call that
    brings only what the small-batch kernel needs takes that one (the bits of
    the knob that asks for it).  (K one group longer than the small kernel takes
    without a split: layers up to there are its own.)"""
    M, N, K = 32, 16512, 2176
    p = awq_problem(M, N, K, seed=3, device="cuda")
    dev = _device(p)
    with G_.env("RAG_AWQ_SM_SPLITS", 1):
        size = binding.rag_awq_workspace_size(M, N, K)
        small = _run(p, *dev)
    assert binding.rag_awq_workspace_size(M, N, K) > size
    y = _run(p, *dev, ws=torch.zeros(size, dtype=torch.uint8, device="cuda"))
    assert torch.equal(y.view(torch.int16), small.view(torch.int16))
    _check(p, y, cols=list(range(0, N, 31)))


@pytest.mark.parametrize("M,N,K", [(17, 32768, 512), (32, 16512, 2048), (33, 32768, 1024),
                                   (64, 20480, 1024), (17, 32896, 512), (40, 18432, 1152)])
def test_wide_layers_at_the_small_kernels_edge(M, N, K):
    """17 to 64 rows of wide layers on both sides of the small kernel's limits:
    256 workgroups, no split."""
    p = awq_problem(M, N, K, seed=M + N + K, device="cuda")
    _check(p, _run(p, *_device(p)), cols=list(range(0, N, 61)) + [N - 1])


def _small_kernel(p, dev):
    """The same call 64 rows at a time through the small-batch kernel (one fp32
    FMA per group and output: y + s (P - (128 + z) S))."""
    x, out = p.x, []
    with G_.env("RAG_AWQ_SM_SPLITS", 1):
        for r in range(0, x.shape[0], 64):
            out.append(_run(dataclasses.replace(p, x=x[r:r + 64].contiguous()), *dev))
    return torch.cat(out)


@pytest.mark.parametrize("M,N,K", [(20, 16512, 2176), (48, 4608, 4096), (130, 512, 1024),
                                   (320, 640, 896), (1200, 256, 256)])
def test_scales_and_rows_that_are_not_ordinary(M, N, K):
    """Infinite, NaN, huge and subnormal scales (one such group a column), and
    rows with an infinity, a NaN or nothing but zeros: finite, infinite and NaN
    outputs as from the small-batch kernel."""
    p = awq_problem(M, N, K, seed=M + K, device="cuda")
    kinds = [float("inf"), -float("inf"), float("nan"), 2.0 ** 118, 2.0 ** 127, -2.0 ** 100,
             2.0 ** -130, None, 2.0 ** 41, -2.0 ** 40, 1.5 * 2.0 ** 121]
    s = p.scales.float()
    for col in range(N):
        v = kinds[col % len(kinds)]
        if v is not None:
            s[(col // len(kinds)) % s.shape[0], col] = v
    p.scales = s.to(torch.bfloat16)
    p.x[1, 5], p.x[M // 2, K - 1], p.x[3] = float("inf"), float("nan"), 0.0
    dev = _device(p)
    y, ref = _run(p, *dev).double(), _small_kernel(p, dev).double()
    assert torch.equal(y.isnan(), ref.isnan())
    assert torch.equal(y.isinf(), ref.isinf()) and torch.equal(y.sign()[y.isinf()],
                                                               ref.sign()[y.isinf()])
    ok = y.isfinite()
    assert bool(ok.any()) and not bool(ok.all())
    # both within test_gpu_awq's bound of the exact sum: half an ulp of bf16 each,
    # and the fp32 sums' part of the magnitudes A entering them
    g = torch.arange(K, device="cuda") // 128
    mag = (torch.from_numpy(p.codes).cuda().double() + dev[2][g].double() + 256) * \
        dev[1][g].double().abs()
    A = p.x.double().abs().nan_to_num(0.0, posinf=0.0) @ mag.nan_to_num(0.0, posinf=0.0)
    bound = 2.0 ** -7 * ref.abs() + 2 * (2.0 ** -17 + (K // 128) * 2.0 ** -22) * A
    assert bool(((y - ref).abs() <= bound)[ok].all())
