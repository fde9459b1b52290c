"""The work that is timed: prompt prefill, paged decode, mixed batches and the
int4-weight linear layers, each through the public binding, from one tiny
prompt to a 70B-head long prompt.

A case is a dict of plain values.  Its `kind` picks the path:
  prefill  one packed launch over the prompts of `queries` queries, stuffed
           (one prompt of all chunks per query) or mapped (one prompt per
           chunk), with the K/V rows not written to the paged cache, written by
           a second call, or written by the same launch
  decode   one decode step of `rows` running calls against the paged cache
           (`append`: the step's new token stored by the same launch)
  mixed    one launch of decode rows and chunked-prefill pieces
  step     `layers` transformer layers of one decode step (int4 projections and
           MLP around the appending attention), captured once in a HIP graph
           and replayed, as a serving loop runs its per-token launches
  linear   the four int4 linear layers of one transformer layer at `rows` rows

Lengths are drawn from the case's own `sizes` seed, so that they belong to the
case; values (Q, K, V ~ N(0, 1) in bf16, codes and zero points uniform on
0..15, scales that keep outputs of order 1, pages in random physical order)
are drawn on the GPU from prepare()'s seed.
"""
import math
import random

import torch

from paper_2412_10543_amd import binding

BLOCK = 16
GROUP = 128
HEADS_7B = dict(hq=32, hkv=8, d=128)
LAYER_7B = dict(hidden=4096, inner=14336)


def listed():
    return [
        # the smallest prompt: a 32-token query with two 128-token chunks on a
        # small model; launch latency and a few workgroups
        dict(name="tiny_prompt", kind="prefill", method="stuff", queries=1, query_len=32,
             chunks_lo=2, chunks_hi=2, chunk_len=128, hq=4, hkv=2, d=64, write="none", lse=True,
             sizes=1001),
        # one stuff query admitted at low load (7B heads, nine 512-token
        # chunks), its K/V then written to the pages, as the engine loop does
        dict(name="stuff_prompt_alone", kind="prefill", method="stuff", queries=1, query_len=77,
             chunks_lo=9, chunks_hi=9, chunk_len=512, **HEADS_7B, write="separate", lse=False,
             sizes=1002),
        # a batch of 16 stuff queries of 5 to 20 chunks (7B heads)
        dict(name="stuff_prompts", kind="prefill", method="stuff", queries=16, query_len=64,
             chunks_lo=5, chunks_hi=20, chunk_len=512, **HEADS_7B, write="none", lse=False,
             sizes=1002),
        # the map phase of 16 map_reduce queries: 320 short mapper prompts, the
        # launch that also fills their pages
        dict(name="mapper_prompts", kind="prefill", method="map", queries=16, query_len=64,
             chunks_lo=20, chunks_hi=20, chunk_len=512, **HEADS_7B, write="fused", lse=False,
             sizes=1003),
        # one long stuff query with the 70B model's heads (35 chunks of 1024)
        dict(name="long_prompt_70b", kind="prefill", method="stuff", queries=1, query_len=64,
             chunks_lo=35, chunks_hi=35, chunk_len=1024, hq=64, hkv=8, d=128, write="none",
             lse=False, sizes=1004),
        # decode of one map_reduce query's 20 mappers: short rows, few of them,
        # launched one by one from the host
        dict(name="mapper_decode_one_query", kind="decode", rows=20, kv_lo=560, kv_hi=640,
             append=True, **HEADS_7B, sizes=1005),
        # decode of a batch of 16 stuff queries
        dict(name="stuff_decode", kind="decode", rows=16, kv_lo=2624, kv_hi=10304, append=True,
             **HEADS_7B, sizes=1006),
        # decode of all mappers of 16 map_reduce queries
        dict(name="mapper_decode", kind="decode", rows=320, kv_lo=576, kv_hi=640, append=False,
             **HEADS_7B, sizes=1007),
        # continuous batching at full load: 256 decoding calls and four
        # 2048-token chunked-prefill pieces with prior context in one launch
        dict(name="mixed_batch", kind="mixed", rows=256, kv_lo=1024, kv_hi=32768, pieces=4,
             piece_len=2048, prior_hi=8192, **HEADS_7B, sizes=1008),
        # the decode step of a 7B model as a serving loop runs it: two layers
        # of it, 16 running calls of short context, replayed from a graph
        dict(name="decode_step_layers", kind="step", rows=16, layers=2, kv_lo=576, kv_hi=1088,
             **HEADS_7B, **LAYER_7B, sizes=1009),
        # the linear layers when all mappers of 16 queries decode together
        dict(name="linear_mapper_decode", kind="linear", rows=320, **HEADS_7B, **LAYER_7B),
        # the linear layers for four 2048-token prompt chunks
        dict(name="linear_prompt_chunks", kind="linear", rows=8192, **HEADS_7B, **LAYER_7B),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the ranges that the listed ones stand for: prompts of
    one chunk to 36k tokens, decode batches of 1 to 320 rows, linear layers of
    1 to 8192 rows, the model shapes above and generic ones."""
    kind = rng.choice(["prefill", "prefill", "decode", "decode", "mixed", "step", "linear",
                       "linear"])
    hq, hkv, d = rng.choice([(32, 8, 128), (32, 8, 128), (32, 8, 128), (64, 8, 128), (4, 2, 64),
                             (32, 8, 64), (16, 16, 128), (24, 8, 128), (32, 2, 128)])
    heads = dict(hq=hq, hkv=hkv, d=d)
    sizes = rng.randrange(1 << 20)
    if kind == "prefill":
        c = dict(kind=kind, method=rng.choice(["stuff", "map"]), queries=_log_int(rng, 1, 16),
                 query_len=rng.randint(1, 128), chunks_lo=1, chunks_hi=_log_int(rng, 1, 35),
                 chunk_len=_log_int(rng, 64, 1024), **heads,
                 write=rng.choice(["none", "separate", "fused"]), lse=rng.random() < 0.25,
                 sizes=sizes)
        # no more work than the long prompt, no more tokens than the mappers
        while sum(n * n for n in _prompt_lens(c)) * hq * d > 35904 ** 2 * 64 * 128 or \
                sum(_prompt_lens(c)) > 190000:
            c["queries"] = max(1, c["queries"] // 2)
            c["chunks_hi"] = max(1, c["chunks_hi"] // 2)
        return c
    if kind == "decode":
        kv = sorted((_log_int(rng, 32, 36000), _log_int(rng, 32, 36000)))
        rows = min(_log_int(rng, 1, 320), max(1, 2400000 // kv[1]))
        return dict(kind=kind, rows=rows, kv_lo=kv[0], kv_hi=kv[1], append=rng.random() < 0.6,
                    **heads, sizes=sizes)
    if kind == "mixed":
        return dict(kind=kind, rows=_log_int(rng, 4, 256), kv_lo=512,
                    kv_hi=_log_int(rng, 1024, 32768), pieces=rng.randint(1, 4),
                    piece_len=_log_int(rng, 64, 2048), prior_hi=_log_int(rng, 16, 8192),
                    **heads, sizes=sizes)
    hidden, inner = rng.choice([(4096, 14336), (4096, 14336),
                                (128 * rng.randint(16, 48), 128 * rng.randint(32, 112))])
    if kind == "step":
        kv = sorted((_log_int(rng, 64, 8192), _log_int(rng, 64, 8192)))
        return dict(kind=kind, rows=_log_int(rng, 1, 64), layers=rng.randint(1, 2), kv_lo=kv[0],
                    kv_hi=kv[1], hq=32, hkv=8, d=128, hidden=hidden, inner=inner, sizes=sizes)
    return dict(kind=kind, rows=_log_int(rng, 1, 8192), hq=32, hkv=8, d=128, hidden=hidden,
                inner=inner)


# ---------------------------------------------------------------------------
# sizes
# ---------------------------------------------------------------------------
def _prompt_lens(c):
    r = random.Random(c["sizes"])
    lens = []
    for _ in range(c["queries"]):
        n = r.randint(c["chunks_lo"], c["chunks_hi"])
        if c["method"] == "stuff":
            lens.append(n * c["chunk_len"] + c["query_len"])
        else:
            lens += [c["chunk_len"] + c["query_len"]] * n
    return lens


def _kv_lens(c):
    """Keys of each decode row, log-uniform in [kv_lo, kv_hi]."""
    r = random.Random(c["sizes"])
    return [_log_int(r, c["kv_lo"], c["kv_hi"]) for _ in range(c["rows"])]


def _prior_lens(c):
    r = random.Random(c["sizes"] + 1)
    return [r.randint(0, c["prior_hi"]) for _ in range(c["pieces"])]


def _layer_shapes(c):
    """(K, N) of the qkv, output, gate-and-up and down projections."""
    h, i, qd, kvd = c["hidden"], c["inner"], c["hq"] * c["d"], c["hkv"] * c["d"]
    return [(h, qd + 2 * kvd), (qd, h), (h, 2 * i), (i, h)]


def _attn_work(lens_q, lens_k, hq, hkv, d):
    pairs = sum(nq * (nk - nq) + nq * (nq + 1) // 2 for nq, nk in zip(lens_q, lens_k))
    return (4.0 * d * hq * pairs,
            sum(4.0 * d * (nq * hq + nk * hkv) for nq, nk in zip(lens_q, lens_k)))


def _linear_work(m, shapes):
    fl = sum(2.0 * m * k * n for k, n in shapes)
    by = sum(2.0 * m * (k + n) + k * n / 2 + 3.0 * (k // GROUP) * n for k, n in shapes)
    return fl, by


def work(c):
    if c["kind"] == "linear":
        fl, by = _linear_work(c["rows"], _layer_shapes(c))
        return {"bytes": by, "flops": fl}
    hq, hkv, d = c["hq"], c["hkv"], c["d"]
    if c["kind"] == "prefill":
        lens = _prompt_lens(c)
        fl, by = _attn_work(lens, lens, hq, hkv, d)
        total = sum(lens)
        if c["lse"]:
            by += 4.0 * hq * total
        if c["write"] != "none":           # the pages written once (the rows are read anyway)
            by += total * (4.0 * hkv * d + 4)
        return {"bytes": by, "flops": fl}
    kv = _kv_lens(c)
    fl, by = _attn_work([1] * len(kv), kv, hq, hkv, d)
    by += sum(4.0 * ((n + BLOCK - 1) // BLOCK) + 4 for n in kv)
    if c["kind"] == "decode":
        return {"bytes": by, "flops": fl}
    if c["kind"] == "mixed":
        lq = [c["piece_len"]] * c["pieces"]
        f2, b2 = _attn_work(lq, [c["piece_len"] + p for p in _prior_lens(c)], hq, hkv, d)
        return {"bytes": by + b2, "flops": fl + f2}
    f2, b2 = _linear_work(c["rows"], _layer_shapes(c))
    return {"bytes": c["layers"] * (by + b2), "flops": c["layers"] * (fl + f2)}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
class _Draw:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))

    def normal(self, *shape):
        return torch.randn(shape, generator=self.g, device="cuda").to(torch.bfloat16)

    def ints(self, lo, hi, shape, dtype):
        return torch.randint(lo, hi, shape, generator=self.g, device="cuda", dtype=dtype)


def _i32(x):
    return torch.tensor(x, dtype=torch.int32, device="cuda")


def _cu(lens):
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    return cu


def _pages(rng, lens):
    """A block table over a pool a quarter larger than needed, physical pages
    in random order.  Returns (table, number of blocks)."""
    n = torch.tensor([(x + BLOCK - 1) // BLOCK for x in lens])
    need = int(n.sum())
    blocks = need + need // 4 + 1
    perm = torch.randperm(blocks, generator=rng.g, device="cuda")
    table = torch.zeros((len(lens), int(n.max())), dtype=torch.int32, device="cuda")
    used = (torch.arange(table.shape[1])[None, :] < n[:, None]).to("cuda")
    table[used] = perm[:need].to(torch.int32)
    return table.contiguous(), blocks


def _slots(table, lens):
    """The slot (page * 16 + offset) of every token, packed."""
    out = [table[s, :(n + BLOCK - 1) // BLOCK].repeat_interleave(BLOCK)[:n] * BLOCK +
           torch.arange(n, device="cuda", dtype=torch.int32) % BLOCK for s, n in enumerate(lens)]
    return torch.cat(out).to(torch.int32).contiguous()


def _zeros(nbytes):
    return torch.zeros(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None


def _prepare_prefill(c, rng):
    lens = _prompt_lens(c)
    total, hq, hkv, d = sum(lens), c["hq"], c["hkv"], c["d"]
    s = dict(case=c, q=rng.normal(total, hq, d), k=rng.normal(total, hkv, d),
             v=rng.normal(total, hkv, d), cu=_i32(_cu(lens)), max_len=max(lens),
             scale=1.0 / math.sqrt(d))
    s["o"] = torch.empty_like(s["q"])
    s["lse"] = torch.empty((hq, total), device="cuda") if c["lse"] else None
    if c["write"] != "none":
        table, blocks = _pages(rng, lens)
        s["slots"] = _slots(table, lens)
        s["k_cache"] = torch.zeros((blocks, hkv, BLOCK, d), dtype=torch.bfloat16, device="cuda")
        s["v_cache"] = torch.zeros_like(s["k_cache"])
    return s


def _prepare_decode(c, rng):
    kv, hq, hkv, d = _kv_lens(c), c["hq"], c["hkv"], c["d"]
    table, blocks = _pages(rng, kv)
    s = dict(case=c, table=table, kv=_i32(kv), k_cache=rng.normal(blocks, hkv, BLOCK, d),
             v_cache=rng.normal(blocks, hkv, BLOCK, d), q=rng.normal(len(kv), hq, d),
             k_new=rng.normal(len(kv), hkv, d), v_new=rng.normal(len(kv), hkv, d),
             scale=1.0 / math.sqrt(d))
    s["o"] = torch.empty_like(s["q"])
    s["ws"] = _zeros(binding.rag_attn_decode_workspace_size(len(kv), hq, hkv, d, table.shape[1]))
    return s


def _prepare_mixed(c, rng):
    kv, hq, hkv, d = _kv_lens(c), c["hq"], c["hkv"], c["d"]
    lens_q = [1] * len(kv) + [c["piece_len"]] * c["pieces"]
    lens_k = kv + [p + c["piece_len"] for p in _prior_lens(c)]
    table, blocks = _pages(rng, lens_k)
    s = dict(case=c, table=table, kv=_i32(lens_k), k_cache=rng.normal(blocks, hkv, BLOCK, d),
             v_cache=rng.normal(blocks, hkv, BLOCK, d), q=rng.normal(sum(lens_q), hq, d),
             cu=_i32(_cu(lens_q)), scale=1.0 / math.sqrt(d))
    s["o"] = torch.empty_like(s["q"])
    s["ws"] = _zeros(binding.rag_attn_decode_workspace_size(len(kv), hq, hkv, d, table.shape[1]))
    return s


def _prepare_linear(c, rng):
    """The four layers, each with its activations, weights and workspace."""
    layers, m = [], c["rows"]
    for k, n in _layer_shapes(c):
        g = k // GROUP
        # every bit pattern is a valid packing of 4-bit codes
        qw = rng.ints(-2 ** 31, 2 ** 31, (g, n, BLOCK), torch.int64).to(torch.int32)
        sc = (torch.rand((g, n), generator=rng.g, device="cuda") + 0.5) / (6.5 * math.sqrt(k))
        layers.append(dict(x=rng.normal(m, k), qw=qw, sc=sc.to(torch.bfloat16),
                           zp=rng.ints(0, 16, (g, n), torch.uint8),
                           y=torch.empty((m, n), dtype=torch.bfloat16, device="cuda"),
                           ws=torch.zeros(max(256, binding.rag_awq_workspace_size(m, n, k)),
                                          dtype=torch.uint8, device="cuda")))
    return layers


def prepare(c, seed):
    rng = _Draw(seed)
    if c["kind"] == "prefill":
        return _prepare_prefill(c, rng)
    if c["kind"] == "decode":
        return _prepare_decode(c, rng)
    if c["kind"] == "mixed":
        return _prepare_mixed(c, rng)
    if c["kind"] == "linear":
        return dict(case=c, linear=_prepare_linear(c, rng))
    s = dict(case=c, layers=[dict(attn=_prepare_decode(c, rng), linear=_prepare_linear(c, rng))
                             for _ in range(c["layers"])])
    torch.cuda.synchronize()
    _step(s)                                   # as a program does before it captures
    torch.cuda.synchronize()
    s["graph"] = torch.cuda.CUDAGraph()
    with torch.cuda.graph(s["graph"]):
        _step(s)
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def _append(s):
    binding.rag_attn_decode_paged_append(s["q"], s["k_new"], s["v_new"], s["k_cache"],
                                         s["v_cache"], s["o"], s["table"], s["kv"], s["scale"],
                                         workspace=s["ws"])


def _gemm(w):
    binding.rag_awq_gemm(w["x"], w["qw"], w["sc"], w["zp"], w["y"], w["ws"])


def _step(s):
    for layer in s["layers"]:
        qkv, out, gate_up, down = layer["linear"]
        _gemm(qkv)
        _append(layer["attn"])
        _gemm(out)
        _gemm(gate_up)
        _gemm(down)


def run(s):
    c = s["case"]
    if c["kind"] == "prefill":
        if c["write"] == "fused":
            binding.rag_attn_prefill_varlen_kvcache(
                s["q"], s["k"], s["v"], s["o"], s["lse"], s["cu"], s["max_len"], s["scale"],
                s["k_cache"], s["v_cache"], s["slots"])
        else:
            binding.rag_attn_prefill_varlen(s["q"], s["k"], s["v"], s["o"], s["lse"], s["cu"],
                                            s["cu"], s["max_len"], s["max_len"], s["scale"])
        out = dict(o=s["o"])
        if c["lse"]:
            out["lse"] = s["lse"]
        if c["write"] == "separate":
            binding.rag_kv_cache_write(s["k"], s["v"], s["k_cache"], s["v_cache"], s["slots"])
        if c["write"] != "none":
            out.update(k_cache=s["k_cache"], v_cache=s["v_cache"])
        return out
    if c["kind"] == "decode":
        if c["append"]:
            _append(s)
            return dict(o=s["o"], k_cache=s["k_cache"], v_cache=s["v_cache"])
        binding.rag_attn_decode_paged(s["q"], s["k_cache"], s["v_cache"], s["o"], s["table"],
                                      s["kv"], s["scale"], workspace=s["ws"])
        return dict(o=s["o"])
    if c["kind"] == "mixed":
        binding.rag_attn_decode_paged(s["q"], s["k_cache"], s["v_cache"], s["o"], s["table"],
                                      s["kv"], s["scale"], cu_seqlens_q=s["cu"],
                                      num_decode_seqs=c["rows"], max_seqlen_q=c["piece_len"],
                                      workspace=s["ws"])
        return dict(o=s["o"])
    if c["kind"] == "linear":
        for w in s["linear"]:
            _gemm(w)
        return [w["y"] for w in s["linear"]]
    s["graph"].replay()
    return [dict(o=x["attn"]["o"], k_cache=x["attn"]["k_cache"], v_cache=x["attn"]["v_cache"],
                 y=[w["y"] for w in x["linear"]]) for x in s["layers"]]


# ---------------------------------------------------------------------------
# 64-bit results and tolerances
# ---------------------------------------------------------------------------
def tolerance(c):
    """Outputs are bf16 (2^-9 relative rounding); attention rounds its weights
    to bf16 as well.  Against exact() the paths are 1.6e-3 to 2.3e-3 off (the
    log-sum-exp 5e-8): about four times that."""
    return {"rel": 1e-2, "max": 0.1}


def _attn64(q, k, v, scale):
    """Bottom-right causal attention of one sequence in 64 bits: q [nq, hq, d],
    k and v [nk, hkv, d] -> ([nq, hq, d], log-sum-exp [hq, nq])."""
    nq, hq, d = q.shape
    nk, hkv, _ = k.shape
    g = hq // hkv
    kt = k.double().permute(1, 2, 0).contiguous()                # [hkv, d, nk]
    vv = v.double().permute(1, 0, 2).contiguous()                # [hkv, nk, d]
    o = torch.empty((nq, hq, d), dtype=torch.float64, device=q.device)
    lse = torch.empty((hq, nq), dtype=torch.float64, device=q.device)
    step = max(1, min(nq, (1 << 27) // max(1, hq * nk)))
    for r in range(0, nq, step):
        n = min(step, nq - r)
        keys = nk - nq + r + n
        qq = q[r:r + n].double().view(n, hkv, g, d).permute(1, 2, 0, 3).reshape(hkv, g * n, d)
        sc = torch.matmul(qq, kt[:, :, :keys].contiguous()).view(hkv, g, n, keys) * scale
        row = torch.arange(n, device=q.device) + (nk - nq + r)
        sc.masked_fill_(torch.arange(keys, device=q.device)[None, :] > row[:, None],
                        float("-inf"))
        z = torch.logsumexp(sc, dim=-1)
        sc.sub_(z[..., None]).exp_()
        out = torch.matmul(sc.view(hkv, g * n, keys), vv[:, :keys].contiguous())
        o[r:r + n] = out.view(hkv, g, n, d).permute(2, 0, 1, 3).reshape(n, hq, d)
        lse[:, r:r + n] = z.reshape(hq, n)
    return o, lse


def _gather(cache, table_row, n):
    """Keys 0..n-1 of one sequence from the paged cache, [n, hkv, d]."""
    hkv, d = cache.shape[1], cache.shape[3]
    x = cache[table_row[:(n + BLOCK - 1) // BLOCK].long()]
    return x.permute(0, 2, 1, 3).reshape(-1, hkv, d)[:n]


def _put(cache, slots, rows):
    """`rows` [t, hkv, d] at their slots."""
    cache[(slots // BLOCK).long(), :, (slots % BLOCK).long()] = rows
    return cache


def _exact_decode(s):
    if s["case"].get("append", True):
        last = s["kv"] - 1
        page = s["table"].gather(1, (last // BLOCK).long()[:, None])[:, 0]
        slots = page * BLOCK + last % BLOCK
        _put(s["k_cache"], slots, s["k_new"])
        _put(s["v_cache"], slots, s["v_new"])
    o = [_attn64(s["q"][i:i + 1], _gather(s["k_cache"], s["table"][i], n),
                 _gather(s["v_cache"], s["table"][i], n), s["scale"])[0]
         for i, n in enumerate(_kv_lens(s["case"]))]
    return torch.cat(o)


def _exact_gemm(w):
    """x W with W[k, n] = (q - z) s; word 8a + 4b + c of a (group, column)
    holds k-octet 4c + 2b + a, code j at bits 4 (j / 2) + 16 (j % 2)."""
    g, n, _ = w["qw"].shape
    words = w["qw"].view(g, n, 2, 2, 4).permute(0, 1, 4, 3, 2).reshape(g, n, BLOCK, 1)
    shift = torch.tensor([4 * (j // 2) + 16 * (j % 2) for j in range(8)], device="cuda",
                         dtype=torch.int32)
    q = ((words >> shift) & 15).reshape(g, n, GROUP).permute(0, 2, 1).double()
    wt = (q - w["zp"].double()[:, None]) * w["sc"].double()[:, None]
    return torch.matmul(w["x"].double(), wt.reshape(g * GROUP, n).contiguous())


def exact(c, seed):
    if c["kind"] == "step":
        rng = _Draw(seed)
        out = []
        for _ in range(c["layers"]):
            a, lin = _prepare_decode(c, rng), _prepare_linear(c, rng)
            o = _exact_decode(a)
            out.append(dict(o=o, k_cache=a["k_cache"], v_cache=a["v_cache"],
                            y=[_exact_gemm(w) for w in lin]))
        return out
    s = prepare(c, seed)
    if c["kind"] == "linear":
        return [_exact_gemm(w) for w in s["linear"]]
    if c["kind"] == "decode":
        o = _exact_decode(s)
        return dict(o=o, k_cache=s["k_cache"], v_cache=s["v_cache"]) if c["append"] \
            else dict(o=o)
    if c["kind"] == "mixed":
        o = [_exact_decode(dict(s, case=dict(c, append=False)))]
        at = c["rows"]
        for i, p in enumerate(_prior_lens(c)):
            n, row = p + c["piece_len"], c["rows"] + i
            o.append(_attn64(s["q"][at:at + c["piece_len"]],
                             _gather(s["k_cache"], s["table"][row], n),
                             _gather(s["v_cache"], s["table"][row], n), s["scale"])[0])
            at += c["piece_len"]
        return dict(o=torch.cat(o))
    o, lse, at = [], [], 0
    for n in _prompt_lens(c):
        a, z = _attn64(s["q"][at:at + n], s["k"][at:at + n], s["v"][at:at + n], s["scale"])
        o.append(a)
        lse.append(z)
        at += n
    out = dict(o=torch.cat(o))
    if c["lse"]:
        out["lse"] = torch.cat(lse, dim=1)
    if c["write"] != "none":
        out.update(k_cache=_put(s["k_cache"], s["slots"], s["k"]),
                   v_cache=_put(s["v_cache"], s["slots"], s["v"]))
    return out
