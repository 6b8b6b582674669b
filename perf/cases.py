"""The work a user of this library has it do, as a list of cases: one pass each through the public entry points
(the block loop of a prefill engine, one block by itself, attention over the compacted cache, the block's own
attention), from one small block to a whole 128k-token layer.

Inputs are drawn on the GPU from the seed alone and have the structure of `paper_2602_02199_amd/synth.py`: Gaussian
filler, a few outlier key channels, needle keys turned towards a window query, per-key scales and repeated keys
where a case asks for them.
"""
from __future__ import annotations

import math

import torch

from paper_2602_02199_amd import binding, synth
from paper_2602_02199_amd.driver import LayerCompressor

DEV = "cuda:0"


def _layer(name, kind, heads, head_dim, dtype, l_ctx, s_block, window, n_div, tables, bits, sigma=0.0, dup=0.0, needles=8):
    return dict(name=name, kind=kind, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=head_dim, dtype=dtype, l_ctx=l_ctx,
                s_block=s_block, window=window, n_div=n_div, tables=tables, bits=bits, sigma=sigma, dup=dup, needles=needles)


def _attend(name, kind, heads, head_dim, dtype, n_q, cache_len, s_t=0):
    return dict(name=name, kind=kind, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=head_dim, dtype=dtype, n_q=n_q,
                cache_len=cache_len, s_t=s_t)


def listed():
    return [
        # One block of the small fp32 configuration, compressed by one call in the middle of a context: what
        # launches and latencies cost.
        _layer("block-tiny", "block", (4, 2), 64, "f32", 4096, 512, 32, 4, 8, 8, needles=2),
        # One layer of a 16k-token prefill: eight blocks, the engine's prepared call list.
        _layer("layer-16k", "layer", (32, 8), 128, "bf16", 16384, 2048, 64, 4, 16, 10),
        # A context whose length is no multiple of the block, through the unprepared loop (selection and append as two
        # calls per block; the last block is short).
        _layer("layer-64k-ragged", "loop", (32, 8), 128, "bf16", 64749, 2048, 64, 8, 16, 10, needles=2),
        # One layer of a 128k-token prefill: the benchmark's workload.
        _layer("layer-128k", "layer", (32, 8), 128, "bf16", 131072, 4096, 128, 8, 32, 12, sigma=0.5),
        # The same layer in an engine whose attention hands over the window rows' log-sum-exp.
        _layer("layer-128k-complete", "complete", (32, 8), 128, "bf16", 131072, 4096, 128, 8, 32, 12, sigma=0.5),
        # Groups of eight query heads, long blocks, 16-bit hash codes, repeated keys.
        _layer("layer-gqa8-128k", "layer", (64, 8), 128, "bf16", 131072, 8192, 64, 16, 32, 16, dup=0.05),
        # One layer of a 16k-token prefill with the library's attention in front of every selection.
        _layer("model-16k", "model", (32, 8), 128, "bf16", 16384, 2048, 64, 4, 16, 10),
        # A decoding step after a 16k-token prefill (its kept rows and a few generated ones).
        _attend("decode-16k", "attend", (32, 8), 128, "bf16", 1, 7301),
        # A decoding step after a 128k-token prefill.
        _attend("decode-128k", "attend", (32, 8), 128, "bf16", 1, 63520),
        # The window rows of a block over the cache of a 128k-token context.
        _attend("window-128k", "attend", (32, 8), 128, "bf16", 128, 63520),
        # Their normaliser alone, over the cache of a 64k-token context.
        _attend("normaliser-64k", "normaliser", (32, 8), 128, "bf16", 64, 31681),
        # The last block of a 128k-token prefill: all of its rows over the cache and, causally, over the block.
        _attend("prefill-128k", "prefill", (32, 8), 128, "bf16", 4096, 61535, 4096),
    ]


# The model shapes that drawn cases take: heads, head dimension, type, hash tables and bits, longest window.
_SHAPES = [
    ((4, 2), 64, "f32", 8, 8, 32),
    ((16, 4), 128, "bf16", 16, 10, 64),
    ((32, 8), 128, "bf16", 16, 10, 64),
    ((32, 8), 128, "bf16", 32, 12, 128),
    ((64, 8), 128, "bf16", 32, 16, 64),
]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["block", "layer", "loop", "complete", "model", "attend", "attend", "normaliser", "prefill"])
    heads, d, dtype, tables, bits, w_max = rng.choice(_SHAPES)
    small = dtype == "f32"
    if kind in ("attend", "normaliser", "prefill"):
        n = _log(rng, 64, 1900 if small else 63520)
        if kind == "prefill":
            s = _log(rng, 256, 512 if small else (2048 if heads[0] > 32 else 4096))
            # the whole block, or its window rows alone
            c = _attend("", kind, heads, d, dtype, s if rng.random() < 0.7 else rng.randint(16, w_max), min(n, 61535), s)
        elif kind == "attend":
            # decoding (one query, sometimes a few), or the window rows of the next block
            n_q = rng.choice([1, 1, 1, rng.randint(2, 8), rng.randint(16, w_max), rng.randint(16, w_max)])
            c = _attend("", kind, heads, d, dtype, n_q, n)
        else:
            c = _attend("", kind, heads, d, dtype, rng.randint(16, w_max), n)
    else:
        s = _log(rng, 256, 512 if small else (2048 if kind == "model" else 8192))
        most = (8192 if heads[0] > 32 else 24576) if kind == "model" else 131072
        n_blocks = 1 if kind == "block" else _log(rng, 1, min(32, max(1, most // s)))
        l_ctx = s * max(n_blocks, 8) if kind == "block" else s * n_blocks
        if kind in ("loop", "model") and n_blocks > 1:
            l_ctx -= rng.randint(0, s // 2)  # a short last block
        c = _layer("", kind, heads, d, dtype, l_ctx, s, rng.randint(16, w_max), rng.choice([4, 8, 16]), tables, bits,
                   sigma=rng.choice([0.0, 0.5]), dup=rng.choice([0.0, 0.05]), needles=rng.choice([2, 8]))
    del c["name"]
    return c


# ---- inputs ----
def _dt(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _redirect(old, target, cos):
    """Vectors with old's norms whose cosine to `target` is `cos`; the rest is old's part orthogonal to target."""
    t = target / target.norm(dim=-1, keepdim=True)
    perp = old - (old * t).sum(-1, keepdim=True) * t
    new = cos * t + (1.0 - cos * cos) ** 0.5 * perp / perp.norm(dim=-1, keepdim=True)
    return new * old.norm(dim=-1, keepdim=True)


def _slots(gen, shape, lo, hi):
    """One random position in each of shape[-1] equal parts of [lo, hi): distinct, ascending."""
    n = shape[-1]
    u = torch.rand(shape, generator=gen, device=DEV)
    return (lo + (torch.arange(n, device=DEV) + u) * ((hi - lo) / n)).long().clamp_(max=hi - 1)


def _layer_inputs(case, seed, n_tok, n_blocks, n_protect):
    """planes [L*K, d], q_win [blocks, H_q, W, d], k and v [H_kv, n_tok, d]."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    hq, hkv, d, s, w = case["n_q_heads"], case["n_kv_heads"], case["head_dim"], case["s_block"], case["window"]
    randn = lambda *sh: torch.randn(*sh, generator=gen, device=DEV)
    planes = randn(case["tables"] * case["bits"], d)
    q = randn(n_blocks, hq, w, d)
    k = randn(hkv, n_tok, d)
    v = randn(hkv, n_tok, d)
    if d == 128:
        k[:, :, torch.randperm(d, generator=gen, device=DEV)[:4]] *= 8.0
    whole = n_tok // s
    lo, hi = n_protect, s - n_protect
    first = torch.arange(whole, device=DEV)[:, None, None] * s
    head = torch.arange(hkv, device=DEV)[None, :, None]
    if whole and hi - lo > case["needles"]:
        sh = (whole, hkv, case["needles"])
        pos = first + _slots(gen, sh, lo, hi)
        gi = torch.randint(0, hq // hkv, sh, generator=gen, device=DEV)
        ji = torch.randint(0, w, sh, generator=gen, device=DEV)
        tgt = q[torch.arange(whole, device=DEV)[:, None, None], head * (hq // hkv) + gi, ji]
        k[head, pos] = _redirect(k[head, pos], tgt, 0.9)
    if case["sigma"]:
        k *= torch.exp(case["sigma"] * randn(hkv, n_tok, 1))
    n_dup = int(case["dup"] * (hi - lo))
    if whole and n_dup:
        sh = (whole, hkv, n_dup)
        dst = _slots(gen, sh, lo + 1, hi)
        src = (torch.rand(sh, generator=gen, device=DEV) * dst).long().clamp_(max=s - 1)
        copies = k[head, first + torch.minimum(src, dst - 1)]
        near = _redirect(randn(*copies.shape) * copies.norm(dim=-1, keepdim=True) / d ** 0.5, copies, 0.99)
        k[head, first + dst] = torch.where((torch.arange(n_dup, device=DEV) < n_dup // 2)[None, None, :, None], copies, near)
    dt = _dt(case)
    return dict(planes=planes.to(dt), q_win=q.to(dt), k=k.to(dt), v=v.to(dt))


def _complete_lse(case, data, n_blocks, n_local):
    """Every window row's log-sum-exp over the look-back keys and the block keys it sees, per block."""
    hq, hkv, d, s, w = case["n_q_heads"], case["n_kv_heads"], case["head_dim"], case["s_block"], case["window"]
    hidden = torch.arange(s, device=DEV)[None, :] > (s - w + torch.arange(w, device=DEV))[:, None]
    out = []
    for t in range(n_blocks):
        lo = t * s
        first = max(lo - n_local, 0) if t else lo
        keys = data["k"][:, first:lo + s].float().transpose(1, 2).contiguous()
        logits = torch.matmul(data["q_win"][t].float().view(hkv, -1, d), keys) / d ** 0.5
        logits = logits.view(hkv, hq // hkv, w, -1)
        logits[..., keys.shape[2] - s:].masked_fill_(hidden, float("-inf"))
        out.append(torch.logsumexp(logits, dim=-1).reshape(hq, w).contiguous())
    return out


def _attend_inputs(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    hq, hkv, d, n = case["n_q_heads"], case["n_kv_heads"], case["head_dim"], case["cache_len"] + case["s_t"]
    q = torch.randn(hq, case["n_q"], d, generator=gen, device=DEV)
    k = torch.randn(hkv, n, d, generator=gen, device=DEV)
    v = torch.randn(hkv, n, d, generator=gen, device=DEV)
    k[:, :, torch.randperm(d, generator=gen, device=DEV)[:4]] *= 8.0
    # some keys of every head are turned towards a query: a few rows are peaked
    pos = _slots(gen, (hkv, 8), 0, n)
    head = torch.arange(hkv, device=DEV)[:, None]
    gi = torch.randint(0, hq // hkv, (hkv, 8), generator=gen, device=DEV)
    ji = torch.randint(0, case["n_q"], (hkv, 8), generator=gen, device=DEV)
    k[head, pos] = _redirect(k[head, pos], q[head * (hq // hkv) + gi, ji], 0.9)
    dt = _dt(case)
    return q.to(dt), k.to(dt), v.to(dt)


def _workload(case):
    return synth.Workload("case", 0, case["n_q_heads"], case["n_kv_heads"], case["head_dim"], case["dtype"], case["l_ctx"],
                          case["s_block"], case["window"], case["n_div"], case["tables"], case["bits"])


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("attend", "normaliser", "prefill"):
        q, k, v = _attend_inputs(case, seed)
        n, s_t, n_q = case["cache_len"], case["s_t"], case["n_q"]
        lib = binding.LaserKV(case["n_q_heads"], case["n_kv_heads"], case["head_dim"], case["dtype"], 16, 10,
                              max_block=max(s_t, n_q, 256), max_window=min(n_q, 128), max_ctx_keys=0)
        size = lib.laserkv_attend_block_workspace_bytes(n_q, n, s_t) if kind == "prefill" else lib.laserkv_attend_workspace_bytes(n_q, n)
        st = dict(kind=kind, lib=lib, q=q, n=n, workspace=torch.empty(size, dtype=torch.uint8, device=DEV),
                  k_cache=k[:, :n].contiguous(), v_cache=v[:, :n].contiguous(),
                  out=None if kind == "normaliser" else torch.empty(q.shape, dtype=torch.float32, device=DEV),
                  lse=torch.empty(q.shape[:2], dtype=torch.float32, device=DEV))
        if kind == "prefill":
            st.update(k_blk=k[:, n:].contiguous(), v_blk=v[:, n:].contiguous())
        return st

    wl = _workload(case)
    if kind == "block":
        # the second block of its context: the cache holds the first block's kept rows, whose last ones are looked back at
        comp = LayerCompressor(wl, DEV, max_blocks=2)
        na, nl, ke, kl = comp.parts
        data = _layer_inputs(case, seed, 2 * wl.s_block, 2, na)
        comp.run_layer(data, n_blocks=1)
        s, b = wl.s_block, comp.cache_len
        return dict(kind=kind, comp=comp, q=data["q_win"][1], k=data["k"][:, s:], v=data["v"][:, s:],
                    ctx=comp.k_cache[:, b - nl:b] if nl else None, planes=data["planes"],
                    args=dict(block_pos0=s, n_anchor=na, n_local=nl, k_exact=ke, k_lsh=kl, keep_idx=comp.keep,
                              k_cache=comp.k_cache, v_cache=comp.v_cache, cache_pos=comp.cache_pos, cache_len=b))
    comp = LayerCompressor(wl, DEV)
    nb = wl.n_blocks
    data = _layer_inputs(case, seed, wl.l_ctx, nb, comp.parts[0])
    st = dict(kind=kind, comp=comp, data=data)
    if kind in ("layer", "complete"):
        lse = _complete_lse(case, data, nb, comp.parts[1]) if kind == "complete" else None
        st.update(lse=lse, plan=comp.plan_layer(data, row_lse_complete=lse))
    elif kind == "model":
        gen = torch.Generator(device=DEV).manual_seed(seed + 1)
        blocks = []
        for t in range(nb):
            s_t = min(wl.s_block, wl.l_ctx - t * wl.s_block)
            q = torch.randn(wl.n_q_heads, s_t, wl.head_dim, generator=gen, device=DEV).to(_dt(case))
            q[:, s_t - wl.window:] = data["q_win"][t]
            blocks.append(q)
        size = max(comp.lib.laserkv_attend_block_workspace_bytes(q.shape[1], t * sum(comp.parts), q.shape[1]) for t, q in enumerate(blocks))
        st.update(q_blocks=blocks, out=torch.empty(wl.n_q_heads, wl.s_block, wl.head_dim, dtype=torch.float32, device=DEV),
                  out_lse=torch.empty(wl.n_q_heads, wl.s_block, dtype=torch.float32, device=DEV),
                  lse_win=torch.empty(wl.n_q_heads, wl.window, dtype=torch.float32, device=DEV),
                  workspace=torch.empty(size, dtype=torch.uint8, device=DEV),
                  last=min(wl.s_block, wl.l_ctx - (nb - 1) * wl.s_block))
    return st


def _bits(t):
    """A cache as whole numbers: its rows are copies of input rows, byte for byte."""
    return t.view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32)


def run(st):
    kind = st["kind"]
    if kind == "attend":
        st["lib"].laserkv_attend_cache(st["q"], st["k_cache"], st["v_cache"], cache_len=st["n"], out=st["out"], out_lse=st["lse"],
                                       workspace=st["workspace"])
        return st["out"], st["lse"]
    if kind == "normaliser":
        st["lib"].laserkv_attend_cache(st["q"], st["k_cache"], st["v_cache"], cache_len=st["n"], out=None, out_lse=st["lse"],
                                       workspace=st["workspace"])
        return st["lse"]
    if kind == "prefill":
        st["lib"].laserkv_attend_block(st["q"], st["k_cache"], st["v_cache"], st["k_blk"], st["v_blk"], cache_len=st["n"],
                                       block_pos0=st["n"], out=st["out"], out_lse=st["lse"], workspace=st["workspace"])
        return st["out"], st["lse"]
    comp = st["comp"]
    more = ()
    if kind == "block":
        comp.lib.laserkv_compress_block(st["q"], st["k"], st["v"], st["ctx"], st["planes"], **st["args"])
        more = (comp.keep,)
    elif kind == "loop":
        comp.run_layer(st["data"])
    elif kind == "model":
        comp.run_layer_with_attention(st["data"], st["q_blocks"], st["out"], st["out_lse"], st["lse_win"], st["workspace"])
        rows = st["out_lse"].shape[0] * st["last"]  # a short last block uses the start of the buffers
        more = (st["out"].view(-1)[:rows * st["out"].shape[2]], st["out_lse"].view(-1)[:rows], st["lse_win"])
    else:
        comp.run_plan(st["plan"])
    n = comp.cache_len if kind == "loop" or kind == "model" else comp.cap
    return (comp.cache_pos[:, :n], _bits(comp.k_cache)[:, :n], _bits(comp.v_cache)[:, :n]) + more


def work(case):
    """Bytes: every input read once, every output written once.  Operations: the contractions with the keys, once each
    (the logits of the window or block rows, the projections on the hyperplanes, the weighted values)."""
    kind, hq, hkv, d = case["kind"], case["n_q_heads"], case["n_kv_heads"], case["head_dim"]
    es = 4 if case["dtype"] == "f32" else 2
    if kind in ("attend", "normaliser", "prefill"):
        n, s_t, n_q = case["cache_len"], case["s_t"], case["n_q"]
        both = 1 if kind == "normaliser" else 2
        pairs = n_q * n + sum(min(s_t, s_t - n_q + j + 1) for j in range(n_q)) if s_t else n_q * n
        out = hq * n_q * 4 * ((d if both == 2 else 0) + 1)
        return dict(bytes=both * hkv * (n + s_t) * d * es + hq * n_q * d * es + out, flops=2 * both * hq * pairs * d)
    s, w, lk = case["s_block"], case["window"], case["tables"] * case["bits"]
    l_ctx = s if kind == "block" else case["l_ctx"]
    budget = 2 * s * case["l_ctx"] // (4 * (s + case["l_ctx"]))
    nbytes = flops = kept_before = 0
    for lo in range(0, l_ctx, s):
        s_t = min(s, l_ctx - lo)
        b = min(budget, s_t)
        nbytes += hkv * s_t * d * es + hq * w * d * es + lk * d * es  # keys, window rows, hyperplanes
        nbytes += hkv * b * (3 * d * es + 4 + 8)                      # kept values read, kept rows, indices, positions written
        flops += 2 * d * hq * w * s_t + 2 * d * lk * hkv * s_t
        if kind == "complete":
            nbytes += hq * w * 4
        if kind == "model":
            # the block's attention over the cache so far and, causally, over the block (keys already counted)
            nbytes += hkv * (2 * kept_before + s_t - b) * d * es + hq * (s_t - w) * d * es + hq * s_t * 4 * (d + 1)
            flops += 4 * hq * d * (s_t * kept_before + s_t * (s_t + 1) // 2)
        kept_before += b
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    """Kept positions, indices and rows are whole numbers; a token whose score lies at the selection's threshold within
    the rounding of a 32-bit sum may give way to its neighbour, and the rows between the two then move by one.
    Attention in bf16 rounds its probabilities to bf16; in fp32, and for the normaliser, sums are 32-bit."""
    kind = case["kind"]
    if kind in ("attend", "prefill", "model"):
        fp = dict(rel=1e-2, max=0.1) if case["dtype"] == "bf16" else dict(rel=2e-5, max=2e-4)
        return dict(fp, differ=0.01) if kind == "model" else fp
    if kind == "normaliser":
        return dict(rel=1e-5, max=1e-4)
    return dict(rel=0.0, differ=0.01)
