"""The attention kernel for many query rows at the edges of its work split, against the oracle: odd numbers of row tiles
(two waves share the middle one from the start), tiles across the rows of two heads, ragged last tiles, pairs that join
inside a chunk, several key splits whose cuts fall into the cache and into the block, whole rounds of row groups followed
by an incomplete one that is cut by keys, blocks shorter than a chunk, and
logits that outgrow the fixed reference (the second pass with exact maxima) in either tile of a pair."""
import pytest
import torch

from paper_2602_02199_amd import binding
from tests.test_gpu_attend import DEV, make_inputs, say
from tests.test_gpu_attend_block import compare_block, run_block

pytestmark = pytest.mark.gpu

CASES = [
    # label, dtype, H_q, H_kv, d, n_q, cache_len, s_t, rows whose logits outgrow the reference
    ("five-tiles-ragged", "bf16", 6, 2, 128, 50, 333, 50, ()),
    ("seven-tiles", "bf16", 6, 2, 64, 70, 95, 131, ()),
    ("nine-tiles-no-cache", "bf16", 4, 1, 128, 72, 0, 72, ()),
    ("head-straddling-tiles", "bf16", 8, 1, 128, 145, 129, 145, ()),
    ("one-key-each", "bf16", 8, 1, 128, 33, 1, 33, ()),
    ("many-splits", "bf16", 4, 1, 128, 300, 5003, 300, ()),
    ("splits-in-the-block", "bf16", 4, 1, 64, 900, 40, 900, ()),
    ("f32-many-splits", "f32", 4, 1, 64, 130, 1111, 130, ()),
    ("f32-d128-joins", "f32", 4, 1, 128, 257, 65, 257, ()),
    ("whole-rounds-and-cut-rest", "bf16", 64, 64, 64, 1040, 600, 1040, ()),
    ("large-logits-early-row", "bf16", 4, 1, 128, 300, 700, 300, (3,)),
    ("large-logits-late-row", "bf16", 4, 1, 128, 300, 700, 300, (290,)),
    ("f32-large-logits", "f32", 4, 1, 64, 200, 300, 200, (5, 190)),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_attend_rows_edges(case):
    label, dtype, h_q, h_kv, d, n_q, n, s_t, hot = case
    say(f"[attend_rows {label}] {dtype} heads {h_q}/{h_kv} d {d} n_q {n_q} cache_len {n} s_t {s_t}")
    q, kk, vv = make_inputs(h_q, h_kv, d, n_q, n + s_t, dtype, seed=3000 + len(label))
    for j in hot:  # a cache key and the query's own block key along the query, far above its other logits
        kk[0, n - 40] = q[0, j] * 12.0
        kk[0, n + s_t - n_q + j] = q[0, j] * 25.0
    kc, vc, kb, vb = kk[:, :n].contiguous(), vv[:, :n].contiguous(), kk[:, n:].contiguous(), vv[:, n:].contiguous()
    if n == 0:
        kc = torch.zeros(h_kv, 1, d, dtype=kk.dtype)
        vc = torch.zeros(h_kv, 1, d, dtype=vv.dtype)
    bp, qp = 1000, 1000 + s_t - n_q
    lib = binding.LaserKV(h_q, h_kv, d, dtype, 8, 8, max_block=max(s_t, 32), max_window=32, max_ctx_keys=0)
    out, lse = run_block(lib, q.to(DEV), kc.to(DEV), vc.to(DEV), n, kb.to(DEV), vb.to(DEV), bp, qp)
    compare_block(out, lse, q, kc, vc, n, kb, vb, bp, qp, True, dtype, label)
    again = run_block(lib, q.to(DEV), kc.to(DEV), vc.to(DEV), n, kb.to(DEV), vb.to(DEV), bp, qp)
    assert (again[0] == out).all() and (again[1] == lse).all()
    lib.close()


def test_long_queries_of_many_heads_per_group():
    """32 query heads per KV head, 15000 queries each: row indices beyond the range of the 32-bit multiplier alone."""
    g, n_q, d, n, s_t = 32, 15000, 64, 40, 64
    q, kk, vv = make_inputs(g, 1, d, n_q, n + s_t, "bf16", seed=32)
    kc, vc, kb, vb = kk[:, :n].contiguous(), vv[:, :n].contiguous(), kk[:, n:].contiguous(), vv[:, n:].contiguous()
    wide = torch.zeros(g, n_q + 2, d, dtype=torch.bfloat16, device=DEV)
    wide[:, 1:1 + n_q] = q.to(DEV)
    lib = binding.LaserKV(g, 1, d, "bf16", 8, 8, max_block=n_q, max_window=32, max_ctx_keys=0)
    bp = 20000
    qp = bp + s_t - n_q
    out, lse = run_block(lib, wide[:, 1:1 + n_q], kc.to(DEV), vc.to(DEV), n, kb.to(DEV), vb.to(DEV), bp, qp)
    for j0, j1 in ((0, 2), (n_q // 2, n_q // 2 + 1), (n_q - s_t - 1, n_q - s_t + 2), (n_q - 3, n_q)):
        compare_block(out[:, j0:j1], lse[:, j0:j1], q[:, j0:j1], kc, vc, n, kb, vb, bp, qp + j0, True, "bf16", f"rows {j0}..{j1 - 1} of 32 heads")
    lib.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("growth", [90, 122, 137, 143, 150, 170])
def test_logits_far_above_the_first_tile(dtype, growth):
    """A cache key whose logit lies that far above the first tile's (in powers of two): within the sums' range, at its end
    and past it (the second pass), in split and in whole key ranges."""
    for g, n_q, n in ((4, 90, 3000), (32, 2048, 300)):
        q, kk, vv = make_inputs(g, 1, 64, n_q, n + 40, dtype, seed=growth, needles=False)
        for i, j in ((0, 5), (g - 1, n_q - 3)):
            qq = q[i, j].float()
            kk[0, n - 50 - 3 * i] = (qq * (growth / 1.4427 * 8.0 / float(qq @ qq))).to(kk.dtype)
        kc, vc, kb, vb = kk[:, :n].contiguous(), vv[:, :n].contiguous(), kk[:, n:].contiguous(), vv[:, n:].contiguous()
        lib = binding.LaserKV(g, 1, 64, dtype, 8, 8, max_block=n_q, max_window=32, max_ctx_keys=0)
        out, lse = run_block(lib, q.to(DEV), kc.to(DEV), vc.to(DEV), n, kb.to(DEV), vb.to(DEV), 5000, 5040 - n_q)
        for rows in (slice(0, 8), slice(n_q - 8, n_q)):
            compare_block(out[:, rows], lse[:, rows], q[:, rows], kc, vc, n, kb, vb, 5000, 5040 - n_q + rows.start, True, dtype,
                          f"growth {growth}, {g * n_q} rows from {rows.start}")
        lib.close()
