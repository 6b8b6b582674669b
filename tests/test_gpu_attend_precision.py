"""How far attention is from 64 bits beyond what rounding probabilities to bf16 (relative error 2^-8 each) allows.

Where a row's reference follows its maximum (decoding; in the kernel of many rows the block's own keys, and the cache's
where a key range holds at most 320 of them), the largest probability is a power of two and exact, so the output
sum w_i v_i is off by at most 2^-8 sum over the OTHER keys of w_i |v_i|: far below 2^-8 of it for a row that one key
dominates.  32-bit sums add at most 4e-6 of sum w_i |v_i|.
"""
import numpy as np
import pytest
import torch

from oracle import laserkv_oracle as O
from paper_2602_02199_amd import binding
from tests.test_gpu_attend import DEV, f64, make_inputs, run_attend, say
from tests.test_gpu_attend_block import run_block

pytestmark = pytest.mark.gpu


def weights(q, keys, hidden=None):
    """Softmax weights [rows, keys] of one query head in float64."""
    x = f64(q) @ f64(keys).T / q.shape[-1] ** 0.5
    if hidden is not None:
        x[hidden] = -np.inf
    w = np.exp(x - x.max(axis=1, keepdims=True))
    return w / w.sum(axis=1, keepdims=True)


def against_bound(out, w, v, first_exact=0):
    """One head: out [rows, d], w [rows, keys], v [keys, d]; rows whose largest weight is at first_exact or later have it exact."""
    v = f64(v)
    slack = 4e-6 * (w @ np.abs(v))
    top = w.argmax(axis=1)
    rounded = w.copy()
    rounded[np.arange(len(w)), top] *= top < first_exact
    bound = 2.0 ** -8 * (rounded @ np.abs(v)) + slack
    return float((np.abs(out - w @ v) / bound).max()), float(w.max())


def verdict(results, label):
    ratio = max(r for r, _ in results)
    say(f"[precision {label}] largest weights up to {max(w for _, w in results):.5f}, error / bound up to {ratio:.3f}")
    assert all(r <= 1.0 for r, _ in results), f"{label}: {ratio:.2f} times the bound"


@pytest.mark.parametrize("g,n_q,d", [(1, 1, 128), (4, 1, 128), (4, 2, 64), (8, 1, 64)])
def test_decoding_rows_that_one_key_dominates(g, n_q, d):
    """Every key far below two: the later of them, less than 2^8 above the earlier, takes nearly all weight."""
    # 32 key splits; the eight waves of a split take tiles of 2048 / d keys in turn, 4 keys per group of lanes
    h_kv, tiles = 8, 8 * 2048 // d
    per_split = tiles + 32
    n = 32 * per_split - 17
    gen = torch.Generator().manual_seed(7 + g)
    lib = binding.LaserKV(g * h_kv, h_kv, d, "bf16", 8, 8, max_block=64, max_window=8, max_ctx_keys=0)
    u = torch.randn(h_kv, d, generator=gen)
    u /= u.norm(dim=-1, keepdim=True)
    q = (u[:, None, None] * (8.0 + 0.05 * torch.rand(h_kv, g, n_q, 1, generator=gen))).expand(h_kv, g, n_q, d).reshape(g * h_kv, n_q, d)
    k = 0.1 * torch.randn(h_kv, n, d, generator=gen) - u[:, None] * (30.0 * d ** 0.5 / 8.0)
    for h in range(h_kv):
        first = per_split * (h + 3) + 5
        k[h, first] = 0.0
        k[h, first + tiles] = u[h] * ((4.0 + 0.17 * h) * d ** 0.5 / 8.0)  # the same group of lanes, a tile later
    v = torch.randn(h_kv, n, d, generator=gen)
    q, k, v = (t.to(torch.bfloat16).contiguous() for t in (q, k, v))
    out, lse = run_attend(lib, q.to(DEV), k.to(DEV), v.to(DEV), n)
    verdict([against_bound(out[i], weights(q[i], k[i // g]), v[i // g]) for i in range(g * h_kv)], f"decode {g}x{n_q} d {d}")
    lib.close()


ROWS = [
    # H_q, H_kv, d, cache_len, s_t
    (8, 2, 128, 0, 300),
    (4, 1, 128, 700, 300),
    (4, 1, 64, 90, 413),
    (64, 64, 128, 500, 1040),
]


@pytest.mark.parametrize("case", ROWS, ids=[f"{c[0]}-heads-{c[3]}-{c[4]}" for c in ROWS])
def test_rows_of_a_block_that_one_of_its_keys_dominates(case):
    """Rows between diffuse and peaked as they come, and sixteen per KV head with a key of the block that takes nearly all."""
    h_q, h_kv, d, n, s_t = case
    g = h_q // h_kv
    q, kk, vv = make_inputs(h_q, h_kv, d, s_t, n + s_t, "bf16", seed=900 + s_t, needles=False)
    q, kk = q.float(), kk.float()
    for h in range(h_kv):
        for t in range(16):
            j = (t * s_t // 16) | 3
            qq = q[h * g + t % g, j]
            kk[h, n + min(t * s_t // 16 + 1, j)] = qq * ((12.0 + 0.31 * t) * d ** 0.5 / float(qq @ qq))
    q, kk = q.to(torch.bfloat16), kk.to(torch.bfloat16)
    lib = binding.LaserKV(h_q, h_kv, d, "bf16", 8, 8, max_block=s_t, max_window=32, max_ctx_keys=0)
    kc, vc = kk[:, :max(n, 1)].contiguous(), vv[:, :max(n, 1)].contiguous()
    kb, vb = kk[:, n:].contiguous(), vv[:, n:].contiguous()
    out, _ = run_block(lib, q.to(DEV), kc.to(DEV), vc.to(DEV), n, kb.to(DEV), vb.to(DEV), 0, 0)
    hidden = np.arange(n + s_t)[None, :] > n + np.arange(s_t)[:, None]
    verdict([against_bound(out[i], weights(q[i], kk[i // g], hidden), vv[i // g], n) for i in range(0, h_q, 3)], f"block {s_t} after {n}")
    lib.close()


@pytest.mark.parametrize("h_q,h_kv,d,n_q,n", [(16, 4, 128, 64, 3000), (4, 1, 64, 40, 1900), (8, 2, 128, 300, 320)])
def test_rows_over_a_short_cache_that_one_key_dominates(h_q, h_kv, d, n_q, n):
    """Window rows whose key ranges hold few cache rows, and a block's rows over a small cache alone: the reference follows."""
    g = h_q // h_kv
    q, k, v = make_inputs(h_q, h_kv, d, n_q, n, "bf16", seed=n)
    lib = binding.LaserKV(h_q, h_kv, d, "bf16", 8, 8, max_block=n_q, max_window=128, max_ctx_keys=0)
    out, _ = run_block(lib, q.to(DEV), k.to(DEV), v.to(DEV), n, k[:, :0].to(DEV), v[:, :0].to(DEV), 0, 0)
    verdict([against_bound(out[i], weights(q[i], k[i // g]), v[i // g]) for i in range(h_q)], f"rows {n_q} over {n}")
    lib.close()


@pytest.mark.parametrize("route", ["normaliser", "rows-split", "rows-whole"])
def test_log_sum_exp_of_diffuse_rows(route):
    """Values below 16: the last addition and the store round by at most half of 2^-20 each (mean 2.4e-7 and, times ln 2,
    1.7e-7, together 3e-7), the logarithm of a number below one adds little, and so do sums of at most a thousand terms per
    lane: a mean error of 4.5e-7 leaves half as much again."""
    h_q, h_kv, d = 32, 8, 128
    n_q, n = (2048, 2000) if route == "rows-whole" else (40, 9000)
    q, k, v = make_inputs(h_q, h_kv, d, n_q, n, "bf16", seed=66, needles=False)
    lib = binding.LaserKV(h_q, h_kv, d, "bf16", 8, 8, max_block=n_q, max_window=64, max_ctx_keys=0)
    if route == "rows-whole":
        assert lib.laserkv_attend_block_workspace_bytes(n_q, n, 0) == 256  # workgroups that see all keys of their rows
        _, lse = run_block(lib, q.to(DEV), k.to(DEV), v.to(DEV), n, k[:, :0].to(DEV), v[:, :0].to(DEV), 0, 0)
    else:
        _, lse = run_attend(lib, q.to(DEV), k.to(DEV), v.to(DEV), n, lse_only=route == "normaliser")
    err = []
    for hq in range(0, h_q, 3):
        x = f64(q[hq, :256]) @ f64(k[hq // (h_q // h_kv)]).T / d ** 0.5
        m = x.max(axis=1)
        want = m + np.log(np.exp(x - m[:, None]).sum(axis=1))
        err.append(np.abs(lse[hq, :256] - want)[want < 16.0])
    err = np.concatenate(err)
    say(f"[precision lse {route}] mean error {err.mean():.2e}, max {err.max():.2e}")
    assert err.mean() <= 4.5e-7
    lib.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [1, 40, 4500])
def test_decoding_row_whose_logits_all_overflow_to_minus_infinity(dtype, n):
    """As every other attention kernel: zero and -inf for that row, the other heads untouched."""
    h_q, h_kv, d = 8, 2, 64
    q, k, v = make_inputs(h_q, h_kv, d, 1, n, dtype, seed=11, needles=False)
    q[3], k[0, :, 0] = 0.0, -1.0e30
    q[:4, :, 0] = 0.0
    q[3, 0, 0] = 1.0e30
    lib = binding.LaserKV(h_q, h_kv, d, dtype, 8, 8, max_block=64, max_window=8, max_ctx_keys=0)
    out, lse = run_attend(lib, q.to(DEV), k.to(DEV), v.to(DEV), n)
    assert not out[3].any() and np.isneginf(lse[3]).all()
    o_out, o_lse = O.attend_cache(f64(q), f64(k), f64(v), n)
    rest = [0, 1, 2, 4, 5, 6, 7]
    assert np.abs(out[rest] - o_out[rest]).max() <= (1e-5 if dtype == "f32" else 2e-2) * 5 and np.abs(lse[rest] - o_lse[rest]).max() <= 1e-4
    lib.close()
