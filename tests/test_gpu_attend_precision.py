"""How far attention is from 64 bits beyond what rounding probabilities to bf16 (relative error 2^-9 each) allows.

Weights w_i, values v_i, exact output o = sum w_i v_i.
  * weights normalised by the sum of the rounded probabilities (kernel of many rows): the output is a mean of the values
    with weights w_i (1 + e_i) / sum w_j (1 + e_j), |e_i| <= 2^-9, hence off by at most 2^-8 sum w_i |v_i - o|;
  * references that follow the maximum (decoding): the row's largest probability is exactly 1, the others are off by 2^-9
    each, hence at most 2^-9 sum over the others of w_i |v_i|.
Either is far below 2^-9 |o| for a row that one key dominates.  32-bit sums add at most 4e-6 of sum w_i |v_i|.
"""
import numpy as np
import pytest
import torch

from paper_2602_02199_amd import binding
from tests.test_gpu_attend import DEV, f64, make_inputs, run_attend, say

pytestmark = pytest.mark.gpu


def weights(q, keys, hidden=None):
    """Softmax weights [rows, keys] of one query head in float64."""
    x = f64(q) @ f64(keys).T / q.shape[-1] ** 0.5
    if hidden is not None:
        x[hidden] = -np.inf
    w = np.exp(x - x.max(axis=1, keepdims=True))
    return w / w.sum(axis=1, keepdims=True)


def against_bound(out, w, v, follows_maximum):
    """One head: out [rows, d], w [rows, keys], v [keys, d]."""
    v = f64(v)
    o = w @ v
    slack = 4e-6 * (w @ np.abs(v))
    if follows_maximum:
        others = w.copy()
        others[np.arange(len(w)), w.argmax(axis=1)] = 0.0
        bound = 2.0 ** -9 * (others @ np.abs(v)) + slack
    else:
        bound = 2.0 ** -8 * np.stack([w[r] @ np.abs(v - o[r]) for r in range(len(w))]) + slack
    return float((np.abs(out - o) / bound).max()), float(w.max())


def verdict(results, label):
    ratio = max(r for r, _ in results)
    say(f"[precision {label}] largest weights up to {max(w for _, w in results):.5f}, error / bound up to {ratio:.3f}")
    assert ratio <= 1.0, f"{label}: {ratio:.2f} times the bound"


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
    verdict([against_bound(out[i], weights(q[i], k[i // g]), v[i // g], True) for i in range(g * h_kv)], f"decode {g}x{n_q} d {d}")
    lib.close()
