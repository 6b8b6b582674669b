"""Row statistics (laserkv_rowstats.h) through the normaliser-only attention: key ranges around the chunks of 128 (64 in
fp32 at d = 128) and the ring of four stages, 1 to 512 rows (eight to one wave over different key tiles), and logits that
outgrow the reference in the first, an inner and the last chunk of a key range.

Bound: a logit is a sum of d products in 32 bits, off by at most d 2^-24 sum |q||k| / sqrt(d) of the keys that carry
weight; scaling, subtracting a reference and the logarithm round at the size of their results (2^-23 each, headroom of
24 included)."""
import numpy as np
import pytest
import torch

from paper_2602_02199_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
H_KV = 32  # eight key ranges on 256 compute units


def check(dtype, d, g, n_q, n, late=()):
    gen = torch.Generator(device=DEV).manual_seed(n + 7 * n_q + d)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q = torch.randn(g * H_KV, n_q, d, generator=gen, device=DEV).to(dt)
    k = torch.randn(H_KV, n, d, generator=gen, device=DEV)
    for pos in late:  # a key far along the first query of every group: a logit of 2^150 or more above the others
        first = q.view(H_KV, g * n_q, d)[:, 0].float()
        k[:, pos] = first * (160.0 * d ** 0.5 / first.pow(2).sum(-1, keepdim=True))
    k = k.to(dt)
    v = torch.zeros_like(k)
    lib = binding.LaserKV(g * H_KV, H_KV, d, dtype, 16, 10, max_block=1024, max_window=min(n_q, 128), max_ctx_keys=0)
    lse = torch.full((g * H_KV, n_q), float("nan"), device=DEV)
    work = torch.empty(lib.laserkv_attend_workspace_bytes(n_q, n), dtype=torch.uint8, device=DEV)
    lib.laserkv_attend_cache(q, k, v, cache_len=n, out=None, out_lse=lse, workspace=work)
    rows = q.double().view(H_KV, g * n_q, d)
    kt = k.double().transpose(1, 2).contiguous()
    x = torch.matmul(rows, kt) / d ** 0.5
    want = torch.logsumexp(x, dim=-1)
    weight = torch.softmax(x, dim=-1)
    size = (weight * torch.matmul(rows.abs(), kt.abs())).sum(-1) / d ** 0.5
    bound = d * 2.0 ** -24 * size + 4 * 2.0 ** -23 * (want.abs() + 24.0)
    err = (lse.double().view(H_KV, -1) - want).abs()
    worst = float((err / bound).max())
    print(f"[rowstats {dtype} d{d} rows {g * n_q} keys {n} late {late}] error / bound {worst:.3f}", flush=True)
    assert np.isfinite(worst) and worst <= 1.0


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("g,n_q", [(1, 9), (2, 32), (4, 32), (4, 64), (4, 128), (8, 70)])
@pytest.mark.parametrize("n", [1, 257, 1024, 1031, 4099, 9000])
def test_key_ranges(dtype, d, g, n_q, n):
    check(dtype, d, g, n_q, n)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 128)])
@pytest.mark.parametrize("g,n_q", [(1, 9), (4, 32), (4, 64), (4, 128)])
@pytest.mark.parametrize("late", [(40,), (700,), (1151,), (8999,), (300, 420, 1100)])
def test_logits_that_outgrow_the_reference(dtype, d, g, n_q, late):
    check(dtype, d, g, n_q, 9000, late)  # ranges of 1152 keys


# ranges of 1536 keys and more: whole chunks in the middle take a loop of their own (one wave per row, and two)
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("g,n_q", [(4, 33), (4, 64), (4, 128), (8, 70)])
@pytest.mark.parametrize("n,late", [(12287, ()), (12288, ()), (12289, ()), (13100, ()), (17000, ()), (13000, (650,)), (13000, (200, 1000, 1600, 8000)),
                                    (17000, (383, 384, 1500, 2120))])
def test_long_ranges(d, g, n_q, n, late):
    check("bf16", d, g, n_q, n, late)
