"""Attention of many rows over long ranges of cache rows (more than 320, before a block 512: the ring of four stages of 64
keys, entered with a whole number of 128 keys) against float64: ranges around those numbers, rows that leave waves of a
workgroup without a tile or share a middle tile, causal blocks behind the ring, and logits that outgrow the fixed reference
inside and behind it.

256 KV heads of one row group each, so that a workgroup takes all keys.  Bounds: probabilities rounded to bf16 (2^-8 each)
against weights in float64, plus 4e-6 for 32-bit sums; a row's log-sum-exp 1e-4."""
import pytest
import torch

from paper_2602_02199_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
H = 256
HEADS = [0, 1, 100, 255]


def run(d, n_q, n, s_t=0, late=(), H=H):
    gen = torch.Generator(device=DEV).manual_seed(n + 3 * n_q + d)
    q = torch.randn(H, n_q, d, generator=gen, device=DEV).bfloat16()
    k = torch.randn(H, n + s_t, d, generator=gen, device=DEV)
    v = torch.randn(H, n + s_t, d, generator=gen, device=DEV).bfloat16()
    for pos in late:  # a key along one query: a logit of 2^190 and more above the first keys'
        k[:, pos] = q[:, n_q // 2].float() * (200.0 * d ** 0.5 / q[:, n_q // 2].float().pow(2).sum(-1, keepdim=True))
    k = k.bfloat16()
    lib = binding.LaserKV(H, H, d, "bf16", 16, 10, max_block=max(s_t, n_q, 256), max_window=n_q, max_ctx_keys=0)
    out = torch.full((H, n_q, d), float("nan"), device=DEV)
    lse = torch.full((H, n_q), float("nan"), device=DEV)
    kc, vc = k[:, :n].contiguous(), v[:, :n].contiguous()
    if s_t:
        ws = torch.empty(lib.laserkv_attend_block_workspace_bytes(n_q, n, s_t), dtype=torch.uint8, device=DEV)
        lib.laserkv_attend_block(q, kc, vc, k[:, n:].contiguous(), v[:, n:].contiguous(), cache_len=n, block_pos0=n, out=out,
                                 out_lse=lse, workspace=ws)
    else:
        ws = torch.empty(lib.laserkv_attend_workspace_bytes(n_q, n), dtype=torch.uint8, device=DEV)
        lib.laserkv_attend_cache(q, kc, vc, cache_len=n, out=out, out_lse=lse, workspace=ws)
    worst = 0.0
    for h in [h for h in HEADS if h < H]:
        x = q[h].double() @ k[h].double().t().contiguous() / d ** 0.5
        if s_t:
            i, j = torch.arange(s_t, device=DEV), torch.arange(n_q, device=DEV)
            x[:, n:] = x[:, n:].masked_fill(i[None, :] > (s_t - n_q + j)[:, None], float("-inf"))
        w = torch.softmax(x, dim=-1)
        vd = v[h].double()
        bound = (2.0 ** -8 + 4e-6) * (w @ vd.abs())
        err = (out[h].double() - w @ vd).abs()
        worst = max(worst, float((err / bound).max()))
        # element by element: a maximum over values that are not numbers compares with nothing
        assert bool((err <= bound).all()), f"output of head {h}: {int((~(err <= bound)).sum())} values beyond the bound, the largest {worst:.3f} times it"
        off = (lse[h].double() - torch.logsumexp(x, dim=-1)).abs()
        assert bool((off <= 1e-4 + 1e-6 * torch.logsumexp(x, dim=-1).abs()).all()), f"log-sum-exp of head {h}: {float(off.max())}"
    print(f"[ring d{d} rows {n_q} cache {n} block {s_t} late {late}] error / bound {worst:.3f}", flush=True)


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("n_q", [129, 160, 192, 256])  # five to eight row tiles: a middle tile, absent pairs
@pytest.mark.parametrize("n", [321, 383, 384, 385, 511, 512, 513, 575, 639, 640, 641, 767, 768, 1000, 1151])
def test_cache_lengths(d, n_q, n):
    run(d, n_q, n)


# a head's second workgroup holds the middle tile and stays out of the ring that the first one takes
@pytest.mark.parametrize("n_q", [288, 352])
@pytest.mark.parametrize("n", [321, 640, 1000])
def test_a_middle_tile_beside_the_ring(n_q, n):
    run(128, n_q, n)


# few heads: key ranges are cut, 32 a head on 256 compute units; about 320 keys each, where a range's references become fixed
# and the launch changes to the instance with the ring, not at the same length, and longer ones
@pytest.mark.parametrize("n_q", [160, 256])
@pytest.mark.parametrize("n", [10239, 10240, 10250, 10271, 10272, 10300, 11300, 15900, 16383, 16384, 16385, 16500, 17000, 17408])
def test_cut_ranges(n_q, n):
    run(128, n_q, n, H=8)


@pytest.mark.parametrize("n_q,n,s_t", [(160, 400, 160), (256, 513, 256), (200, 700, 300), (224, 1024, 224)])
def test_causal_block_behind_the_cache(n_q, n, s_t):
    run(128, n_q, n, s_t)


@pytest.mark.parametrize("late", [(100,), (383,), (500,), (639,), (645,), (200, 641)])
@pytest.mark.parametrize("n_q", [192, 160])
def test_logits_that_outgrow_the_reference(n_q, late):
    run(128, n_q, 650, 0, late)


# the same in ranges that are cut (eight heads, 32 ranges a head), each against a reference of its own, and at d = 64
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("n_q", [160, 256])
@pytest.mark.parametrize("late", [(15000,), (10, 9000, 15999)])
def test_logits_that_outgrow_the_reference_of_a_cut_range(d, n_q, late):
    run(d, n_q, 16000, 0, late, H=8)


# cut ranges of cache rows and the block's keys: all of them long, references overflowing in the last too
@pytest.mark.parametrize("late", [(), (7, 15900)])
def test_cut_ranges_before_a_block(late):
    run(128, 1024, 16000, 1024, late, H=8)


# window rows before a long block: 300 cache rows a split on average, ranges of up to 832 and none
def test_cache_rows_of_ranges_that_a_long_block_makes_longer():
    run(128, 1024, 2400, 4096, H=8)
    run(128, 1024, 2400, 4096, (1500,), H=8)
