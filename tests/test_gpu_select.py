"""The selection kernel by itself (laserkv_select_consensus hands it scores and counts) where its intervals of values and
its thread counts change, against sorting: block lengths around 256, 512 and 1024 threads, scores that tie, vanish, spread
over more than the 16 octaves of the first interval (denormals among them) or lie 30 orders above the rest, counts below and
above one part each.  Whole numbers: exact.  The layer's launch has its own thread counts: against the block loop."""
import numpy as np
import pytest
import torch

from paper_2602_02199_amd import binding, synth
from tests.test_gpu_layer import check_layer

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def scores_of(kind, n, rng):
    if kind == "spread":
        s = np.exp(rng.normal(-8.0, 1.0, n))
    elif kind == "zeros":
        s = np.where(rng.random(n) < 0.9, 0.0, 1e-30)
    elif kind == "ties":
        s = rng.integers(1, 6, n) * 0.125
    elif kind == "wide":
        s = 10.0 ** rng.uniform(-44.0, 0.0, n)
    else:  # one far above
        s = rng.random(n)
        s[n // 2] = 1e30
    return s.astype(np.float32)


def counts_of(kind, n, rng):
    return {"few": rng.integers(0, 5, n), "below": rng.integers(0, 1024, n), "above": rng.integers(0, 50000, n),
            "equal": np.full(n, 7), "edge": rng.choice([0, 1023, 1024, 1025], n)}[kind].astype(np.int32)


def wanted(score, count, na, nl, ke, kl):
    n = len(score)
    cand = np.arange(na, n - nl)
    ex = cand[np.argsort(-score[cand].astype(np.float64), kind="stable")][:ke]
    rest = np.setdiff1d(cand, ex)
    ls = rest[np.argsort(-count[rest].astype(np.int64), kind="stable")][:kl]
    return np.sort(np.concatenate([np.arange(na), np.arange(n - nl, n), ex, ls]))


@pytest.mark.parametrize("n", [17, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 16384])
def test_against_sorting(n):
    lib = binding.LaserKV(2, 1, 64, "bf16", 8, 8, max_block=16384, max_window=8, max_ctx_keys=0)
    rng = np.random.default_rng(n)
    for sk in ("spread", "zeros", "ties", "wide", "above"):
        for ck in ("few", "below", "above", "equal", "edge"):
            score, count = scores_of(sk, n, rng), counts_of(ck, n, rng)
            b = max(n // 4, 4)
            na = nl = b // 8
            for ke in sorted({0, 1, (b - 2 * na) * 3 // 4, b - 2 * na}):
                kl = b - 2 * na - ke
                keep = torch.full((b,), -1, dtype=torch.int32, device=DEV)
                lib.laserkv_select_consensus(torch.from_numpy(score).to(DEV), torch.from_numpy(count).to(DEV), s_t=n, n_anchor=na,
                                             n_local=nl, k_exact=ke, k_lsh=kl, keep_idx=keep)
                got = keep.cpu().numpy()
                assert np.array_equal(got, wanted(score, count, na, nl, ke, kl)), f"{n} {sk} {ck} {ke}"


@pytest.mark.parametrize("s_block", [250, 512, 1000, 1025, 2048, 2100, 4096, 4100])
def test_layer_thread_counts(s_block):
    check_layer(synth.shrink(synth.WORKLOADS["llama8b-16k"], index=61, name=f"threads-{s_block}", l_ctx=2 * s_block + s_block // 2,
                             s_block=s_block, n_q_heads=8, n_kv_heads=2, needles_per_block=2), with_oracle=s_block <= 1025)


# where the interval of counts gets four, two and one counters per value and then parts of several values; few values share
# all positions, the threshold lies in the part that is not counted, above it, or at the largest
@pytest.mark.parametrize("top", [0, 1, 3, 254, 255, 256, 257, 510, 511, 512, 513, 1022, 1023, 1024, 1025, 2047, 2048])
@pytest.mark.parametrize("n", [300, 2000, 4096, 9000])
def test_counters_of_small_intervals(n, top):
    lib = binding.LaserKV(2, 1, 64, "bf16", 8, 8, max_block=16384, max_window=8, max_ctx_keys=0)
    rng = np.random.default_rng(n + top)
    b = n // 4
    na = nl = b // 8
    ke, kl = 3, b - 2 * na - 3
    for p_zero in (0.0, 0.5, 0.99):
        values = np.unique([1, top // 2, max(top - 1, 0), top])
        score = np.where(rng.random(n) < p_zero, 0.0, rng.integers(1, 4, n) * np.float32(0.1234567)).astype(np.float32)
        count = np.where(rng.random(n) < p_zero, 0, np.minimum(rng.choice(values, n), top)).astype(np.int32)
        count[n // 2] = top
        keep = torch.full((b,), -1, dtype=torch.int32, device=DEV)
        lib.laserkv_select_consensus(torch.from_numpy(score).to(DEV), torch.from_numpy(count).to(DEV), s_t=n, n_anchor=na,
                                     n_local=nl, k_exact=ke, k_lsh=kl, keep_idx=keep)
        assert np.array_equal(keep.cpu().numpy(), wanted(score, count, na, nl, ke, kl)), f"{n} {top} {p_zero}"
