"""laserkv_compress_layer with the window rows' complete log-sum-exp from outside: layer_codes_kernel takes the rows' codes (with
its own statistics the layer's statistics kernel does) and one launch scores.  Codes of every cell width and of 16 bits, groups
that share their tables out and groups that do not, few rows and many, bins that hold all rows."""
import numpy as np
import pytest
import torch

from oracle import laserkv_oracle as O
from paper_2602_02199_amd import synth
from paper_2602_02199_amd.driver import LayerCompressor
from tests.test_gpu_layer import layer_plan, oracle_positions
from tests.test_gpu_parity import DEV, f64, say, to_dev

pytestmark = pytest.mark.gpu


def complete_lse(wl, data, B):
    """Per block the natural-log sum of every window row's exponentials over its look-back keys and the block keys it sees."""
    k, out, prev = f64(data["k"]), [], 0
    for t in range(wl.n_blocks):
        lo, hi = t * wl.s_block, min((t + 1) * wl.s_block, k.shape[1])
        q = f64(data["q_win"][t])
        logits = np.einsum("hgwd,hkd->hgwk", q.reshape(wl.n_kv_heads, wl.group, *q.shape[1:]), k[:, lo - prev:hi]) / wl.head_dim ** 0.5
        at = np.arange(lo - prev, hi)[None, :] - lo
        logits = np.where(at <= hi - lo - wl.window + np.arange(wl.window)[:, None], logits, -np.inf)
        top = logits.max(-1, keepdims=True)
        lse = np.log(np.exp(logits - top).sum(-1)) + top[..., 0]
        out.append(torch.tensor(lse.reshape(wl.n_q_heads, wl.window), dtype=torch.float32, device=DEV))
        prev = O.partition(B, wl.n_div, wl.alpha, hi - lo)[1]
    return out


def compress(wl, dev, lse):
    """One call with the statistics of every block; the compressor and the rows it kept."""
    comp = LayerCompressor(wl, DEV)
    table = torch.tensor([t.data_ptr() for t in lse], dtype=torch.int64, device=DEV)
    fn, args, n = comp._layer_call(dev, wl.n_blocks, table)
    comp.lib.laserkv_profile_begin()
    comp.lib._check(fn(*args, comp.lib._stream(None)))
    torch.cuda.synchronize()
    launches = {k: v[1] for k, v in comp.lib.laserkv_profile_end().items() if v[1]}
    assert launches["single"] == 1 and launches["select"] == 1 and "sweep1" not in launches and "sweep2" not in launches, launches
    return comp, n


def check_complete(wl, mutate=None, tol=2e-3):
    B = O.budget(wl.s_block, wl.l_ctx, wl.r_num, wl.r_den)
    data = synth.make_layer(wl, 1, O.partition(B, wl.n_div, wl.alpha, wl.s_block)[0])
    if mutate is not None:
        mutate(data)
    dev, lse = to_dev(data), complete_lse(wl, data, B)
    comp, n = compress(wl, dev, lse)
    pos = comp.cache_pos[:, :n]
    assert bool((pos[:, 1:] > pos[:, :-1]).all()) and bool((comp.cache_pos[:, n:] == -1).all())
    idx = pos[:, :, None].expand(-1, -1, wl.head_dim)
    assert torch.equal(torch.gather(dev["k"], 1, idx), comp.k_cache[:, :n])
    assert torch.equal(torch.gather(dev["v"], 1, idx), comp.v_cache[:, :n])
    want, got = oracle_positions(wl, data, B, wl.n_blocks), pos.cpu().numpy()
    off = sum(len(set(got[h].tolist()) - set(want[h].tolist())) for h in range(wl.n_kv_heads))
    say(f"[complete {wl.name}] rows {n}, tokens kept that the oracle does not keep: {off}")
    assert want.shape == got.shape and off <= tol * n * wl.n_kv_heads


def workload(group, window, tables, bits, head_dim=128, dtype="bf16", heads=8, n_blocks=32):
    # as many groups as compute units with 8 heads and 32 blocks: each takes all its tables; few groups share them out.  Three
    # quarters of the recalled tokens are chosen by their counts.
    return synth.shrink(synth.WORKLOADS["tiny"], index=55, name=f"{heads}x{n_blocks}-{group}x{window}-{tables}x{bits}-{dtype}{head_dim}",
                        n_q_heads=heads * group, n_kv_heads=heads, head_dim=head_dim, dtype=dtype, l_ctx=n_blocks * 72 - 5, s_block=72,
                        window=window, n_div=4, alpha=0.25, lsh_tables=tables, lsh_bits=bits, needles_per_block=2, outlier_channels=2)


CODES = [(32, 12), (31, 12), (16, 10), (32, 11), (32, 16), (30, 16), (32, 13), (40, 1), (31, 5), (2, 11)]


@pytest.mark.parametrize("heads,n_blocks", [(8, 32), (2, 3)])
@pytest.mark.parametrize("tables,bits", CODES)
def test_codes(tables, bits, heads, n_blocks):
    check_complete(workload(4, 40, tables, bits, heads=heads, n_blocks=n_blocks))


@pytest.mark.parametrize("group,window", [(1, 5), (1, 32), (8, 64)])  # part of a row tile, one, sixteen
@pytest.mark.parametrize("tables,bits", [(32, 12), (32, 16)])
def test_rows(group, window, tables, bits):
    check_complete(workload(group, window, tables, bits, n_blocks=5))


@pytest.mark.parametrize("dtype,head_dim", [("bf16", 64), ("f32", 64)])
@pytest.mark.parametrize("tables,bits", [(32, 12), (16, 10), (32, 16)])
def test_types(dtype, head_dim, tables, bits):
    check_complete(workload(4, 40, tables, bits, head_dim, dtype, n_blocks=5))


@pytest.mark.parametrize("heads,n_blocks", [(8, 32), (2, 3)])
@pytest.mark.parametrize("tables,bits", [(32, 12), (32, 11), (16, 10), (8, 3)])  # cells of 4, 8, 16 and 16 bits
def test_equal_window_rows(tables, bits, heads, n_blocks):
    def mutate(data):
        data["q_win"][:] = data["q_win"][:, :1, :1]

    check_complete(workload(8, 64, tables, bits, heads=heads, n_blocks=n_blocks), mutate=mutate)


@pytest.mark.parametrize("s_block,l_ctx", [(640, 1664), (2048, 5000)])
def test_longer_blocks(s_block, l_ctx):
    check_complete(synth.shrink(workload(4, 40, 16, 10), name=f"long-{s_block}", s_block=s_block, l_ctx=l_ctx))


# the score kernel copies the protected rows: ten groups of sixteen ranges with a whole and a short last block, one range a block
@pytest.mark.parametrize("dtype,head_dim", [("bf16", 128), ("bf16", 64), ("f32", 64)])
@pytest.mark.parametrize("heads,n_blocks,s_block,last", [(2, 5, 6144, 6144), (2, 5, 6144, 385), (8, 32, 512, 500)])
@pytest.mark.parametrize("tables,bits", [(16, 10), (32, 12)])
def test_copies_of_protected_rows(heads, n_blocks, s_block, last, dtype, head_dim, tables, bits):
    wl = synth.shrink(workload(2, 20, tables, bits, head_dim, dtype, heads, n_blocks), name=f"copies-{s_block}-{last}-{dtype}{head_dim}",
                      s_block=s_block, l_ctx=(n_blocks - 1) * s_block + last, r_num=1, r_den=2)
    assert layer_plan(wl, complete=True)["copied_rows"] > 0
    check_complete(wl)


def test_the_contexts_setting_holds_for_every_block():
    wl = workload(4, 40, 16, 10, n_blocks=5)
    B = O.budget(wl.s_block, wl.l_ctx, wl.r_num, wl.r_den)
    data = synth.make_layer(wl, 1, O.partition(B, wl.n_div, wl.alpha, wl.s_block)[0])
    dev, lse = to_dev(data), complete_lse(wl, data, B)
    want, n = compress(wl, dev, [lse[2]] * wl.n_blocks)
    comp = LayerCompressor(wl, DEV)
    comp.lib.laserkv_set_row_lse_complete(lse[2])
    assert comp.run_layer(dev) == n
    comp.lib.laserkv_set_row_lse_complete(None)
    assert torch.equal(comp.cache_pos, want.cache_pos) and torch.equal(comp.k_cache, want.k_cache) and torch.equal(comp.v_cache, want.v_cache)
    assert comp.run_layer(dev) == n  # and statistics of its own again
    own = LayerCompressor(wl, DEV)
    own.run_layer(dev)
    assert torch.equal(comp.cache_pos, own.cache_pos)
