"""laserkv_compress_layer where its score kernel copies the blocks' protected rows and where the selection does: either side of
each condition (ranges of three chunks of 128 keys, a fifth of the kept rows protected, twelve plane tiles, workgroups for five
eighths of the chip, rows for a range), short last blocks that leave ranges empty, values of a stride that 32-bit offsets do not
reach."""
import pytest
import torch

from oracle import laserkv_oracle as O
from paper_2602_02199_amd import synth
from tests.test_gpu_layer import check_layer, layer_plan
from tests.test_gpu_parity import DEV

pytestmark = pytest.mark.gpu


def workload(name, s_block, n_div, last=5096, tables=7, bits=11, head_dim=128, dtype="bf16", heads=2, n_blocks=5, window=5, r=(1, 2)):
    return synth.shrink(synth.WORKLOADS["tiny"], index=53, name=f"copies-{name}", n_q_heads=2 * heads, n_kv_heads=heads, head_dim=head_dim,
                        dtype=dtype, l_ctx=(n_blocks - 1) * s_block + last, s_block=s_block, window=window, n_div=n_div, lsh_tables=tables,
                        lsh_bits=bits, needles_per_block=2, outlier_channels=2, r_num=r[0], r_den=r[1])


def protected(wl):
    """Anchors and local rows of all blocks, per KV head."""
    B = O.budget(wl.s_block, wl.l_ctx, wl.r_num, wl.r_den)
    lens = [min(wl.s_block, wl.l_ctx - lo) for lo in range(0, wl.l_ctx, wl.s_block)]
    return sum(sum(O.partition(B, wl.n_div, wl.alpha, s)[:2]) for s in lens)


def check(wl, copied, **kw):
    assert layer_plan(wl)["copied_rows"] == (protected(wl) if copied else 0)
    check_layer(wl, **kw)


# ten groups: a block's keys are cut into sixteen ranges, 160 workgroups
@pytest.mark.parametrize("n_div", [2, 4, 9, 10, 11])  # a fifth of the kept rows and more: up to nine, and ten where it divides them
@pytest.mark.parametrize("s_block", [5600, 6112, 6144, 6400])  # ranges of 352 keys, of 384 (the last one shorter), of 384, of 416
def test_divisors_and_ranges(n_div, s_block):
    wl = workload(f"{n_div}-{s_block}", s_block, n_div)
    fifth = n_div < 10 or (n_div == 10 and O.budget(s_block, wl.l_ctx, wl.r_num, wl.r_den) % 10 == 0)
    check(wl, s_block > 5632 and fifth)


@pytest.mark.parametrize("last", [5, 384, 385, 700])  # tokens of the last block: one range, one, two, two
def test_short_last_block(last):
    check(workload(f"last{last}", 6144, 4, last), True)


@pytest.mark.parametrize("tables,bits", [(8, 8), (32, 12), (24, 16), (25, 16)])  # 2, 12, 12 and 13 plane tiles
@pytest.mark.parametrize("dtype,head_dim", [("bf16", 128), ("bf16", 64), ("f32", 64)])
def test_plane_tiles_and_rows(tables, bits, dtype, head_dim):
    check(workload(f"{tables}x{bits}-{dtype}{head_dim}", 6144, 4, tables=tables, bits=bits, head_dim=head_dim, dtype=dtype), tables * bits <= 384)


@pytest.mark.parametrize("heads,n_blocks,copied", [(3, 3, False), (2, 5, True)])  # 144 workgroups, 160
def test_few_workgroups(heads, n_blocks, copied):
    check(workload(f"few{heads}x{n_blocks}", 6144, 4, heads=heads, n_blocks=n_blocks), copied)


# 63 rows of 256 bytes for a range, 64; 127 of 128 bytes, 128
@pytest.mark.parametrize("head_dim,r_num,copied", [(128, 1981, False), (128, 1985, True), (64, 3993, False), (64, 3996, True)])
def test_rows_of_a_range(head_dim, r_num, copied):
    check(workload(f"rows{head_dim}-{r_num}", 6144, 4, 5144, head_dim=head_dim, r=(r_num, 10000)), copied)


# 256 groups: a block is one range, of 46 protected rows, of 48
@pytest.mark.parametrize("r_num,copied", [(250, False), (260, True)])
@pytest.mark.parametrize("dtype,head_dim", [("bf16", 128), ("bf16", 64), ("f32", 64)])
def test_rows_of_the_only_range(r_num, copied, dtype, head_dim):
    wl = workload(f"only{r_num}-{dtype}{head_dim}", 384, 8, 384, head_dim=head_dim, dtype=dtype, heads=8, n_blocks=32, r=(r_num, 1000))
    assert layer_plan(wl)["score_ranges"] == 1
    check(wl, copied)


def test_values_of_a_long_stride():
    wl = workload("stride", 6144, 4)
    pitch = (1 << 31) // wl.s_block // 2 // 8 * 8 + 8  # elements: a block's values span 2 GiB
    wide = torch.empty(2, wl.l_ctx, pitch, dtype=torch.bfloat16, device=DEV)

    def mutate(data):
        view = wide[:, :, :wl.head_dim]
        view.copy_(data["v"])
        data["v"] = view

    check(wl, True, mutate=mutate, with_oracle=False)  # (the plan is that of rows that follow each other)
