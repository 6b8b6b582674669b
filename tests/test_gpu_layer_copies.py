"""laserkv_compress_layer where its score kernel copies the blocks' protected rows (ranges of at least three chunks of 128
keys, at least a fifth of the kept rows protected, at most twelve plane tiles) and where the selection does: either side of
each condition, short last blocks that leave ranges empty, values of a stride that 32-bit offsets do not reach."""
import pytest
import torch

from paper_2602_02199_amd import synth
from tests.test_gpu_layer import check_layer
from tests.test_gpu_parity import DEV

pytestmark = pytest.mark.gpu


def workload(name, s_block, n_div, l_ctx, tables=7, bits=11, head_dim=128, dtype="bf16", heads=2, window=5):
    return synth.shrink(synth.WORKLOADS["tiny"], index=53, name=f"copies-{name}", n_q_heads=2 * heads, n_kv_heads=heads, head_dim=head_dim,
                        dtype=dtype, l_ctx=l_ctx, s_block=s_block, window=window, n_div=n_div, lsh_tables=tables, lsh_bits=bits,
                        needles_per_block=2, outlier_channels=2)


# few groups: a block's keys are cut into sixteen ranges
@pytest.mark.parametrize("n_div", [2, 4, 9, 10, 11])
@pytest.mark.parametrize("s_block", [6112, 6144, 6177])  # ranges of 384 keys (the last one shorter), of 384, of 416
def test_divisors_and_ranges(n_div, s_block):
    check_layer(workload(f"{n_div}-{s_block}", s_block, n_div, 2 * s_block - 1000))


@pytest.mark.parametrize("last", [5, 384, 385, 700])  # tokens of the last block: one range, one, two, two
def test_short_last_block(last):
    check_layer(workload(f"last{last}", 6144, 4, 6144 + last))


@pytest.mark.parametrize("tables,bits", [(8, 8), (32, 12), (24, 16), (25, 16)])  # 2, 12, 12 and 13 plane tiles
@pytest.mark.parametrize("dtype,head_dim", [("bf16", 128), ("bf16", 64), ("f32", 64)])
def test_plane_tiles_and_rows(tables, bits, dtype, head_dim):
    check_layer(workload(f"{tables}x{bits}-{dtype}{head_dim}", 6144, 4, 9000, tables, bits, head_dim, dtype, heads=1))


def test_values_of_a_long_stride():
    wl = workload("stride", 6144, 4, 8000, heads=1)
    pitch = (1 << 31) // wl.s_block // 2 // 8 * 8 + 8  # elements: a block's values span 2 GiB
    wide = torch.empty(1, wl.l_ctx, pitch, dtype=torch.bfloat16, device=DEV)

    def mutate(data):
        view = wide[:, :, :wl.head_dim]
        view.copy_(data["v"])
        data["v"] = view

    check_layer(wl, mutate=mutate, with_oracle=False)
