"""laserkv_compress_layer where its statistics kernel takes the window rows' codes in one workgroup per group (as many groups
as compute units): sets of tables that fill tiles of hyperplanes or not, waves that share rows and split a set, sixteen-bit
codes that go out eight at a time or one by one, cells of every width, bins that hold all rows."""
import pytest

from paper_2602_02199_amd import synth
from tests.test_gpu_layer import check_layer

pytestmark = pytest.mark.gpu


def workload(group, window, tables, bits, head_dim=128, dtype="bf16"):
    return synth.shrink(synth.WORKLOADS["tiny"], index=54, name=f"codes-{group}x{window}-{tables}x{bits}-{dtype}{head_dim}",
                        n_q_heads=8 * group, n_kv_heads=8, head_dim=head_dim, dtype=dtype, l_ctx=32 * 72 - 5, s_block=72, window=window,
                        n_div=4, lsh_tables=tables, lsh_bits=bits, needles_per_block=2, outlier_channels=2)


@pytest.mark.parametrize("group,window", [(1, 5), (4, 64), (8, 64)])  # waves that share rows: 8, 2, 1
@pytest.mark.parametrize("tables,bits", [(32, 12), (31, 12), (16, 10), (32, 16), (30, 16), (29, 16), (32, 13), (40, 1), (31, 5), (2, 11)])
def test_sets_of_tables(group, window, tables, bits):
    check_layer(workload(group, window, tables, bits))


@pytest.mark.parametrize("dtype,head_dim", [("bf16", 64), ("f32", 64)])
@pytest.mark.parametrize("tables,bits", [(32, 12), (32, 16)])
def test_types(dtype, head_dim, tables, bits):
    check_layer(workload(4, 40, tables, bits, head_dim, dtype))


@pytest.mark.parametrize("tables,bits", [(32, 12), (32, 11), (16, 10), (8, 3)])  # cells of 4, 8, 16 and 16 bits
def test_equal_window_rows(tables, bits):
    def mutate(data):
        data["q_win"][:] = data["q_win"][:, :1, :1]

    check_layer(workload(8, 64, tables, bits), mutate=mutate)


# Key codes in octets of tables: one octet, which half of the lanes write; an odd number of them; through the counting kernel
# whole octets at a time (32 groups and more share a card) and table by table (two groups).
@pytest.mark.parametrize("tables,bits", [(8, 16), (24, 14), (24, 13)])
@pytest.mark.parametrize("heads", [1, 8])
def test_octets_of_key_codes(tables, bits, heads):
    check_layer(synth.shrink(workload(4, 24, tables, bits), name=f"octets-{heads}-{tables}x{bits}", n_q_heads=4 * heads, n_kv_heads=heads,
                             l_ctx=(32 if heads > 1 else 2) * 72 - 5))
