"""laserkv_compress_layer where its score kernel changes from complete chunks of 128 keys (products beside the probabilities
of the step before) to masked ones, for one, two and four row tiles and one to four plane tiles per wave: the kept sets
against the block-by-block loop and the oracle."""
import pytest

from paper_2602_02199_amd import synth
from tests.test_gpu_layer import check_layer

pytestmark = pytest.mark.gpu

ROWS = {3: (4, 24), 4: (4, 32), 5: (4, 40), 8: (4, 64), 9: (4, 66), 16: (4, 128)}  # row tiles: query heads per KV head, window


@pytest.mark.parametrize("row_tiles", sorted(ROWS))
@pytest.mark.parametrize("tables,bits", [(12, 8), (16, 10), (32, 12), (29, 16)])  # 96, 160, 384 and 464 hyperplanes
@pytest.mark.parametrize("head_dim", [128, 64])
def test_row_and_plane_tiles(row_tiles, tables, bits, head_dim):
    g, w = ROWS[row_tiles]
    check_layer(synth.shrink(synth.WORKLOADS["tiny"], index=51, name=f"rows{row_tiles}-{tables}x{bits}-{head_dim}", n_q_heads=2 * g,
                             n_kv_heads=2, head_dim=head_dim, dtype="bf16", l_ctx=1664, s_block=640, window=w, n_div=4,
                             lsh_tables=tables, lsh_bits=bits, needles_per_block=2, outlier_channels=2))


@pytest.mark.parametrize("beyond", [-1, 0, 1, 127])  # of the last row that every window row sees, over two whole chunks
@pytest.mark.parametrize("dtype,head_dim", [("bf16", 128), ("f32", 64)])
def test_blocks_around_whole_chunks(beyond, dtype, head_dim):
    w = 33
    s = 256 + w + beyond
    check_layer(synth.shrink(synth.WORKLOADS["tiny"], index=52, name=f"chunks{beyond}-{dtype}", n_q_heads=8, n_kv_heads=2,
                             head_dim=head_dim, dtype=dtype, l_ctx=3 * s - 40, s_block=s, window=w, n_div=4, lsh_tables=16,
                             lsh_bits=10, needles_per_block=2, outlier_channels=2))


@pytest.mark.parametrize("tables,bits", [(13, 10), (16, 10), (29, 9), (24, 12)])  # 5 and 9 plane tiles, the last with a few planes or 32
@pytest.mark.parametrize("dtype,head_dim", [("bf16", 128), ("f32", 64)])
def test_one_plane_tile_more_than_whole_rounds(tables, bits, dtype, head_dim):
    """The last tile is shared out over the key tiles of a complete chunk."""
    check_layer(synth.shrink(synth.WORKLOADS["tiny"], index=53, name=f"spread-{tables}x{bits}-{dtype}", n_q_heads=8, n_kv_heads=2,
                             head_dim=head_dim, dtype=dtype, l_ctx=1664, s_block=640, window=40, n_div=4, lsh_tables=tables,
                             lsh_bits=bits, needles_per_block=2, outlier_channels=2))
