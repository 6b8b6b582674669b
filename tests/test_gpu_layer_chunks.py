"""laserkv_compress_layer where its score kernel changes from complete chunks of 128 keys (products beside the probabilities
of the step before) to masked ones, for one, two and four row tiles and one to four plane tiles per wave: the kept sets
against the block-by-block loop and the oracle."""
import pytest

from paper_2602_02199_amd import synth
from tests.test_gpu_layer import check_layer, layer_plan

pytestmark = pytest.mark.gpu

ROWS = {3: (4, 24), 4: (4, 32), 5: (4, 40), 8: (4, 64), 9: (4, 66), 16: (4, 128)}  # row tiles: query heads per KV head, window


@pytest.mark.parametrize("row_tiles", sorted(ROWS))
@pytest.mark.parametrize("tables,bits", [(12, 8), (16, 10), (32, 12), (29, 16)])  # 96, 160, 384 and 464 hyperplanes
@pytest.mark.parametrize("head_dim", [128, 64])
# ranges of 64 keys, whose tiles are all masked ones; of 416: three complete chunks and a part of one
@pytest.mark.parametrize("heads,s_block,l_ctx,keys", [(2, 640, 1664, 64), (1, 6177, 11354, 416)])
def test_row_and_plane_tiles(heads, s_block, l_ctx, keys, row_tiles, tables, bits, head_dim):
    g, w = ROWS[row_tiles]
    wl = synth.shrink(synth.WORKLOADS["tiny"], index=51, name=f"rows{row_tiles}-{tables}x{bits}-{head_dim}-{keys}", n_q_heads=heads * g,
                      n_kv_heads=heads, head_dim=head_dim, dtype="bf16", l_ctx=l_ctx, s_block=s_block, window=w, n_div=4,
                      lsh_tables=tables, lsh_bits=bits, needles_per_block=2, outlier_channels=2)
    assert layer_plan(wl)["score_keys"] == keys
    check_layer(wl)


# As many groups as compute units: a block is one range.
@pytest.mark.parametrize("beyond", [-1, 0, 1, 127])  # of the last row that every window row sees, over two whole chunks
@pytest.mark.parametrize("dtype,head_dim", [("bf16", 128), ("f32", 64)])
def test_blocks_around_whole_chunks(beyond, dtype, head_dim):
    w = 33
    s = 256 + w + beyond
    wl = synth.shrink(synth.WORKLOADS["tiny"], index=52, name=f"chunks{beyond}-{dtype}", n_q_heads=32, n_kv_heads=8,
                      head_dim=head_dim, dtype=dtype, l_ctx=32 * s - 40, s_block=s, window=w, n_div=4, lsh_tables=16,
                      lsh_bits=10, needles_per_block=2, outlier_channels=2)
    assert layer_plan(wl)["score_ranges"] == 1
    check_layer(wl)


@pytest.mark.parametrize("tables,bits", [(13, 10), (16, 10), (29, 9), (24, 12)])  # 5 and 9 plane tiles, the last with a few planes or 32
@pytest.mark.parametrize("dtype,head_dim", [("bf16", 128), ("bf16", 64), ("f32", 64)])
# few keys a range: masked tiles; one range of 700 keys a block: five complete chunks and a part of one
@pytest.mark.parametrize("heads,n_blocks,s_block", [(2, 3, 640), (8, 32, 700)])
def test_one_plane_tile_more_than_whole_rounds(heads, n_blocks, s_block, tables, bits, dtype, head_dim):
    """The last tile is shared out over the key tiles of a complete chunk."""
    wl = synth.shrink(synth.WORKLOADS["tiny"], index=53, name=f"spread-{tables}x{bits}-{dtype}{head_dim}-{s_block}", n_q_heads=4 * heads,
                      n_kv_heads=heads, head_dim=head_dim, dtype=dtype, l_ctx=n_blocks * s_block - 256, s_block=s_block, window=40,
                      n_div=4, lsh_tables=tables, lsh_bits=bits, needles_per_block=2, outlier_channels=2)
    plan = layer_plan(wl)
    assert plan["score_keys"] == 64 if heads == 2 else plan["score_ranges"] == 1
    check_layer(wl)
