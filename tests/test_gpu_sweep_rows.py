"""A single block's sweeps by row tiles (one to nine tiles of 32 window rows; up to four, the waves without a tile hash the
window rows), and the counts of one row group in one step (8, 16 and 32 tables) or table by table: every stage against the
oracle."""
import pytest

from paper_2602_02199_amd import synth
from tests.test_gpu_parity import run_and_check

pytestmark = pytest.mark.gpu


# window rows per KV head: query heads per KV head, window
ROWS = {9: (1, 9), 32: (4, 8), 33: (3, 11), 64: (2, 32), 96: (4, 24), 128: (4, 32), 129: (1, 129), 160: (4, 40), 256: (4, 64), 288: (4, 72)}


@pytest.mark.parametrize("rows", sorted(ROWS))
@pytest.mark.parametrize("dtype,head_dim", [("bf16", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("tables,bits", [(8, 8), (16, 10), (13, 9)])
def test_row_tiles(rows, dtype, head_dim, tables, bits):
    g, w = ROWS[rows]
    run_and_check(synth.shrink(synth.WORKLOADS["tiny"], index=71, name=f"rows{rows}-{dtype}-{head_dim}-{tables}x{bits}", n_q_heads=2 * g,
                               n_kv_heads=2, head_dim=head_dim, dtype=dtype, l_ctx=700, s_block=350, window=w, n_div=4,
                               lsh_tables=tables, lsh_bits=bits, needles_per_block=2, outlier_channels=2))
