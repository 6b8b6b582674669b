"""The kernel of laserkv_attend_cache for few query rows (G * n_q <= 8) against the oracle: every row count it is built
for, both types and head dimensions, caches at the edges of its tiles and key splits; its counters over many launches."""
import pytest
import torch

from paper_2602_02199_amd import binding
from tests.test_gpu_attend import DEV, compare, make_inputs, run_attend, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("g,n_q", [(1, 1), (2, 1), (1, 3), (4, 1), (5, 1), (4, 2), (8, 1)])
def test_few_rows_against_oracle(dtype, d, g, n_q):
    h_kv = 2
    lib = binding.LaserKV(g * h_kv, h_kv, d, dtype, 8, 8, max_block=64, max_window=8, max_ctx_keys=0)
    for n in (1, 15, 33, 128, 129, 1000, 4097):
        say(f"[decode] {dtype} d {d} rows {g}x{n_q} cache {n}")
        q, k, v = make_inputs(g * h_kv, h_kv, d, n_q, n + 40, dtype, seed=100 * g + n)
        k[:, n:] = float("nan")  # rows past the length are never read
        v[:, n:] = float("nan")
        out, lse = run_attend(lib, q.to(DEV), k.to(DEV), v.to(DEV), n)
        compare(out, lse, q, k, v, n, dtype, f"decode-{dtype}-{d}-{g}x{n_q}-{n}")
    lib.close()


def test_a_late_key_far_above_the_rest():
    """The reference follows the maximum."""
    q, k, v = make_inputs(8, 2, 64, 1, 3000, "bf16", seed=5, needles=False)
    q, k = q.float(), k.float()
    u = q[0, 0] / q[0, 0].norm()
    q[0, 0], k[0, 1777] = 40.0 * u, 40.0 * u
    q, k = q.bfloat16(), k.bfloat16()
    lib = binding.LaserKV(8, 2, 64, "bf16", 8, 8, max_block=64, max_window=8, max_ctx_keys=0)
    out, lse = run_attend(lib, q.to(DEV), k.to(DEV), v.to(DEV), 3000)
    compare(out, lse, q, k, v, 3000, "bf16", "decode-late-key")
    lib.close()


def test_launches_of_changing_length_in_a_row():
    """The splits' counters return to zero with every launch, whatever the number of splits: eager and replayed."""
    h_q, h_kv, d, cap = 32, 8, 128, 6000
    q, k, v = (t.to(DEV) for t in make_inputs(h_q, h_kv, d, 1, cap, "bf16", seed=9))
    lib = binding.LaserKV(h_q, h_kv, d, "bf16", 8, 8, max_block=64, max_window=8, max_ctx_keys=0)
    lens = [1, 6000, 100, 2049, 128, 5999, 4096]
    ws = torch.empty(max(lib.laserkv_attend_workspace_bytes(1, n) for n in lens), dtype=torch.uint8, device=DEV)
    outs = [torch.empty(h_q, 1, d, device=DEV) for _ in lens]
    lses = [torch.empty(h_q, 1, device=DEV) for _ in lens]

    def run():
        for n, o, l in zip(lens, outs, lses):
            lib.laserkv_attend_cache(q, k, v, cache_len=n, out=o, out_lse=l, workspace=ws)

    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        run()
        stream.synchronize()
        ref = [o.clone() for o in outs]
        for n, o, l in zip(lens, outs, lses):
            compare(o.cpu().numpy(), l.cpu().numpy(), q.cpu(), k.cpu(), v.cpu(), n, "bf16", f"decode-row-{n}")
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            run()
        for _ in range(20):
            for o in outs:
                o.zero_()
            graph.replay()
            stream.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(ref, outs))
            run()
    stream.synchronize()
    lib.close()
