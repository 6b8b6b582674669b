"""The traffic that bench.py prints beside a launch is that launch's: a kernel that reads the keys reads at least those of the
blocks it takes, and not of more than a handful of passes over them."""
import pytest

import bench
from paper_2602_02199_amd import synth


@pytest.mark.parametrize("whole_layer", [True, False])
@pytest.mark.parametrize("name,lse,kernels", [("llama8b-128k", "own", ("sweep1", "sweep2")), ("llama8b-128k", "complete", ("single",)),
                                              ("gqa8-128k", "own", ("sweep1", "sweep2"))])
def test_traffic_belongs_to_the_launch(name, lse, kernels, whole_layer):
    wl = synth.WORKLOADS[name]
    keys = wl.n_kv_heads * (wl.l_ctx if whole_layer else wl.s_block) * wl.head_dim * 2
    for kernel in kernels:
        assert keys <= bench.measured_traffic(name, lse, whole_layer, kernel) <= 4 * keys


def test_no_traffic_for_what_was_not_profiled():
    assert bench.measured_traffic("no-such-workload", "own", True, "sweep1") is None
