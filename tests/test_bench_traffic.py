"""The traffic that bench.py prints beside a launch is that launch's: a kernel that reads the keys reads at least those of the
blocks it takes, and not of more than a handful of passes over them.  Rows that scoring copies are not the selection's."""
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


def test_rows_that_scoring_copies_are_not_the_selections():
    wl, B = synth.WORKLOADS["tiny"], 200
    work = bench.algorithmic_work(wl, B)
    work["select"] = ("hbm", work["select"][1] + work["append"][1])
    row = wl.n_kv_heads * 4 * wl.head_dim * 4  # fp32 keys and values, read and written
    assert bench.layer_work(wl, work, 0)["select"] == work["select"]
    assert bench.layer_work(wl, work, wl.n_blocks * 50)["select"] == ("hbm", work["select"][1] - 50 * row)


@pytest.mark.gpu
@pytest.mark.parametrize("name,copies", [("tiny", False), ("llama8b-16k", True), ("llama8b-64k", True), ("llama8b-128k", True), ("gqa8-128k", False)])
def test_the_library_says_what_scoring_copies(name, copies):
    from tests.test_gpu_layer import layer_plan
    wl = synth.WORKLOADS[name]
    for complete in (False, True):
        assert (layer_plan(wl, complete)["copied_rows"] > 0) == copies
