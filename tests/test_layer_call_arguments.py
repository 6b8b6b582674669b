"""What LayerCompressor hands to laserkv_compress_layer, without a GPU: a stand-in records the calls.  The window, the strides
and the number of blocks are those of the tensors, and what a block's own call refuses is refused."""
import types

import pytest
import torch

from paper_2602_02199_amd import binding, synth
from paper_2602_02199_amd.driver import LayerCompressor

WL = synth.Workload("layer-args", 0, 4, 2, 64, "f32", 2048, 512, 32, 4, 8, 8)
Q_WIN, N_TOK, S_BLOCK, W = 1, 12, 13, 14  # positions in the argument list


class Recorder:
    """The library functions a LayerCompressor calls, every shape supported."""

    def __init__(self):
        self.layer, self.blocks, self.asked = [], [], []
        self._ctx = 0
        self._lib = types.SimpleNamespace(
            laserkv_layer_workspace_bytes=lambda ctx, n_tok, s, w, n_local: self.asked.append((n_tok, w)) or 1000 + 100 * n_tok // s,
            laserkv_compress_layer=lambda *a: self.layer.append(a) or 0,
            laserkv_compress_block=None, laserkv_select_block=None, laserkv_append=None, laserkv_set_row_lse_complete=None)

    def _stream(self, stream):
        return stream

    def _check(self, rc):
        assert rc == 0

    def laserkv_select_block(self, q_win, k_blk, *a, **kw):
        self.blocks.append((binding._rows3(q_win, 64), binding._rows3(k_blk, 64)))

    def laserkv_append(self, *a, **kw):
        pass


def compressor(wl=WL, **kw):
    return LayerCompressor(wl, "cpu", lib=Recorder(), **kw)


def inputs(w=WL.window, n_win=4, l_ctx=2048):
    return dict(q_win=torch.zeros(n_win, 4, w, 64), k=torch.zeros(2, l_ctx, 64), v=torch.zeros(2, l_ctx, 64), planes=torch.zeros(64, 64))


def test_a_shorter_window_is_handed_over_as_it_is():
    comp, data = compressor(), inputs(w=20)
    comp.run_layer(data)
    args = comp.lib.layer[-1]
    assert args[W] == 20 and args[N_TOK] == 2048 and args[S_BLOCK] == 512
    assert args[Q_WIN:Q_WIN + 4] == (data["q_win"].data_ptr(), 4 * 20 * 64, 20 * 64, 64)
    assert comp.plan_layer(data)[0][1][W] == 20


def test_views_keep_their_strides():
    comp, data = compressor(), inputs()
    kv = torch.zeros(2, 2048, 2, 64)
    data.update(k=kv[:, :, 0], v=kv[:, :, 1])
    comp.run_layer(data, n_blocks=2)
    args = comp.lib.layer[-1]
    assert args[5:11] == (kv.data_ptr(), 2048 * 128, 128, kv.data_ptr() + 64 * 4, 2048 * 128, 128)
    assert args[N_TOK] == 1024


@pytest.mark.parametrize("name,make", [
    ("planes", lambda t: torch.zeros(64, 128)[:, ::2]),
    ("k", lambda t: torch.zeros(2, 2048, 128)[..., ::2]),
    ("v", lambda t: torch.zeros(2, 64, 2048).transpose(1, 2)),
    ("q_win", lambda t: torch.zeros(4, 4, 32, 128)[..., ::2]),
    ("k", lambda t: torch.zeros(2, 2048, 32)),
    ("v", lambda t: t[:, :2000]),
])
def test_tensors_a_block_call_refuses(name, make):
    comp, data = compressor(), inputs()
    data[name] = make(data[name])
    for call in (comp.run_layer, comp.plan_layer):
        with pytest.raises(AssertionError):
            call(data)
    assert not comp.lib.layer


def test_more_blocks_than_windows():
    comp = compressor()
    for call in (comp.run_layer, comp.plan_layer):
        with pytest.raises(IndexError):
            call(inputs(n_win=3), n_blocks=4)
    assert not comp.lib.layer


def test_statistics_of_another_window_are_refused():
    comp = compressor()
    lse = [torch.zeros(4, 32) for _ in range(4)]
    assert comp.plan_layer(inputs(), row_lse_complete=lse)
    with pytest.raises(AssertionError):
        comp.plan_layer(inputs(w=20), row_lse_complete=lse)


def test_plans_take_a_short_last_block_that_keeps_the_full_budget():
    wl = synth.Workload("short-last", 0, 4, 2, 64, "f32", 1900, 512, 32, 4, 8, 8)
    comp = compressor(wl)
    assert sum(comp.parts) <= 364  # the last block's tokens
    plan = comp.plan_layer(inputs(l_ctx=1900))
    assert len(plan) == 1 and plan[0][1][N_TOK] == 1900
    assert len(compressor(wl).plan_layer(inputs(l_ctx=1900), fused=False)) == 2 * 4
    wl = synth.Workload("too-short-last", 0, 4, 2, 64, "f32", 1640, 512, 32, 4, 8, 8)
    comp = compressor(wl)
    assert sum(comp.parts) > 104
    for fused in (True, False):
        with pytest.raises(AssertionError):
            comp.plan_layer(inputs(l_ctx=1640), fused=fused)


def test_the_scratch_is_there_from_the_start_and_stays():
    """Calls of growing length, a plan among them: one scratch tensor, sized for the longest; what the object was not made
    for brings its own."""
    comp = compressor()
    first = comp._layer_ws
    assert first is not None and first.numel() == 1000 + 100 * 4
    for n in (2, 3, 4):
        comp.run_layer(inputs(), n_blocks=n)
    plan = comp.plan_layer(inputs())
    assert all(a[-3] == first.data_ptr() and a[-2] == first.numel() for a in comp.lib.layer)
    assert comp._layer_ws is first and plan.tensors[1] is first
    longer = comp.plan_layer(inputs(n_win=6, l_ctx=3072))
    assert comp._layer_ws is first and longer.tensors[1].numel() == 1000 + 100 * 6
    assert longer[0][1][-2:] == (longer.tensors[1].data_ptr(), longer.tensors[1].numel())


def test_windows_in_a_list_go_block_by_block():
    comp, data = compressor(), inputs()
    data["q_win"] = list(data["q_win"])
    assert comp.run_layer(data, n_blocks=4) == comp.cap
    assert len(comp.lib.blocks) == 4 and not comp.lib.layer


def test_keys_that_only_fit_a_descriptor_block_by_block():
    """Rows so far apart that a block spans just under 2 GiB, with its look-back keys more."""
    comp, data = compressor(), inputs()
    stride = ((1 << 31) // (4 * 512) - 1) // 4 * 4
    data["k"] = _Strided(stride)
    assert comp._layer_call(data, 4) is None


class _Strided:
    """Shape and strides of a key tensor that would take 4 GiB."""

    def __init__(self, stride):
        self.shape, self._stride = (2, 2048, 64), (2048 * stride, stride, 1)

    def stride(self):
        return self._stride

    def data_ptr(self):
        return 0
