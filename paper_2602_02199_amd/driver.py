"""Block loop of one layer on the GPU: the sequence of library calls a prefill engine makes.

For every context block (Sec. 3.2) it calls laserkv_select_block and laserkv_append on the
current stream without any host synchronisation: each block adds exactly B_t rows per head, so
cache lengths are known on the host.  Look-back keys of block t are the previous block's local
window, i.e. the last n_local rows already in the cache (passed as a strided view, no copy).
"""
from __future__ import annotations

import torch

from . import binding


class _Plan(list):
    """A call list and the device tensors its arguments point to."""
    tensors = ()


class _Args(tuple):
    """Arguments of a laserkv_compress_layer and the scratch they point to."""
    workspace = None


class LayerCompressor:
    def __init__(self, wl, device="cuda:0", max_blocks=None, budget=None, tail=0, lib=None):
        """budget: per-block budget B of this layer (default: the App. B equation for the workload; a
        per-layer schedule passes its own).  tail: tokens a block defers to the next one (run_layer_deferred);
        blocks handed to the library are then up to s_block + tail long.  lib: an existing library context
        of sufficient limits to share (its workspace does not depend on the budget)."""
        self.wl = wl
        self.device = torch.device(device)
        self.B = binding.laserkv_budget(wl.s_block, wl.l_ctx, wl.r_num, wl.r_den) if budget is None else int(budget)
        self.parts = binding.laserkv_partition(self.B, wl.n_div, wl.alpha, wl.s_block)
        nb = wl.n_blocks if max_blocks is None else max_blocks
        self.tail = int(tail)
        self.cap = nb * min(self.B, wl.s_block + self.tail)
        max_local = binding.laserkv_partition(self.B, wl.n_div, wl.alpha, wl.s_block + self.tail)[1]
        self.lib = lib if lib is not None else binding.LaserKV(
            wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.dtype, wl.lsh_tables, wl.lsh_bits,
            max_block=wl.s_block + self.tail, max_window=wl.window, max_ctx_keys=max_local)
        dt = wl.torch_dtype
        self.k_cache = torch.zeros(wl.n_kv_heads, self.cap, wl.head_dim, dtype=dt, device=self.device)
        self.v_cache = torch.zeros_like(self.k_cache)
        self.cache_pos = torch.full((wl.n_kv_heads, self.cap), -1, dtype=torch.int64, device=self.device)
        self.keep = torch.empty(wl.n_kv_heads, min(self.B, wl.s_block), dtype=torch.int32, device=self.device)
        # scratch of laserkv_compress_layer for every number of blocks this object is made for: like the cache it is never
        # replaced, so no call on any stream and no captured graph loses it while this object lives
        size = max((self._layer_ws_bytes(n * wl.s_block, wl.window) for n in range(2, nb + 1)), default=-1)
        self._layer_ws = torch.empty(size, dtype=torch.uint8, device=self.device) if size > 0 else None
        self.cache_len = 0

    def reset(self):
        self.cache_len = 0

    def _layer_ws_bytes(self, n_tok, window):
        """Scratch of laserkv_compress_layer; -1 for shapes it has no kernels for."""
        return self.lib._lib.laserkv_layer_workspace_bytes(self.lib._ctx, n_tok, self.wl.s_block, window, self.parts[1])

    def run_layer_deferred(self, data, n_blocks=None, dbg_for=None):
        """The layer loop with each block's last `tail` tokens deferred to the next block's call (the look-back
        of Sec. 3.2 read as judging a block's edge only once later context exists): call t covers positions
        [block start - tail, block end - tail) (the first starts with its block, the last ends with its block)
        and is scored by the block's own last W tokens at their real positions.  Pointer arithmetic only.

        dbg_for: optional callable(t, seg_len) -> (dbg dict or None, keep tensor or None) supplying stage-output
        buffers for segment t.  Returns [(seg_lo, seg_hi, n_ctx, keep)] per segment."""
        wl, tail = self.wl, self.tail
        self.reset()
        nb = data["q_win"].shape[0] if n_blocks is None else n_blocks
        l_tot = data["k"].shape[1]
        prev_local, out = 0, []
        for t in range(nb):
            blk_lo, blk_hi = t * wl.s_block, min((t + 1) * wl.s_block, l_tot)
            lo = blk_lo - (tail if t else 0)
            hi = blk_hi - (tail if t < nb - 1 else 0)
            na, nl, ke, kl = binding.laserkv_partition(self.B, wl.n_div, wl.alpha, hi - lo)
            b_t = na + nl + ke + kl
            dbg, keep = dbg_for(t, hi - lo) if dbg_for else (None, None)
            if keep is None:
                keep = torch.empty(wl.n_kv_heads, b_t, dtype=torch.int32, device=self.device)
            dbg = dbg or {}
            k_ctx = self.k_cache[:, self.cache_len - prev_local:self.cache_len] if (self.cache_len and prev_local) else None
            k_seg, v_seg = data["k"][:, lo:hi], data["v"][:, lo:hi]
            self.lib.laserkv_select_block(data["q_win"][t], k_seg, k_ctx, data["planes"], block_pos0=lo,
                                          q_pos0=blk_hi - wl.window, causal=True,
                                          n_anchor=na, n_local=nl, k_exact=ke, k_lsh=kl, keep_idx=keep,
                                          dbg_s_exact=dbg.get("s_exact"), dbg_sig_k=dbg.get("sig_k"),
                                          dbg_sig_q=dbg.get("sig_q"), dbg_count=dbg.get("cnt"))
            self.lib.laserkv_append(k_seg, v_seg, keep, b_t=b_t, block_pos0=lo, k_cache=self.k_cache,
                                    v_cache=self.v_cache, cache_pos=self.cache_pos, cache_len=self.cache_len)
            self.cache_len += b_t
            out.append((lo, hi, prev_local, keep))
            prev_local = nl
        return out

    def block_budget(self, s_t):
        """(n_anchor, n_local, k_exact, k_lsh) of a block with s_t tokens."""
        if s_t == self.wl.s_block:
            return self.parts
        return binding.laserkv_partition(self.B, self.wl.n_div, self.wl.alpha, s_t)

    def step(self, q_win, k_blk, v_blk, planes, block_pos0, prev_local, dbg=None, keep_out=None):
        """One block: select + append.  Returns (this block's n_local, the keep tensor used).

        keep_out: optional [H_kv, B_t] int32 device tensor to receive the kept indices (the internal
        buffer is reused from block to block otherwise).  dbg: optional dict of device tensors for the
        stage outputs (s_exact, sig_k, sig_q, cnt).
        """
        s_t = k_blk.shape[1]
        na, nl, ke, kl = self.block_budget(s_t)
        b_t = na + nl + ke + kl
        k_ctx = None
        if self.cache_len and prev_local:
            k_ctx = self.k_cache[:, self.cache_len - prev_local:self.cache_len]
        if keep_out is not None:
            keep = keep_out
        elif b_t == self.keep.shape[1]:
            keep = self.keep
        else:
            keep = torch.empty(self.wl.n_kv_heads, b_t, dtype=torch.int32, device=self.device)
        assert keep.shape == (self.wl.n_kv_heads, b_t) and keep.is_contiguous()
        dbg = dbg or {}
        self.lib.laserkv_select_block(q_win, k_blk, k_ctx, planes, block_pos0=block_pos0, causal=True,
                                      n_anchor=na, n_local=nl, k_exact=ke, k_lsh=kl, keep_idx=keep,
                                      dbg_s_exact=dbg.get("s_exact"), dbg_sig_k=dbg.get("sig_k"),
                                      dbg_sig_q=dbg.get("sig_q"), dbg_count=dbg.get("cnt"))
        self.lib.laserkv_append(k_blk, v_blk, keep, b_t=b_t, block_pos0=block_pos0, k_cache=self.k_cache,
                                v_cache=self.v_cache, cache_pos=self.cache_pos, cache_len=self.cache_len)
        self.cache_len += b_t
        return nl, keep

    def _layer_call(self, data, nb, row_lse_complete=None):
        """(c_function, argument tuple without the stream) of one laserkv_compress_layer over the first nb blocks and
        the rows it leaves in the cache, or None for shapes it has no kernels for.  row_lse_complete: device tensor
        of per-block pointers, or None.  The library is told what the tensors hold (a window shorter than the workload's
        is one) and tensors that a block's own call refuses are refused here."""
        wl, lib = self.wl, self.lib
        if not torch.is_tensor(data["q_win"]):  # windows as a list: no common stride
            return None
        q, qsb, qsh, qst, n_win, w = binding._rows4(data["q_win"], wl.head_dim)
        k, ksh, kst, l_tot = binding._rows3(data["k"], wl.head_dim)
        v, vsh, vst, l_v = binding._rows3(data["v"], wl.head_dim)
        planes = data["planes"]
        assert planes.is_contiguous()
        if nb > n_win:
            raise IndexError(f"{nb} blocks, but window queries of {n_win}")
        n_tok = min(nb * wl.s_block, l_tot)
        assert l_v >= n_tok, "fewer values than keys"
        last = n_tok - (nb - 1) * wl.s_block
        # a block and its look-back keys go through one buffer descriptor; a block alone may just fit where both do not
        one_span = (wl.s_block + self.parts[1]) * kst * self.k_cache.element_size() < 1 << 31
        size = self._layer_ws_bytes(n_tok, w) if last >= w and one_span else -1
        if size < 0:
            return None
        ws = self._layer_ws
        if ws is None or ws.numel() < size:  # more blocks or another window: this call's (or plan's) own
            ws = torch.empty(size, dtype=torch.uint8, device=self.device)
        b_last = sum(self.block_budget(last))
        keep = self.keep if b_last == self.keep.shape[1] else None
        args = _Args((lib._ctx, q, qsb, qsh, qst, k, ksh, kst, v, vsh, vst, planes.data_ptr(), n_tok, wl.s_block, w,
                self.B, wl.n_div, wl.alpha, None if row_lse_complete is None else row_lse_complete.data_ptr(),
                None if keep is None else keep.data_ptr(), self.k_cache.data_ptr(), self.v_cache.data_ptr(),
                self.k_cache.stride(0), self.cache_pos.data_ptr(), self.cache_pos.stride(0), self.cap,
                ws.data_ptr(), ws.numel()))
        args.workspace = ws
        return lib._lib.laserkv_compress_layer, args, (nb - 1) * sum(self.parts) + b_last

    def run_layer(self, data, n_blocks=None):
        """All blocks of one layer, no host sync: one laserkv_compress_layer call, or, where a block's shape has no
        layer kernels, block by block.  data: device tensors from synth.make_layer."""
        wl = self.wl
        self.reset()
        nb = data["q_win"].shape[0] if n_blocks is None else n_blocks
        prev_local = 0
        l_tot = data["k"].shape[1]
        call = self._layer_call(data, nb) if nb > 1 else None
        if call is not None:
            fn, args, n = call
            self.lib._check(fn(*args, self.lib._stream(None)))
            self.cache_len = n
            return n
        for t in range(nb):
            lo, hi = t * wl.s_block, min((t + 1) * wl.s_block, l_tot)
            prev_local, _ = self.step(data["q_win"][t], data["k"][:, lo:hi], data["v"][:, lo:hi], data["planes"],
                                      lo, prev_local)
        return self.cache_len

    def run_layer_with_attention(self, data, q_blocks, out, lse, lse_win, workspace, n_blocks=None):
        """The block loop as a model runs it (Sec. 3 first paragraph; Sec. 3.3 "Precision"): block t's queries
        attend to the compacted cache and, causally, to the block itself (laserkv_attend_block); the window
        rows' log-sum-exp that kernel reports is handed to the selection as the complete row statistic
        (laserkv_set_row_lse_complete: one sweep over the block, no statistics of its own); the kept rows join
        the cache the next block attends to.  No host synchronisation.

        q_blocks[t]: [H_q, S_t, d] queries of block t, whose last W rows are the observation window (passed to
        the selection as a view).  out [H_q, S, d] and lse [H_q, S] float32 receive each block's attention,
        lse_win [H_q, W] float32 the window rows' statistics, workspace the attention scratch (sized for the
        last block); all are reused from block to block."""
        wl = self.wl
        self.reset()
        nb = len(q_blocks) if n_blocks is None else n_blocks
        l_tot = data["k"].shape[1]
        w = wl.window
        for t in range(nb):
            lo, hi = t * wl.s_block, min((t + 1) * wl.s_block, l_tot)
            s_t = hi - lo
            q, k_blk, v_blk = q_blocks[t], data["k"][:, lo:hi], data["v"][:, lo:hi]
            # contiguous [H_q, s_t, ...] tensors at the start of the buffers (a short last block uses less of them)
            out_now = out.view(-1)[:q.shape[0] * s_t * wl.head_dim].view(q.shape[0], s_t, wl.head_dim)
            lse_now = lse.view(-1)[:q.shape[0] * s_t].view(q.shape[0], s_t)
            self.lib.laserkv_attend_block(q, self.k_cache, self.v_cache, k_blk, v_blk, cache_len=self.cache_len, block_pos0=lo,
                                          out=out_now, out_lse=lse_now, workspace=workspace)
            lse_win.copy_(lse_now[:, s_t - w:])
            self.lib.laserkv_set_row_lse_complete(lse_win)
            na, nl, ke, kl = self.block_budget(s_t)
            b_t = na + nl + ke + kl
            keep = self.keep if b_t == self.keep.shape[1] else torch.empty(wl.n_kv_heads, b_t, dtype=torch.int32, device=self.device)
            self.lib.laserkv_compress_block(q[:, s_t - w:], k_blk, v_blk, None, data["planes"], block_pos0=lo, n_anchor=na,
                                            n_local=nl, k_exact=ke, k_lsh=kl, keep_idx=keep, k_cache=self.k_cache,
                                            v_cache=self.v_cache, cache_pos=self.cache_pos, cache_len=self.cache_len)
            self.cache_len += b_t
        self.lib.laserkv_set_row_lse_complete(None)
        return self.cache_len

    # ---- pre-marshalled call lists: one ctypes call per library entry point, nothing else ----
    def plan_layer(self, data, n_blocks=None, fused=True, row_lse_complete=None):
        """Builds the layer's call list once: [(c_function, argument tuple without the stream)].

        The tensors in `data`, the cache and the keep buffer must stay alive and in place while the
        plan is used.  run_plan() then issues the calls back to back with no per-call Python work
        beyond the foreign call itself (and can be captured into a HIP graph).  fused=True uses
        laserkv_compress_layer (one call for all blocks) where it has kernels for the shape, else
        laserkv_compress_block (one call per block); fused=False laserkv_select_block + laserkv_append.
        row_lse_complete: optional list of per-block float32 [H_q, W] device tensors with the window rows'
        complete log-sum-exp (what the model's attention kernel reports): handed to laserkv_compress_layer as a
        table of pointers, or set by laserkv_set_row_lse_complete in front of each block's call, and look-back
        keys are not passed.
        """
        import ctypes as C
        wl, lib = self.wl, self.lib._lib
        ctx = self.lib._ctx
        vp = C.c_void_p
        nb = data["q_win"].shape[0] if n_blocks is None else n_blocks
        l_tot = data["k"].shape[1]
        d = wl.head_dim
        calls, cache_len, prev_local = _Plan(), 0, 0
        if row_lse_complete is not None:
            assert all(q.shape[1] == wl.window for q in data["q_win"][:nb]), "statistics are those of the workload's window"
            for lse in row_lse_complete[:nb]:
                assert lse.is_contiguous() and lse.dtype == torch.float32 and lse.shape == (wl.n_q_heads, wl.window)
        if fused and nb > 1:
            table = None
            if row_lse_complete is not None:
                table = torch.tensor([t.data_ptr() for t in row_lse_complete[:nb]], dtype=torch.int64, device=self.device)
            call = self._layer_call(data, nb, table)
            if call is not None:
                assert call[2] == nb * sum(self.parts), "plans cover blocks that keep equally many rows only"
                calls.tensors = (table, call[1].workspace)
                calls.append((call[0], call[1], True))
                if row_lse_complete is not None:
                    calls.append((lib.laserkv_set_row_lse_complete, (ctx, None), False))
                self._plan_len = call[2]
                return calls
        assert data["planes"].is_contiguous()
        planes = data["planes"].data_ptr()
        kc_sh, kc_st = self.k_cache.stride(0), self.k_cache.stride(1)
        es = self.k_cache.element_size()
        for t in range(nb):
            lo, hi = t * wl.s_block, min((t + 1) * wl.s_block, l_tot)
            s_t = hi - lo
            na, nl, ke, kl = self.block_budget(s_t)
            b_t = na + nl + ke + kl
            assert b_t == self.keep.shape[1], "plans cover blocks that keep equally many rows only"
            q, qsh, qst, w = binding._rows3(data["q_win"][t], d)
            k, ksh, kst, _ = binding._rows3(data["k"][:, lo:hi], d)
            v, vsh, vst, _ = binding._rows3(data["v"][:, lo:hi], d)
            t_ctx = prev_local if cache_len else 0
            if row_lse_complete is not None:
                lse = row_lse_complete[t]
                calls.append((lib.laserkv_set_row_lse_complete, (ctx, vp(lse.data_ptr())), False))
                t_ctx = 0
            ctx_ptr = vp(self.k_cache.data_ptr() + (cache_len - t_ctx) * kc_st * es) if t_ctx else None
            if fused:
                calls.append((lib.laserkv_compress_block, (
                    ctx, q, qsh, qst, k, ksh, kst, v, vsh, vst,
                    ctx_ptr, kc_sh if t_ctx else 0, kc_st if t_ctx else 0, planes,
                    s_t, w, t_ctx, lo, binding.LKV_WINDOW_AT_BLOCK_END, 1, na, nl, ke, kl,
                    vp(self.keep.data_ptr()), vp(self.k_cache.data_ptr()), vp(self.v_cache.data_ptr()), kc_sh,
                    vp(self.cache_pos.data_ptr()), self.cache_pos.stride(0), cache_len, self.cap), True))
            else:
                calls.append((lib.laserkv_select_block, (
                    ctx, q, qsh, qst, k, ksh, kst,
                    ctx_ptr, kc_sh if t_ctx else 0, kc_st if t_ctx else 0, planes,
                    s_t, w, t_ctx, lo, binding.LKV_WINDOW_AT_BLOCK_END, 1, na, nl, ke, kl,
                    vp(self.keep.data_ptr()), None, None, None, None), True))
                calls.append((lib.laserkv_append, (
                    ctx, k, ksh, kst, v, vsh, vst,
                    vp(self.keep.data_ptr()), b_t, s_t, lo, vp(self.k_cache.data_ptr()), vp(self.v_cache.data_ptr()),
                    kc_sh, vp(self.cache_pos.data_ptr()), self.cache_pos.stride(0), cache_len, self.cap), True))
            cache_len += b_t
            prev_local = nl
        if row_lse_complete is not None:   # leave the context computing its own statistics again
            calls.append((lib.laserkv_set_row_lse_complete, (ctx, None), False))
        self._plan_len = cache_len
        return calls

    def run_plan(self, calls, stream=None):
        sp = self.lib._stream(stream)
        for fn, args, takes_stream in calls:
            rc = fn(*args, sp) if takes_stream else fn(*args)
            if rc != 0:
                self.lib._check(rc)
        self.cache_len = self._plan_len
        return self.cache_len
