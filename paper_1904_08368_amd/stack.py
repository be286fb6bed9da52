"""A network as a sequence of fused primitive functions called one after another on
preallocated buffers (paper Section 3.3: operator invocations replaced by calls to the
compiled operators, inputs and outputs preallocated).

Set-up (filter packing, channel padding of filters, buffer allocation) is compile-time
work and happens once in the constructor; ``run()`` only enqueues kernels of the library
on torch's current stream, so it can also be captured into a HIP graph.
"""
from __future__ import annotations

import threading
import time
from typing import Dict, List, Optional

import numpy as np
import torch

from . import binding as B


def _round_up(a: int, b: int) -> int:
    return (a + b - 1) // b * b


class PassGraph(torch.cuda.CUDAGraph):
    """A captured pass, which counts what ends a copy of it."""

    held = 0

    def capture_begin(self, *args, **kwargs) -> None:
        self.held += 1
        super().capture_begin(*args, **kwargs)

    def reset(self) -> None:
        self.held += 1
        super().reset()


class FusedNet:
    """mode 'f16': fp16 NHWC, fp32 accumulation.  mode 'i8': int8 NHWC, int32 accumulation,
    ``shifts[i] = {'s': out_rshift, 'l': residual_lshift}`` per conv."""

    def __init__(self, ops, params: List[dict], batch: int, h: int, w: int, mode: str = "f16",
                 shifts: Optional[List[dict]] = None, in_channels: int = 3, device: str = "cuda:0",
                 overlap_shortcuts: bool = False, fused: bool = True, combine: bool = False,
                 fold_scale: bool = False, fuse_pool: bool = True, fuse_dwpw: bool = True,
                 first_layer_direct: bool = True):
        assert mode in ("f16", "i8")
        assert fused or mode == "f16"
        # combine: convs that share input, window and tail run as one launch ("windows": also a 1x1 conv
        # beside a wider odd window of the same stride, and tails that differ in relu); fold_scale: the
        # batch-norm scale is multiplied into the filters ahead of time (paper Section 4.4, both)
        assert not (combine or fold_scale) or (mode == "f16" and fused)
        self.fold_scale = fold_scale
        # fuse_pool: a conv whose only reader is a 3x3 / stride 2 / pad 1 max pool runs with it as one
        # launch where the library takes the shape; the conv's own output tensor then does not exist
        self.fuse_pool = fuse_pool and fused
        # fuse_dwpw: a depthwise conv whose only reader is a plain 1x1 conv runs with it as one launch where
        # the library expects that to be faster (by layer and batch: nearly everywhere at batch 1, the first
        # blocks and the 512-channel ones at batch 32); the depthwise output tensor then does not exist
        # ("always": wherever the library has a kernel for the shape, profitable or not)
        self.fuse_dwpw = fuse_dwpw if (fused and mode == "f16" and not fold_scale) else False
        # fused=False launches every elementwise operator behind a contraction as a kernel of its
        # own on a tensor of its own: the pipeline of a framework without operator fusion, kept
        # for the fusion ablation (paper Section 5.2)
        self.fused = fused
        self.ops, self.mode, self.batch = ops, mode, batch
        self.dev = torch.device(device)
        self.dtype = B.RELAY_F16 if mode == "f16" else B.RELAY_I8
        self.tdtype = torch.float16 if mode == "f16" else torch.int8
        self.ve = 8 if mode == "f16" else 16
        self.calls = []                      # (callable, args) in execution order
        self.call_names: List[str] = []
        self.bufs: Dict[str, torch.Tensor] = {}
        self.shape: Dict[str, tuple] = {}    # name -> (C_logical, H, W), physical C = padded
        self.keep = []                       # parameter tensors kept alive

        cpad = _round_up(in_channels, self.ve)
        self.x_nchw = torch.zeros((batch, in_channels, h, w), dtype=self.tdtype, device=self.dev)
        self.shape["x"] = (in_channels, h, w)
        first = ops[0]
        only_reader = first.kind == "conv" and first.src == "x" and \
            sum(1 for o in ops if o.src == "x" or o.res == "x") == 1
        # a first-layer conv the library reads straight from the NCHW image (3 channels, 3x3 / stride 2): no
        # converted or padded copy of the image at all
        self.stem_direct = False
        if only_reader and fused and mode == "f16" and not (combine or fold_scale) and first_layer_direct and \
                not first.res:
            d0 = B.conv_desc(batch, in_channels, h, w, first.cout, first.r, first.r, first.stride, first.pad,
                             self.dtype, B.RELAY_NCHW, 0)
            try:
                self.stem_direct = B.relay_conv2d_first_layer_supported(d0)
            except B.RelayError:
                self.stem_direct = False
        # a first-layer conv on <= 4 channels reads the pre-padded NHWC4 form of the image
        self.stem_nhwc4 = only_reader and in_channels <= 4 and not self.stem_direct
        if self.stem_direct:
            self.bufs["x"] = self.x_nchw
        elif self.stem_nhwc4:
            d0 = B.conv_desc(batch, in_channels, h, w, first.cout, first.r, first.r, first.stride, first.pad,
                             self.dtype, B.RELAY_NHWC4_PADDED, 0)
            hp, wp = B.relay_nhwc4_padded_shape(d0)
            self.bufs["x"] = torch.zeros((batch, hp, wp, 4), dtype=self.tdtype, device=self.dev)
            self._add("pack_input_nhwc4", B.relay_pack_input_nhwc4, (d0, self.x_nchw, self.bufs["x"]))
            self.keep.append(d0)
        else:
            self.bufs["x"] = torch.zeros((batch, h, w, cpad), dtype=self.tdtype, device=self.dev)
            self._add("nchw_to_nhwc", B.relay_nchw_to_nhwc,
                      (self.dtype, batch, in_channels, h, w, cpad, self.x_nchw, self.bufs["x"]))

        from .fusion import combine_parallel
        group_of = {min(g): g for g in (combine_parallel(ops, windows=(combine == "windows")) if combine else [])}
        absorbed = {j for i, g in group_of.items() for j in g if j != i}
        self._plan_concats(ops, batch, h, w, in_channels, cpad)

        for i, (op, p) in enumerate(zip(ops, params)):
            if i in absorbed:
                continue
            cin_l, hi, wi = self.shape[op.src]
            src = self.bufs[op.src]
            cin_p = src.shape[-1]
            if op.kind == "concat":
                # nothing to launch: every producer has already written its channel range
                assert all(self.view_of.get(s_, (None,))[0] == op.dst for s_ in op.srcs)
                self.shape[op.dst] = (self.bufs[op.dst].shape[-1], hi, wi)
            elif op.kind == "conv" and (i in group_of or op.dst in self.view_of or not src.is_contiguous()):
                idxs = group_of.get(i, [i])
                self._emit_conv_views([ops[j] for j in idxs], [params[j] for j in idxs], batch)
            elif op.kind == "conv" and i == 0 and self.stem_direct:
                flags = B.flags_of(p.get("bias"), p.get("scale"), None, op.relu)
                d = B.conv_desc(batch, cin_l, hi, wi, op.cout, op.r, op.r, op.stride, op.pad, self.dtype, B.RELAY_NCHW, flags)
                ho, wo = B.relay_conv2d_out_shape(d)
                wsrc = torch.from_numpy(np.ascontiguousarray(p["w"])).to(self.dev)
                y = torch.empty((batch, ho, wo, op.cout), dtype=self.tdtype, device=self.dev)
                bias, sc, sf = (self._f32(p.get(k)) for k in ("bias", "scale", "shift"))
                wp = torch.empty(B.relay_first_layer_packed_weight_bytes(d), dtype=torch.uint8, device=self.dev)
                B.relay_prepack_first_layer_weights(d, wsrc, wp)
                self._add(op.name, B.relay_fused_conv2d_first_layer, (d, src, wp, bias, sc, sf, y))
                self.keep += [wp, d]
                self.bufs[op.dst], self.shape[op.dst] = y, (op.cout, ho, wo)
            elif op.kind == "conv":
                flags = B.flags_of(p.get("bias"), p.get("scale"), op.res, op.relu)
                if i == 0 and self.stem_nhwc4:
                    d = B.conv_desc(batch, cin_l, hi, wi, op.cout, op.r, op.r, op.stride, op.pad, self.dtype,
                                    B.RELAY_NHWC4_PADDED, flags)
                else:
                    d = B.conv_desc(batch, cin_p, hi, wi, op.cout, op.r, op.r, op.stride, op.pad, self.dtype,
                                    B.RELAY_NHWC, flags)
                ho, wo = B.relay_conv2d_out_shape(d)
                wsrc = torch.from_numpy(np.ascontiguousarray(p["w"])).to(self.dev)
                wp = torch.empty(B.relay_packed_weight_bytes(d), dtype=torch.uint8, device=self.dev)
                B.relay_prepack_conv2d_weights(d, wsrc, cin_l, wp)
                pool = self._pool_behind(ops, i) if self.fuse_pool and B.relay_conv2d_maxpool_fusable(d) else None
                if pool is not None:
                    absorbed.add(pool)
                    y = torch.empty((batch, ho // 2, wo // 2, op.cout), dtype=self.tdtype, device=self.dev)
                    name = op.name + "+" + ops[pool].name
                    if mode == "f16" and fold_scale and p.get("scale") is not None:
                        bias = self._fold(op, p, wsrc, cin_l)
                        B.relay_prepack_conv2d_weights(d, wsrc, cin_l, wp)
                        d = B.conv_desc(d.n, d.c, d.h, d.w, d.k, d.r, d.s, d.stride_h, d.pad_h, self.dtype, d.layout,
                                        B.flags_of(True, None, None, op.relu))
                        self._add(name, B.relay_fused_conv2d_bn_relu_maxpool, (d, src, wp, bias, None, None, y))
                    elif mode == "f16":
                        bias, sc, sf = (self._f32(p.get(k)) for k in ("bias", "scale", "shift"))
                        self._add(name, B.relay_fused_conv2d_bn_relu_maxpool, (d, src, wp, bias, sc, sf, y))
                    else:
                        qb = None
                        if p.get("bias") is not None:
                            qb = torch.from_numpy(np.ascontiguousarray(p["bias"], dtype=np.int32)).to(self.dev)
                            self.keep.append(qb)
                        self._add(name, B.relay_qconv2d_requant_maxpool, (d, src, wp, qb, int(shifts[i]["s"]), y))
                    self.keep += [wp, d]
                    self.bufs[ops[pool].dst], self.shape[ops[pool].dst] = y, (op.cout, ho // 2, wo // 2)
                    continue
                y = torch.empty((batch, ho, wo, op.cout), dtype=self.tdtype, device=self.dev)
                res = self.bufs[op.res] if op.res else None
                ws = self._workspace(d)     # None for most layers
                if mode == "f16" and not fused and flags:
                    d0 = B.conv_desc(d.n, d.c, d.h, d.w, d.k, d.r, d.s, d.stride_h, d.pad_h, self.dtype, d.layout, 0)
                    raw = torch.empty_like(y)
                    self._add(op.name, B.relay_fused_conv2d_bias_bn_relu, (d0, src, wp, None, None, None, None, raw))
                    self.keep.append(d0)
                    y = self._unfused_tail(op, p, raw, batch * ho * wo, op.cout, res)
                elif mode == "f16" and fold_scale and p.get("scale") is not None:
                    # the filters were packed unscaled above: pack the folded ones over them
                    bias = self._fold(op, p, wsrc, cin_l)
                    B.relay_prepack_conv2d_weights(d, wsrc, cin_l, wp)
                    d1 = B.conv_desc(d.n, d.c, d.h, d.w, d.k, d.r, d.s, d.stride_h, d.pad_h, self.dtype, d.layout,
                                     B.flags_of(True, None, op.res, op.relu))
                    self._add(op.name, B.relay_fused_conv2d_bias_bn_relu, (d1, src, wp, bias, None, None, res, y, ws))
                    self.keep.append(d1)
                elif mode == "f16":
                    bias, sc, sf = (self._f32(p.get(k)) for k in ("bias", "scale", "shift"))
                    self._add(op.name, B.relay_fused_conv2d_bias_bn_relu, (d, src, wp, bias, sc, sf, res, y, ws))
                else:
                    sh = shifts[i]
                    qb = None
                    if p.get("bias") is not None:
                        qb = torch.from_numpy(np.ascontiguousarray(p["bias"], dtype=np.int32)).to(self.dev)
                        self.keep.append(qb)
                    self._add(op.name, B.relay_qconv2d_requant,
                              (d, src, wp, qb, res, int(sh.get("l", 0)), int(sh["s"]), y, ws))
                self.keep += [wp, d]
                self.bufs[op.dst], self.shape[op.dst] = y, (op.cout, ho, wo)
            elif op.kind == "dwconv":
                flags = B.flags_of(p.get("bias"), p.get("scale"), None, op.relu)
                d = B.conv_desc(batch, cin_p, hi, wi, cin_p, op.r, op.r, op.stride, op.pad, self.dtype,
                                B.RELAY_NHWC, flags)
                ho, wo = B.relay_conv2d_out_shape(d)
                wsrc = torch.from_numpy(np.ascontiguousarray(p["w"])).to(self.dev)
                wp = torch.empty((op.r * op.r, cin_p), dtype=self.tdtype, device=self.dev)
                B.relay_prepack_dwconv_weights(d, wsrc, wp)
                pw = self._pointwise_behind(ops, i, group_of, absorbed) if self.fuse_dwpw and op.r == 3 and op.pad == 1 \
                    and cin_p % 32 == 0 and src.is_contiguous() else None
                if pw is not None and (self.fuse_dwpw == "always" or B.relay_dwconv_pwconv_few_pixels(d, ops[pw].cout) or
                                       B.relay_dwconv_pwconv_fusion_pays(d, ops[pw].cout)):
                    q, pp = ops[pw], params[pw]
                    pflags = B.flags_of(pp.get("bias"), pp.get("scale"), None, q.relu)
                    pd = B.conv_desc(batch, cin_p, ho, wo, q.cout, 1, 1, 1, 0, self.dtype, B.RELAY_NHWC, pflags)
                    pwp = torch.empty(B.relay_packed_weight_bytes(pd), dtype=torch.uint8, device=self.dev)
                    B.relay_prepack_conv2d_weights(pd, torch.from_numpy(np.ascontiguousarray(pp["w"])).to(self.dev), cin_l, pwp)
                    y = torch.empty((batch, ho, wo, q.cout), dtype=self.tdtype, device=self.dev)
                    bias, sc, sf = (self._f32(p.get(k)) for k in ("bias", "scale", "shift"))
                    pb, psc, psf = (self._f32(pp.get(k)) for k in ("bias", "scale", "shift"))
                    self._add(op.name + "+" + q.name, B.relay_fused_dwconv_pwconv,
                              (d, src, wp, bias, sc, sf, q.cout, pflags, pwp, pb, psc, psf, y))
                    absorbed.add(pw)
                    self.keep += [wp, d, pwp, pd]
                    self.bufs[q.dst], self.shape[q.dst] = y, (q.cout, ho, wo)
                    continue
                y = torch.empty((batch, ho, wo, cin_p), dtype=self.tdtype, device=self.dev)
                if not fused and flags:
                    d0 = B.conv_desc(d.n, d.c, d.h, d.w, d.k, d.r, d.s, d.stride_h, d.pad_h, self.dtype, d.layout, 0)
                    raw = torch.empty_like(y)
                    self._add(op.name, B.relay_fused_dwconv_bias_relu, (d0, src, wp, None, None, None, raw))
                    self.keep.append(d0)
                    y = self._unfused_tail(op, p, raw, batch * ho * wo, cin_p, None)
                else:
                    bias, sc, sf = (self._f32(p.get(k)) for k in ("bias", "scale", "shift"))
                    self._add(op.name, B.relay_fused_dwconv_bias_relu, (d, src, wp, bias, sc, sf, y))
                self.keep += [wp, d]
                self.bufs[op.dst], self.shape[op.dst] = y, (op.cout, ho, wo)
            elif op.kind == "maxpool":
                ho = (hi + 2 * op.pad - op.r) // op.stride + 1
                wo = (wi + 2 * op.pad - op.r) // op.stride + 1
                y = torch.empty((batch, ho, wo, cin_p), dtype=self.tdtype, device=self.dev)
                self._add(op.name, B.relay_maxpool2d, (self.dtype, batch, cin_p, hi, wi, op.r, op.stride, op.pad, src, y))
                self.bufs[op.dst], self.shape[op.dst] = y, (cin_l, ho, wo)
            elif op.kind == "avgpool":
                y = torch.empty((batch, 1, 1, cin_p), dtype=self.tdtype, device=self.dev)
                self._add(op.name, B.relay_global_avgpool, (self.dtype, batch, cin_p, hi * wi, src, y))
                self.bufs[op.dst], self.shape[op.dst] = y, (cin_l, 1, 1)
            elif op.kind == "dense":
                wd = torch.from_numpy(np.ascontiguousarray(p["w"])).to(self.dev)
                if hi * wi > 1:
                    # a dense layer over a [C, H, W] tensor: its filters are given for (channel, row, column)
                    # order; the NHWC buffer holds (row, column, channel), so the columns are permuted once here
                    if cin_p != cin_l or op.cin != cin_l * hi * wi:
                        raise ValueError(f"{op.name}: dense over a padded or mismatched [{cin_l},{hi},{wi}] tensor")
                    wd = wd.reshape(op.cout, cin_l, hi, wi).permute(0, 2, 3, 1).reshape(op.cout, op.cin).contiguous()
                bias = self._f32(p.get("bias"))
                y = torch.empty((batch, 1, 1, op.cout), dtype=self.tdtype, device=self.dev)
                if not fused and mode == "f16" and (bias is not None or op.relu) and op.cout % 8 == 0:
                    raw = torch.empty_like(y)
                    self._add(op.name, B.relay_fused_dense_bias_act,
                              (batch, op.cout, op.cin, self.dtype, src, wd, None, 0, raw))
                    y = self._unfused_tail(op, p, raw, batch, op.cout, None)
                else:
                    self._add(op.name, B.relay_fused_dense_bias_act,
                              (batch, op.cout, op.cin, self.dtype, src, wd, bias, 1 if op.relu else 0, y))
                self.keep += [wd]
                self.bufs[op.dst], self.shape[op.dst] = y, (op.cout, 1, 1)
            else:
                raise ValueError(op.kind)
        # calls that may run beside their predecessor: a conv that reads the same tensor as the
        # conv before it and whose output is first needed as a residual.  Off by default: with the
        # fork placed in front of the sibling conv the two kernels really do overlap, and the whole
        # ResNet-18 stack is then slower than the serial order (batch 32: 0.322 against 0.303 ms per
        # step, batch 1: 0.191 against 0.161 ms, replayed from a HIP graph)
        self.side_calls, self.join_before = set(), set()
        self.side = None
        if overlap_shortcuts and fused:   # (the unfused tails would have to follow their conv onto the side stream)
            idx_of = {name: i for i, name in enumerate(self.call_names)}
            for j in range(1, len(ops)):
                a0, a1 = ops[j - 1], ops[j]
                if a0.kind == "conv" and a1.kind == "conv" and a0.src == a1.src and not a1.res and not a0.res:
                    users = [o for o in ops if o.src == a1.dst or o.res == a1.dst]
                    if len(users) == 1 and users[0].res == a1.dst and a1.name in idx_of and users[0].name in idx_of \
                            and idx_of.get(a0.name) == idx_of[a1.name] - 1:
                        self.side_calls.add(idx_of[a1.name])
                        self.join_before.add(idx_of[users[0].name])
            if self.side_calls:
                self.side = torch.cuda.Stream(device=self.dev)
        self._plan_launches()
        if combine and not self.side_calls:
            self._move_pools()
        if self.stem:
            self.bufs["x"] = self.x_nchw   # (as the launch reads it: the copy would be what an earlier run left there)
        torch.cuda.synchronize(self.dev)
        self.graph = None

    stem = None
    merged: Dict[int, tuple] = {}

    def _plan_launches(self):
        """Which neighbours in `calls` run as one launch."""
        # a block's first conv and the shortcut conv beside it
        self.pairs = {} if self.side_calls else self._independent_pairs()
        # the first calls on the image itself: its padded copy (not written then), the conv and the pool behind it
        self.stem = self._image_stem()
        # further calls that one launch stands for, writing the same tensors
        self.merged = {**self._merged_calls(), **self._combined_groups()}

    def _move_pools(self):
        """Puts a max pool right behind a conv on the tensor that it reads where a run then makes fewer launches: the two share one, or the conv on the
        pool's result shares one with the convs that it now follows.  (Only there: a pool between calls that share a launch parts them.)"""
        convs = (B.relay_fused_conv2d_combined, B.relay_fused_conv2d_combined_windows, B.relay_fused_conv2d_bias_bn_relu)
        for pool in [c for c in self.calls if c[0] is B.relay_maxpool2d]:
            listed = self.calls, self.call_names
            best, launches = listed, len(self._steps())
            at = next(i for i, c in enumerate(self.calls) if c is pool)
            for to in [i + 1 for i, (fn, a) in enumerate(self.calls[:max(at - 1, 0)]) if fn in convs and a[1] is pool[1][8]]:
                self.calls, self.call_names = ([*v[:to], v[at], *v[to:at], *v[at + 1:]] for v in listed)
                self._plan_launches()
                if len(self._steps()) < launches:
                    best, launches = (self.calls, self.call_names), len(self._steps())
            self.calls, self.call_names = best
            self._plan_launches()

    def _merged_calls(self):
        """{i: (calls, function, arguments)} of a conv and the 2x2 max pool on its outputs, of the two convs of a residual block, and of the
        average pool and the dense layer on its result, where the library takes them together and that pays."""
        merged = {}
        for i in range(len(self.calls) - 1):
            (f0, a0), (f1, a1) = self.calls[i], self.calls[i + 1]
            # (no residual, no workspace; the pool reads what the conv wrote)
            if f0 is B.relay_fused_conv2d_bias_bn_relu and len(a0) == 9 and a0[6] is None and a0[8] is None and \
                    f1 is B.relay_maxpool2d and a1[5:8] == (2, 2, 0) and a1[8] is a0[7] and B.relay_conv2d_pool2x2_pays(a0[0]):
                merged[i] = (self.calls[i:i + 2], B.relay_fused_conv2d_pool2x2, tuple(a0[:6]) + (a0[7], a1[9]))
            elif i - 1 not in merged and f0 is f1 is B.relay_fused_conv2d_bias_bn_relu and a1[1] is a0[7] and a0[6] is None and \
                    (a1[6] is None or a1[6] is a0[1]) and B.relay_conv2d_block_pays(a0[0], a1[0]):
                merged[i] = (self.calls[i:i + 2], B.relay_fused_conv2d_block, (*a0[:6], a0[7], a1[0], *a1[2:6], a1[7]))
            elif i - 1 not in merged and f0 is f1 is B.relay_qconv2d_requant and a1[1] is a0[7] and a0[4] is None and \
                    (a1[4] is None or a1[4] is a0[1]) and B.relay_conv2d_block_pays(a0[0], a1[0]):
                merged[i] = (self.calls[i:i + 2], B.relay_qconv2d_block, (*a0[:4], a0[6], a0[7], a1[0], a1[2], a1[3], a1[5], a1[6], a1[7]))
            elif f0 is B.relay_global_avgpool and f1 is B.relay_fused_dense_bias_act and a1[4] is a0[5] and a1[2] == a0[2] and \
                    a1[3] == a0[0] and B.relay_avgpool_dense_pays(*a0[:4], a1[1]):
                merged[i] = (self.calls[i:i + 2], B.relay_fused_avgpool_dense, (*a0[:4], a1[1], a0[4], *a1[5:8], a0[5], a1[8]))
        return merged

    def _combined_groups(self):
        """{i: (calls, function, arguments)} of two or three neighbouring convs into channel segments, or of one and the max pool of the tensor it
        reads, none reading what another of them writes, that run as one launch."""
        groups = {}
        at = lambda t: t.untyped_storage().data_ptr()
        for i in range(len(self.calls)):
            if i + 1 < len(self.calls) and not any(j + len(g[0]) > i for j, g in groups.items()):   # (a conv and the pool of the same tensor)
                (f0, a0), (f1, a1) = self.calls[i:i + 2]
                if f0 is B.relay_fused_conv2d_combined and f1 is B.relay_maxpool2d and a1[0] == B.RELAY_F16 and a1[8] is a0[1] and \
                        not any(at(t) in (at(a0[1]), at(a1[9])) for t in a0[8]) and B.relay_conv2d_combined_maxpool_pays(a0, a1):
                    groups[i] = (self.calls[i:i + 2], B.relay_fused_conv2d_combined_maxpool, (a0, a1))
                    continue
            for n in (3, 2):
                part = self.calls[i:i + n]
                if len(part) < n or any(f is not B.relay_fused_conv2d_combined for f, _ in part) or any(j + len(g[0]) > i for j, g in groups.items()):
                    continue
                if any(at(a[1]) == at(y) for _, a in part for _, b in part if a is not b for y in b[8]):
                    continue
                if B.relay_conv2d_combined_group_pays(*[a for _, a in part]):
                    groups[i] = (part, B.relay_fused_conv2d_combined_group, tuple(a for _, a in part))
                    break
        return groups

    def _image_stem(self):
        """(calls, function, arguments) of the launch that stands for the first two or three calls -- the padded copy of the image,
        the conv on it, its 3x3 / stride 2 / pad 1 max pool -- where the library takes them together and that pays, else None."""
        if len(self.calls) < 2 or self.calls[0][0] is not B.relay_pack_input_nhwc4:
            return None
        (_, a0), (f1, a1) = self.calls[:2]
        x, packed, d = a0[1], a0[2], a1[0]
        if len(a1) < 2 or a1[1] is not packed:
            return None
        pooled_only = f1 in (B.relay_fused_conv2d_bn_relu_maxpool, B.relay_qconv2d_requant_maxpool)
        if f1 is B.relay_fused_conv2d_bias_bn_relu and len(a1) == 9 and a1[6] is None and a1[8] is None:   # (no residual, no workspace)
            fn, args, y = B.relay_fused_image_conv2d, (d, x) + tuple(a1[2:6]), a1[7]
        elif f1 is B.relay_qconv2d_requant and a1[4] is None and a1[8] is None:
            fn, args, y = B.relay_qimage_conv2d, (d, x, a1[2], a1[3], a1[6]), a1[7]
        elif f1 is B.relay_fused_conv2d_bn_relu_maxpool:
            fn, args, y = B.relay_fused_image_conv2d, (d, x) + tuple(a1[2:6]), None
        elif f1 is B.relay_qconv2d_requant_maxpool:
            fn, args, y = B.relay_qimage_conv2d, (d, x, a1[2], a1[3], a1[4]), None
        else:
            return None
        if pooled_only:
            return (self.calls[:2], fn, args + (None, a1[-1])) if B.relay_image_conv2d_pays(d, True) else None
        if len(self.calls) > 2 and self.calls[2][0] is B.relay_maxpool2d:
            a2 = self.calls[2][1]
            if a2[5:8] == (3, 2, 1) and a2[8] is y and B.relay_image_conv2d_pays(d, True):
                return self.calls[:3], fn, args + (y, a2[9])
        return (self.calls[:2], fn, args + (y, None)) if B.relay_image_conv2d_pays(d, False) else None

    def _independent_pairs(self):
        """{i: (call i, call i + 1)} of calls that share a launch: plain convs over the same tensor, neither reading what the
        other writes, where the library takes the two together."""
        pairs = {}
        for i in range(len(self.calls) - 1):
            (f0, a0), (f1, a1) = self.calls[i], self.calls[i + 1]
            if i - 1 in pairs or f0 is not f1 or f0 not in (B.relay_fused_conv2d_bias_bn_relu, B.relay_qconv2d_requant):
                continue
            y0, y1 = a0[7], a1[7]
            reads = [t for t in a0[1:7] + a1[1:7] if torch.is_tensor(t)]
            if a0[1] is a1[1] and not any(t is y0 or t is y1 for t in reads) and B.relay_conv2d_pair_fusable(a0[0], a1[0]):
                pairs[i] = (self.calls[i], self.calls[i + 1])
        return pairs

    def _pointwise_behind(self, ops, i, group_of, absorbed):
        """Index of the plain 1x1 / stride 1 conv that is the only reader of depthwise conv i's output, or None."""
        op = ops[i]
        users = [j for j, o in enumerate(ops) if o.src == op.dst or o.res == op.dst or op.dst in (getattr(o, "srcs", None) or ())]
        if len(users) != 1 or users[0] != i + 1:
            return None
        q = ops[users[0]]
        plain = q.kind == "conv" and q.src == op.dst and q.r == 1 and q.stride == 1 and q.pad == 0 and not q.res
        if not plain or users[0] in group_of or users[0] in absorbed or q.dst in self.view_of or op.dst in self.view_of:
            return None
        return users[0]

    @staticmethod
    def _pool_behind(ops, i):
        """Index of the 3x3 / stride 2 / pad 1 max pool that is the only reader of conv i's output, or None."""
        op = ops[i]
        if op.res:
            return None
        users = [j for j, o in enumerate(ops) if o.src == op.dst or o.res == op.dst or op.dst in (o.srcs or ())]
        if len(users) != 1 or users[0] != i + 1:
            return None
        q = ops[users[0]]
        return users[0] if (q.kind == "maxpool" and q.src == op.dst and (q.r, q.stride, q.pad) == (3, 2, 1)) else None

    def _plan_concats(self, ops, batch, h, w, in_channels, cpad):
        """A channel concatenation is free when every tensor it joins is written by a conv: the
        conv stores straight into its channel range of the joined tensor.  Allocates those joined
        tensors and records view_of[name] = (joined tensor, first channel)."""
        self.view_of: Dict[str, tuple] = {}
        if not any(o.kind == "concat" for o in ops):
            return
        if self.mode != "f16" or not self.fused:
            raise ValueError("concatenation needs the fp16 fused pipeline")
        phys, hw = {"x": cpad}, {"x": (h, w)}      # physical channels and spatial size of every tensor
        producer = {}
        for o in ops:
            hi, wi = hw[o.src]
            out = lambda e: (e + 2 * o.pad - o.r) // o.stride + 1
            if o.kind in ("conv", "dwconv", "maxpool"):
                phys[o.dst] = o.cout if o.kind == "conv" else phys[o.src]
                hw[o.dst] = (out(hi), out(wi))
            elif o.kind in ("avgpool", "dense"):
                phys[o.dst], hw[o.dst] = (phys[o.src] if o.kind == "avgpool" else o.cout), (1, 1)
            elif o.kind == "concat":
                phys[o.dst], hw[o.dst] = sum(phys[s_] for s_ in o.srcs), hw[o.srcs[0]]
                off = 0
                for s_ in o.srcs:
                    if producer.get(s_) != "conv" or s_ in self.view_of or phys[s_] % 8 or hw[s_] != hw[o.dst]:
                        raise ValueError(f"concat {o.name}: {s_} must be a conv output of the same size, used in one "
                                         "concatenation, with a multiple of 8 channels")
                    self.view_of[s_] = (o.dst, off)
                    off += phys[s_]
                self.bufs[o.dst] = torch.empty((batch, *hw[o.dst], off), dtype=self.tdtype, device=self.dev)
            producer[o.dst] = o.kind

    def _emit_conv_views(self, members, mparams, batch):
        """One launch for one or more fp16 convs over the same input (a channel range of a wider
        tensor or a plain one), each storing into its own tensor or channel range."""
        op0 = members[0]          # (a member with the widest window: combine_parallel lists those first)
        cin_l, hi, wi = self.shape[op0.src]
        src = self.bufs[op0.src]
        cin_p = src.shape[-1]
        if any(m.res for m in members):
            raise ValueError(f"{op0.name}: a conv with a residual operand cannot store into a view")
        has_bias = mparams[0].get("bias") is not None
        has_bn = mparams[0].get("scale") is not None
        fold = self.fold_scale and has_bn
        any_relu = any(m.relu for m in members)
        mixed = any(m.r != op0.r or m.relu != any_relu for m in members)   # needs the per-segment windows / tails
        flags = B.flags_of(True if (has_bias or fold) else None, None if fold or not has_bn else True, None, any_relu)
        ktot = sum(m.cout for m in members)
        d = B.conv_desc(batch, cin_p, hi, wi, ktot, op0.r, op0.r, op0.stride, op0.pad, self.dtype, B.RELAY_NHWC, flags)
        ho, wo = B.relay_conv2d_out_shape(d)
        wp = torch.empty(B.relay_packed_weight_bytes(d), dtype=torch.uint8, device=self.dev)
        consts = {k: [] for k in ("bias", "scale", "shift")}
        ys, off = [], 0
        for m, p in zip(members, mparams):
            dm = B.conv_desc(batch, cin_p, hi, wi, m.cout, op0.r, op0.r, m.stride, op0.pad, self.dtype, B.RELAY_NHWC, flags)
            nbytes = B.relay_packed_weight_bytes(dm)
            wsrc = torch.from_numpy(np.ascontiguousarray(p["w"])).to(self.dev)
            if fold:
                consts["bias"].append(self._fold(m, p, wsrc, cin_l))
            else:
                consts["bias"].append(self._f32(p.get("bias")))
                consts["scale"].append(self._f32(p.get("scale")))
                consts["shift"].append(self._f32(p.get("shift")))
            if m.r != op0.r:      # a 1x1 member: its filters at the centre tap of the group's window, zeros around
                assert m.r == 1 and m.pad == 0 and op0.r % 2 == 1 and op0.pad == op0.r // 2 and m.stride == op0.stride
                wide = torch.zeros((m.cout, wsrc.shape[1], op0.r, op0.r), dtype=wsrc.dtype, device=self.dev)
                wide[:, :, op0.r // 2, op0.r // 2] = wsrc[:, :, 0, 0]
                wsrc = wide
            B.relay_prepack_conv2d_weights(dm, wsrc, cin_l, wp[off:off + nbytes])
            off += nbytes
            if m.dst in self.view_of:
                cat, c0 = self.view_of[m.dst]
                y = self.bufs[cat][..., c0:c0 + m.cout]
            else:
                y = torch.empty((batch, ho, wo, m.cout), dtype=self.tdtype, device=self.dev)
            assert tuple(y.shape) == (batch, ho, wo, m.cout)
            ys.append(y)
            self.bufs[m.dst], self.shape[m.dst] = y, (m.cout, ho, wo)
            self.keep.append(dm)
        joined = {k: (torch.cat(v) if v and v[0] is not None else None) for k, v in consts.items()}
        name = "+".join(m.name for m in members)
        if mixed:
            self._add(name, B.relay_fused_conv2d_combined_windows,
                      (d, src, src.stride(2), wp, joined["bias"], joined["scale"], joined["shift"],
                       [m.cout for m in members], ys, [y.stride(2) for y in ys],
                       [B.WINDOW_FULL if m.r == op0.r else B.WINDOW_CENTRE for m in members],
                       [1 if m.relu else 0 for m in members]))
        else:
            self._add(name, B.relay_fused_conv2d_combined,
                      (d, src, src.stride(2), wp, joined["bias"], joined["scale"], joined["shift"],
                       [m.cout for m in members], ys, [y.stride(2) for y in ys]))
        self.keep += [wp, d, joined]

    def _workspace(self, d):
        """Zeroed scratch of a conv whose reduction the library splits over workgroups (the deep
        layers at small batch), one buffer per conv so that convs on forked streams cannot share one."""
        need = B.relay_workspace_bytes(d)
        if need == 0:
            return None
        ws = torch.zeros(need, dtype=torch.uint8, device=self.dev)
        self.keep.append(ws)
        return ws

    def _fold(self, op, p, wsrc, cin_l):
        """Axis scale folding: multiplies the OIHW filters on the device by the conv's batch-norm
        scale, in place, and returns the bias that replaces "add bias, scale, shift"."""
        sc, sf = self._f32(p["scale"]), self._f32(p["shift"])
        B.relay_fold_scale_axis(self.dtype, op.cout, cin_l, op.r * op.r, B.FOLD_OUT, wsrc, sc, wsrc)
        folded = torch.empty(op.cout, dtype=torch.float32, device=self.dev)
        B.relay_fold_bias(op.cout, self._f32(p.get("bias")), sc, sf, folded)
        self.keep.append(folded)
        return folded

    def _f32(self, a):
        if a is None:
            return None
        t = torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(self.dev)
        self.keep.append(t)
        return t

    def _unfused_tail(self, op, p, cur, npix, c, res):
        """bias add, scale/shift, residual add, relu as separate launches, each into a new tensor."""
        def step(tag, ew, p0, p1, other):
            nonlocal cur
            nxt = torch.empty_like(cur)
            self._add(f"{op.name}.{tag}", B.relay_elementwise_f16, (ew, npix, c, cur, p0, p1, other, nxt))
            cur = nxt
        if p.get("bias") is not None:
            step("bias_add", B.EW_BIAS_ADD, self._f32(p["bias"]), None, None)
        if p.get("scale") is not None:
            step("scale_shift", B.EW_SCALE_SHIFT, self._f32(p["scale"]), self._f32(p["shift"]), None)
        if res is not None:
            step("add", B.EW_ADD, None, None, res)
        if op.relu:
            step("relu", B.EW_RELU, None, None, None)
        return cur

    def _add(self, name, fn, args):
        self.calls.append((fn, args))
        self.call_names.append(name)

    def load_input(self, x_nchw: np.ndarray) -> None:
        self.x_nchw.copy_(torch.from_numpy(np.ascontiguousarray(x_nchw)).to(self.dev))

    def run(self) -> None:
        """Enqueue the whole network on the current stream (layout conversion included).

        A conv whose output is only used as a later residual (the 1x1 shortcut of a ResNet
        block) is launched on a side stream between two events, so that it overlaps the block's
        first conv: both read the block input, neither reads the other.  The fork event is
        recorded BEFORE that first conv is enqueued, so the side stream waits only for the
        producer of the block input."""
        if not self.side_calls:
            if not self.pairs and not self.stem and not self.merged:
                for fn, args in self.calls:
                    fn(*args)
                return
            for _, _, fn, args in self._steps():
                fn(*args)
            return
        main = torch.cuda.current_stream()
        pending = fork = None
        for i, n, fn, args in self._steps():
            if i + n in self.side_calls:      # the next call runs beside this one
                fork = torch.cuda.Event()
                fork.record(main)
            if i in self.side_calls:
                self.side.wait_event(fork)
                with torch.cuda.stream(self.side):
                    fn(*args)
                    pending = torch.cuda.Event()
                    pending.record(self.side)
                continue
            if pending is not None and i in self.join_before:
                main.wait_event(pending)
                pending = None
            fn(*args)
        if pending is not None:
            main.wait_event(pending)

    def _steps(self):
        """(first call, number of calls, function, arguments) of every launch a run makes.  Calls share one only while all entries
        are those it was made for: `calls` may be edited, entries wrapped or cut off."""
        calls, steps, i = self.calls, [], 0
        same = lambda at, entries: len(calls) >= at + len(entries) and all(a is b for a, b in zip(entries, calls[at:]))
        # (a forced tile or split of the calling thread is for the conv of the list, which the image's launch would pass by)
        if self.stem and same(0, self.stem[0]) and not any(j <= len(self.stem[0]) for j in self.side_calls) and not B.relay_conv_forced():
            i = len(self.stem[0])
            steps.append((0, i) + tuple(self.stem[1:]))
        while i < len(calls):
            merged, pair = self.merged.get(i), self.pairs.get(i)
            if merged and same(i, merged[0]) and not self._crosses_streams(i, len(merged[0])):
                steps.append((i, len(merged[0])) + tuple(merged[1:]))
            elif pair and same(i, pair):
                steps.append((i, 2, B.relay_conv2d_pair, (pair[0][1], pair[1][1])))
            else:
                steps.append((i, 1) + tuple(calls[i]))
            i += steps[-1][1]
        return steps

    def _crosses_streams(self, i, n):
        """Does a fork or join fall between calls i .. i + n - 1, or a fork behind the last of them?"""
        return bool(self.side_calls) and (any(j in self.side_calls for j in range(i, i + n + 1)) or
                                          any(j in self.join_before for j in range(i + 1, i + n)))

    def launches(self):
        """(names of the calls joined by +, function, arguments) of what run() enqueues, in order."""
        return [("+".join(self.call_names[i:i + n]), fn, args) for i, n, fn, args in self._steps()]

    def capture(self) -> None:
        """Record run() into a HIP graph (kernel launches only; nothing in it clears memory).  Where that is a chain of the library's
        kernels, replay() can also enqueue the recorded launches one by one from native code.

        The list saves the idle time between two replays of a graph (4 to 6 us a pass) and costs the host 2.5 us a launch, the
        graph's replay 13 to 30 us whatever its length.  So the list runs passes of at most 6 launches (deep Q-network 21.4 -> 18.4 us one after
        another, 38 -> 28 waited for; the first ten operators of ResNet-18, six launches, 33 -> 30 and 46 -> 40, but waited for twelve, eight launches,
        53 -> 63) and passes with work for the whole chip in a launch, which keep the GPU busy longer than the host (an average of 400 K outputs:
        ResNet-18 of 7 images 129 -> 124 and 142 -> 137 us; of 3 images 106 -> 100, but waited for 117 -> 123).  In between (one image: 15 or 16 launches
        of 4 to 5 us) the list wins where the GPU has passes queued (ResNet-18 80 -> 75 us, int8 60 -> 58, MobileNet-v1 86 -> 83) and loses where it
        idles until the first launch (waited for, int8 ResNet-18 72 -> 69 to 87, MobileNet-v1 97 -> 108; with 80 us of a program's own work between
        passes 110 -> 125): see replay().  Such a graph is instantiated and launched once here, because its first launch takes 10 us
        more than a later one; any other that has a list is instantiated when it is first launched itself."""
        self.run()
        torch.cuda.synchronize(self.dev)
        g = PassGraph(keep_graph=True)
        with torch.cuda.graph(g):
            self.run()
        try:
            self.launch_list = B.LaunchList(g)
            launches = len(self.launches())
            outputs = self.batch * sum(c * h * w for c, h, w in self.shape.values())
            self.list_always = launches <= 6 or outputs >= 400_000 * launches
        except B.RelayError:
            self.launch_list = None
        if self.launch_list is None:
            g.instantiate()
        elif not self.list_always:
            g.replay()
        self.graph = g

    launch_list = None
    list_always = True
    _enqueued = threading.local()   # .at: when this thread last enqueued a pass of many short launches, of any network

    def replay(self) -> None:
        """Enqueue the captured pass on the current stream; refused (nothing enqueued, the capture stays usable) where that stream is
        being captured: run() is what a program records into a graph of its own.

        Between list and graph (capture()) a pass of many short launches goes by whether the GPU has work queued, for which the
        10 us since the calling thread's last such pass stand: asking the stream takes 20 us.  Both enqueue the same launches."""
        recorded = self.launch_list
        if recorded is None or not recorded.is_of(self.graph) or \
                not (self.list_always or time.perf_counter_ns() - getattr(self._enqueued, "at", 0) < 10_000):
            self.graph.replay()
        elif not recorded.run():
            raise B.RelayError(4, "a captured pass is not replayed into a stream that is being captured")
        if not self.list_always:
            self._enqueued.at = time.perf_counter_ns()

    def tensor(self, name: str) -> np.ndarray:
        """Download a named tensor as NCHW with the logical channel count."""
        if name == "x":
            return self.x_nchw.cpu().numpy()
        if name not in self.bufs:
            raise KeyError(f"{name} is not stored: its producer runs fused with the operator that reads it")
        c, _, _ = self.shape[name]
        t = self.bufs[name][..., :c].permute(0, 3, 1, 2).contiguous().cpu().numpy()
        return t
