"""Runs a conv stack (workloads.Op list) through the library: mask propagation and
kept-position lists are built once per (mask, window geometry) and shared by every
layer that sees the same mask through the same geometry (Sec. III-B: one mask,
rescaled per layer) - by one fc_mask_pyramid call per pass when the mask levels form
a chain, as they do in a feed-forward network; each conv is one fc_focused_conv2d
call, each depthwise conv one fc_focused_dwconv2d call.

Plumbing only: the order of library calls and which tensor feeds which.  The calls of a pass are
laid out once per way of running the stack and enqueued by one fc_run_calls.  Max-pools
(not part of the paper's method) go through the library's helper, which with a mask
computes only the pooled positions the mask keeps.
"""
from __future__ import annotations

import ctypes
from typing import Dict, List, Optional

import numpy as np

from . import binding as B
from . import synth


MAX_PYRAMIDS = 16
HEAD_CALLS = 6
ARENA_CACHED = 224 << 20    # bytes of an arena that the last cache level (256 MB) holds beside weights and input


class _Plan:
    """The fc_run_calls sequence of one way of running a stack.

    Slots: 0 the input, 1 its mask, then mask / list / count of every pyramid level, weights and bias of
    every layer, the outputs.  All are filled in per run; the plan itself holds no address.  Outputs that the
    caller does not get live in one arena, at offsets such that tensors in use at the same time do not overlap."""

    def __init__(self, stack: "ConvStack", masked: bool, keep_outputs: bool, chain: bool, compact: bool):
        ops, n = stack.ops, len(stack.ops)
        readers = stack._readers()
        n_slots = 2 + (3 * len(stack.pyramid_steps) if masked else 0)

        def slot():
            nonlocal n_slots
            n_slots += 1
            return n_slots - 1

        out_slot = {-1: 0}
        compacted = set()
        calls = []
        self.dtype = B.torch_dtype(stack.dtype)
        self.levels = [(i, stack._level_of[i] if masked else -1) for i in range(n)]
        params = []         # (place in the order, op, slot of its weights, slot of its bias)
        self.returned, arena_ops, arena_slots = [], [], []
        self.order = _order(ops, readers)
        place = {i: at for at, i in enumerate(self.order)}
        # outputs that only the op behind reads, both of them 1x1 convs of unit stride: the library may run the two as one, unless irrelevant
        # rows are to be cleared (their ranges kept longer for nothing cost a zero-filled MobileNetV2, batch 32, 468 -> 478 us)
        next_only = [not keep_outputs and (chain or not masked) and at + 1 < n and readers.get(i) == [self.order[at + 1]] and stack._pointwise(i) and
                     stack._pointwise(self.order[at + 1]) for at, i in enumerate(self.order)]
        for at, i in enumerate(self.order):
            op = ops[i]
            ho, wo = stack.sizes[i]
            shape = (stack.n, ho, wo, op.c_out)
            m_in = m_out = idx = count = -1
            if masked:
                src_level, level = stack._level_of[op.src], stack._level_of[i]
                m_in = 1 if src_level < 0 else 2 + 3 * src_level
                m_out, idx, count = (2 + 3 * level + k for k in range(3))
            src = out_slot[op.src]
            out_slot[i] = slot()
            if op.kind == "maxpool":
                hi, wi = stack.sizes[op.src]
                d = B.conv_desc(stack.n, hi, wi, op.c_in, op.c_in, (op.k, op.k), (op.stride, op.stride), (op.pad, op.pad),
                                (1, 1), stack.dtype)
                calls.append(B.Call(d, B.CALL_MAXPOOL, src, -1, -1, -1, m_out, -1, -1, out_slot[i]))
            else:
                # (an output that nobody reads and the caller does not get: its irrelevant rows are nobody's either; the four
                # projections of a ResNet-50 on 32 frames of 120 x 160 wrote 640 MB instead of 330)
                unseen = not readers.get(i) and not keep_outputs and i < n - 1
                skip = chain and masked and (unseen or stack._gated_readers_only(i, readers))
                extra = B.SKIP_ZERO_FILL if skip else 0
                if op.src in compacted:
                    extra |= B.COMPACT_IN
                if compact and stack._compact_out(i, skip, readers):
                    extra |= B.COMPACT_OUT
                    compacted.add(i)
                    shape = (stack.n * ho * wo, op.c_out)
                w, b = slot(), slot()
                params.append((at, i, w, b))
                if op.kind == "dwconv":
                    # labels come from the input mask inside the call: no list, no workspace
                    calls.append(B.Call(stack.desc(i, flags_extra=extra), B.CALL_DWCONV, src, m_in, w, b, -1, -1, -1,
                                        out_slot[i]))
                else:
                    calls.append(B.Call(stack.desc(i, flags_extra=extra | B.WORKSPACE_READY), B.CALL_CONV, src, m_in, w, b,
                                        m_out, idx, count, out_slot[i]))
            if keep_outputs or i == n - 1:
                self.returned.append((i, out_slot[i], shape))
            else:
                # (a reader that may run as one with the op behind it reads this output for as long as that op runs)
                last = max(place[j] for j in readers.get(i, [i]))
                arena_ops.append((at, last + next_only[last], int(np.prod(shape)) * self.dtype.itemsize))
                arena_slots.append(out_slot[i])
        self.returned.sort()
        # the pass is enqueued in two parts: the device runs the first layers while the host fills in the others' slots
        # (MobileNetV2's 104 tensors take it tens of microseconds)
        cut = min(HEAD_CALLS, n)
        cut += next_only[cut - 1]       # (not between two ops that may run as one)
        spans = [(lo, hi) for lo, hi in ((0, cut), (cut, n)) if hi > lo]
        self.parts = [([q[1:] for q in params if lo <= q[0] < hi], (B.Call * (hi - lo))(*calls[lo:hi])) for lo, hi in spans]
        self.unseen = [bytes(next_only[lo:hi]) for lo, hi in spans]
        self.slots = ctypes.c_void_p * n_slots
        # A range is given out again some ops after its tensor's last reader while the arena stays inside the
        # chip's last cache level: writing over what the ops just before have read or written costs (MobileNetV2,
        # batch 32: 427 us with ranges reused at once, 403 us six ops later; after 512 MB of other data 458 and 437 us;
        # the other networks within 1 % either way, warm and cold).  A larger arena is packed tightly
        # (ResNet-50 on 12 frames of 100 x 100: 711 us tight in 153 MB, 735 us in 322 MB).
        for rest in (12, 8, 6, 4, 2, 0):
            offsets, self.arena_bytes = _place(arena_ops, rest)
            if self.arena_bytes <= ARENA_CACHED:
                break
        self.in_arena = list(zip(arena_slots, offsets))


def _order(ops, readers):
    """The order the ops are enqueued in: their own, but an op that nobody reads (a block's projection; not the last op) directly
    after the op it reads.  Later it would stand between a block's last layer and its reader and put its own output between
    them in the last cache level (ResNet-50, 32 frames of 120 x 160: the 256 -> 64 layer behind it 60 -> 49 us, a chained pass 1667 -> 1639, E4M3
    1093 -> 1055)."""
    n = len(ops)
    early = [i for i in range(n - 1) if not readers.get(i)]
    order = [i for i in range(n) if i not in early]
    for i in reversed(early):
        order.insert(order.index(ops[i].src) + 1 if ops[i].src >= 0 else 0, i)
    return order


def _place(tensors, rest: int):
    """Offsets for (op, op of the last reader, bytes), and the bytes in all: first fit, in the order the ops run; a
    range is taken from its tensor's own op to `rest` ops after the last reader's."""
    placed, total = [], 0
    for i, last, size in tensors:
        size = -(-size // 256) * 256
        at = 0
        for p_at, p_size in sorted((a, sz) for a, sz, p_last in placed if p_last >= i - rest):
            if at + size <= p_at:
                break
            at = max(at, p_at + p_size)
        placed.append((at, size, last))
        total = max(total, at + size)
    return [at for at, _, _ in placed], total


class ConvStack:
    def __init__(self, ops, n: int, h: int, w: int, dtype: int = B.BF16, seed: int = 0, relu: bool = True):
        import torch
        self.torch = torch
        self.ops = list(ops)
        self.n, self.h, self.w, self.dtype = n, h, w, dtype
        self.dev = torch.device("cuda:0")
        self.relu = relu
        if dtype == B.FP8 and not all(op.kind == "conv" and op.c_in % 16 == 0 and op.c_out % 16 == 0 for op in self.ops):
            raise ValueError("an 8-bit stack takes convolutions with multiples of 16 channels only")
        self.weights: Dict[int, object] = {}
        self.biases: Dict[int, object] = {}
        self.host_weights: Dict[int, np.ndarray] = {}
        self.host_biases: Dict[int, np.ndarray] = {}
        for i, op in enumerate(self.ops):
            if op.kind not in ("conv", "dwconv"):
                continue
            if op.kind == "dwconv":
                wt = np.ascontiguousarray(synth.he_weights(op.c_out, op.k, op.k, 1, dtype, seed, i, 2)[..., 0])
            else:
                wt = synth.he_weights(op.c_out, op.k, op.k, op.c_in, dtype, seed, i, 2)
            bs = synth.bias(op.c_out, seed, i, 3)
            self.host_weights[i], self.host_biases[i] = wt, bs
            self.weights[i] = self._to_dev(wt)
            self.biases[i] = torch.from_numpy(bs).to(self.dev)
        # spatial size of every op's output
        self.sizes = {-1: (h, w)}
        for i, op in enumerate(self.ops):
            hi, wi = self.sizes[op.src]
            d = B.conv_desc(n, hi, wi, 1, 1, (op.k, op.k), (op.stride, op.stride), (op.pad, op.pad), (1, 1), B.F32)
            self.sizes[i] = B.out_dims(d)
        # one workspace for all layers (calls are ordered on one stream): lets small layers
        # split their reduction over more workgroups
        need = max(B.workspace_bytes(self.desc(i)) for i, op in enumerate(self.ops) if op.kind == "conv")
        self.workspace = torch.empty((need,), dtype=torch.uint8, device=self.dev)
        # its arrival counters are cleared once here; every library call leaves them at zero,
        # so the calls carry FC_WORKSPACE_READY and none of them launches a clear
        B.ready_workspace(self.workspace)
        # the mask levels the ops need, when they form one chain (input -> level 0 -> level 1 ...):
        # then one fc_mask_pyramid call per pass builds all of them
        self.pyramid_steps = self._pyramid_steps()
        self._pyramids: Dict[int, object] = {}
        self._plans: Dict[tuple, _Plan] = {}

    def _same_view(self, i: int) -> bool:
        op = self.ops[i]
        return op.stride == 1 and self.sizes[i] == self.sizes[op.src] and op.pad == (op.k - 1) // 2

    def _pyramid_steps(self):
        """The windows that take each mask level to the next, in the order the ops first need them,
        or None when the levels do not form a single chain (then every level is built by its own
        fc_mask_downsample + fc_active_index_compact calls)."""
        level_of = {-1: -1}       # op -> level its output mask is (-1: the input mask)
        plans: Dict[tuple, int] = {}
        steps = []
        for i, op in enumerate(self.ops):
            src_level = level_of[op.src]
            key = (src_level, op.stride, (op.k - 1) // 2 - op.pad, self.sizes[i])
            if self._same_view(i) and src_level >= 0:
                level = src_level
            elif key in plans:
                level = plans[key]
            else:
                if src_level != len(steps) - 1:
                    return None
                steps.append(((op.k, op.k), (op.stride, op.stride), (op.pad, op.pad), (1, 1)))
                level = plans[key] = len(steps) - 1
            level_of[i] = level
        self._level_of = level_of
        return steps if 0 < len(steps) <= B.MAX_PYRAMID_LEVELS else None

    def _to_dev(self, storage: np.ndarray):
        torch = self.torch
        if self.dtype == B.F32:
            return torch.from_numpy(np.ascontiguousarray(storage, dtype=np.float32)).to(self.dev)
        if self.dtype == B.FP8:
            return torch.from_numpy(np.ascontiguousarray(storage, dtype=np.uint8)).to(self.dev).view(torch.float8_e4m3fn)
        t = torch.from_numpy(np.ascontiguousarray(storage).view(np.int16)).to(self.dev)
        return t.view(torch.bfloat16 if self.dtype == B.BF16 else torch.float16)

    def desc(self, i: int, out_dtype: Optional[int] = None, flags_extra: int = 0) -> B.ConvDesc:
        op = self.ops[i]
        hi, wi = self.sizes[op.src]
        flags = (B.RELU if (self.relu and op.relu) else 0) | flags_extra
        if out_dtype is None and self.dtype == B.FP8:
            out_dtype = B.FP8       # an 8-bit stack hands on 8-bit activations
        return B.conv_desc(self.n, hi, wi, op.c_in, op.c_out, (op.k, op.k), (op.stride, op.stride),
                           (op.pad, op.pad), (1, 1), self.dtype, out_dtype, flags)

    def _pointwise(self, i: int) -> bool:
        op = self.ops[i]
        return op.kind == "conv" and op.k == 1 and op.stride == 1 and op.pad == 0

    def _matrix_core_shape(self, i: int) -> bool:
        op = self.ops[i]
        if self.dtype == B.FP8:
            return op.kind == "conv" and op.c_in % 16 == 0 and op.c_out % 16 == 0 and op.k * op.k <= 32
        return (op.kind == "conv" and self.dtype in (B.BF16, B.F16) and op.c_in % 8 == 0 and op.c_out % 8 == 0
                and op.k * op.k <= 32)

    def _pyramid(self, mask):
        """The prepared pyramid call of a mask tensor; the last few masks' are kept."""
        pyr = self._pyramids.get(mask.data_ptr())
        if pyr is None or pyr.mask_in is not mask:
            self._pyramids.pop(mask.data_ptr(), None)
            if len(self._pyramids) >= MAX_PYRAMIDS:
                del self._pyramids[next(iter(self._pyramids))]
            pyr = self._pyramids[mask.data_ptr()] = B.PreparedPyramid(mask, self.pyramid_steps)
        return pyr

    def _readers(self):
        readers: Dict[int, List[int]] = {}
        for j, op in enumerate(self.ops):
            readers.setdefault(op.src, []).append(j)
        return readers

    def _gated_readers_only(self, i: int, readers) -> bool:
        return bool(readers.get(i)) and all(self.ops[j].kind in ("conv", "dwconv") for j in readers[i])

    def _compact_out(self, i: int, skip: bool, readers) -> bool:
        """May op i hand its output on as a list of kept rows?"""
        return (skip and bool(readers.get(i)) and self.ops[i].kind == "conv" and self._matrix_core_shape(i)
                and all(self._pointwise(j) and self._matrix_core_shape(j) for j in readers[i]))

    def _run_planned(self, x, mask, keep_outputs: bool, chain: bool, compact: bool):
        way = (mask is not None, keep_outputs, chain, compact)
        plan = self._plans.get((way, self.relu))
        if plan is None:
            plan = self._plans[way, self.relu] = _Plan(self, *way)
        B._require_cuda(x, mask)
        torch = self.torch
        slots = plan.slots()
        slots[0] = x.data_ptr()
        masks: Dict[int, object] = {-1: mask}
        if mask is not None:
            pyr = self._pyramid(mask)
            levels = pyr()
            slots[1] = mask.data_ptr()
            at = 2
            for level in levels:
                for t in level:
                    slots[at] = t.data_ptr()
                    at += 1
            for i, level in plan.levels:
                masks[i] = levels[level][0]
        else:
            for i, _ in plan.levels:
                masks[i] = None
        outs: Dict[int, object] = {-1: x}
        dev = x.device
        if plan.arena_bytes:
            arena = torch.empty((plan.arena_bytes,), dtype=torch.uint8, device=dev)
            base = arena.data_ptr()
            for slot, offset in plan.in_arena:
                slots[slot] = base + offset
        # (a small network's pass is bound by these two loops and the launches: a tensor like x is 0.2 us cheaper to make than
        # one of a stated type and device, and the tensors' checks stand here instead of in calls)
        like_x = x.dtype == plan.dtype
        for i, slot, shape in plan.returned:
            out = outs[i] = x.new_empty(shape) if like_x else x.new_empty(shape, dtype=plan.dtype)
            slots[slot] = out.data_ptr()
        weights, biases = self.weights, self.biases
        for (params, calls), unseen in zip(plan.parts, plan.unseen):
            for i, w_slot, b_slot in params:        # whatever tensors the dicts hold now
                w, b = weights[i], biases[i]
                if not (w.is_cuda and w.is_contiguous() and (b is None or (b.is_cuda and b.is_contiguous()))):
                    raise ValueError("tensors must be contiguous device tensors")
                slots[w_slot] = w.data_ptr()
                if b is not None:
                    slots[b_slot] = b.data_ptr()
            B.run_calls(calls, slots, self.workspace, unseen=unseen)
        return outs, masks

    def run(self, x, mask=None, keep_outputs: bool = True, chain: bool = False, canary=None, compact: bool = False):
        """x: device NHWC tensor; mask: device uint8 [N,H,W] or None (dense).
        Returns (outputs, masks): per-op output tensors and per-op output masks
        (index -1 = the stack's input).

        chain: a conv whose output is read only by other convs leaves its irrelevant rows
        unwritten (FC_SKIP_ZERO_FILL): every reader gates its taps by the same mask, so those
        rows are never looked at (Sec. III-A: irrelevant pixels are excluded from the
        product; Sec. III-B: the mask is the same all the way).  Outputs that a pooling
        layer reads, and those nobody reads that the caller gets, are still zero-filled.
        compact (with chain): a conv read only by 1x1 convs of unit stride writes its kept rows
        compacted, in list order (FC_COMPACT_OUT), and those readers read them that way
        (FC_COMPACT_IN): they see the same mask through the same geometry, hence the same list.
        canary: value every conv output buffer is pre-filled with (tests)."""
        if canary is None and (mask is None or self.pyramid_steps is not None):
            return self._run_planned(x, mask, keep_outputs, chain, compact)
        readers = self._readers()
        compacted: Dict[int, bool] = {}   # op -> its output is stored compacted
        outs: Dict[int, object] = {-1: x}
        masks: Dict[int, object] = {-1: mask}
        plans: Dict[tuple, tuple] = {}
        produced: Dict[int, tuple] = {}   # 0/1 masks this run wrote, with their kept lists
        levels = None                     # all mask levels from one call, taken in order
        if mask is not None and self.pyramid_steps is not None:
            levels = list(self._pyramid(mask)())
        last_use = {}
        for i, op in enumerate(self.ops):
            last_use[op.src] = i
        for i, op in enumerate(self.ops):
            src, m_in = outs[op.src], masks[op.src]
            geo = ((op.k, op.k), (op.stride, op.stride), (op.pad, op.pad), (1, 1))
            plan = None
            if m_in is not None:
                hi, wi = self.sizes[op.src]
                same_view = self._same_view(i)
                # two windows with the same stride, the same centre-tap offset and the same output
                # size keep the same positions (a 3x3/2 pad 1 conv and the 1x1/2 projection beside it)
                key = (id(m_in), op.stride, (op.k - 1) // 2 - op.pad, self.sizes[i])
                if same_view and id(m_in) in produced:
                    # the window is centred and does not change the resolution: the mask this op
                    # keeps is the (already 0/1) mask it reads, and so is the kept list
                    plan = produced[id(m_in)]
                elif key in plans:
                    plan = plans[key]
                elif levels is not None:
                    m_out, idx, count = levels.pop(0)
                    plan = plans[key] = produced[id(m_out)] = (m_out, idx, count)
                else:
                    m_out = B.mask_downsample(m_in, *geo)
                    idx, count = B.active_index_compact(m_out)
                    plan = plans[key] = produced[id(m_out)] = (m_out, idx, count)
            if op.kind in ("conv", "dwconv"):
                skip = chain and plan is not None and self._gated_readers_only(i, readers)
                extra = B.WORKSPACE_READY | (B.SKIP_ZERO_FILL if skip else 0)
                out = None
                ho, wo = self.sizes[i]
                if compacted.get(op.src, False):
                    extra |= B.COMPACT_IN
                if compact and self._compact_out(i, skip, readers):
                    extra |= B.COMPACT_OUT
                    compacted[i] = True
                    out = (self.torch.empty if canary is None else
                           (lambda *a, **k: self.torch.full(*a, canary, **k)))(
                        (self.n * ho * wo, op.c_out), dtype=B.torch_dtype(self.dtype), device=self.dev)
                elif canary is not None:
                    out = self.torch.full((self.n, ho, wo, op.c_out), canary, dtype=B.torch_dtype(self.dtype),
                                          device=self.dev)
                d = self.desc(i, flags_extra=extra)
                if op.kind == "dwconv":
                    # labels come from the input mask inside the call: no list, no workspace
                    d.flags &= ~B.WORKSPACE_READY
                    outs[i] = B.focused_dwconv2d(d, src, self.weights[i], self.biases[i],
                                                 mask_in=m_in if plan is not None else None, out=out)
                elif plan is None:
                    outs[i] = B.focused_conv2d(d, src, self.weights[i], self.biases[i], out=out,
                                               workspace=self.workspace)
                else:
                    outs[i] = B.focused_conv2d(d, src, self.weights[i], self.biases[i], mask_in=m_in,
                                               mask_out=plan[0], idx=plan[1], count=plan[2], out=out,
                                               workspace=self.workspace)
            else:
                # with a mask, only the pooled positions it keeps are computed; the rest is zero
                outs[i] = B.maxpool2d(src, op.k, op.stride, op.pad, self.dtype,
                                      keep=None if plan is None else plan[0])
            masks[i] = None if plan is None else plan[0]
            if not keep_outputs:
                for j in [j for j in outs if j != i and last_use.get(j, -2) <= i and j != -1]:
                    del outs[j]
        return outs, masks

    def conv_flops(self, masks_host: Optional[Dict[int, np.ndarray]] = None):
        """(dense FLOPs, kept FLOPs) of the stack; kept needs the host copies of the masks."""
        dense = kept = 0.0
        for i, op in enumerate(self.ops):
            if op.kind not in ("conv", "dwconv"):
                continue
            ho, wo = self.sizes[i]
            per_pos = 2.0 * op.k * op.k * op.c_in * (op.c_out if op.kind == "conv" else 1)
            dense += self.n * ho * wo * per_pos
            if masks_host is not None:
                kept += float(np.count_nonzero(masks_host[i])) * per_pos
        return dense, kept
