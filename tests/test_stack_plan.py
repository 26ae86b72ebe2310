"""Host-side checks of what a planned stack run rests on, without a GPU: where the arena puts tensors, and what fc_run_calls
refuses before anything is enqueued."""
import ctypes
import random

import pytest

from paper_2207_10741_amd import binding as B, stacks, workloads


def _tensors(rng, n):
    """(op, op of the last reader, bytes) in op order: mostly read by the next op, some by a later one."""
    out = []
    for i in range(n):
        if rng.random() < 0.1:          # (an output the caller gets has no place in the arena)
            continue
        last = min(n - 1, i + rng.choice([0, 1, 1, 1, 2, 3, rng.randrange(1, n + 1)]))
        out.append((i, last, rng.choice([1, 255, 256, 257, 1000, 4096, 100000, rng.randrange(1, 1 << 20)])))
    return out


@pytest.mark.parametrize("rest", [0, 1, 2, 4, 6, 8, 12])
def test_arena_ranges_in_use_at_the_same_time_do_not_overlap(rest):
    rng = random.Random(1000 + rest)
    for _ in range(200):
        tensors = _tensors(rng, rng.randrange(1, 60))
        offsets, total = stacks._place(tensors, rest)
        assert len(offsets) == len(tensors)
        assert total == max([at + -(-size // 256) * 256 for at, (_, _, size) in zip(offsets, tensors)], default=0)
        assert all(at % 256 == 0 for at in offsets)
        for b, (op_b, _, size_b) in enumerate(tensors):
            for a in range(b):
                _, last_a, size_a = tensors[a]
                if last_a + rest >= op_b:       # a is still read, or resting, when b is written
                    assert offsets[a] + size_a <= offsets[b] or offsets[b] + size_b <= offsets[a], (a, b)


def test_arena_of_a_chain_reuses_its_ranges():
    chain = [(i, i + 1, 1000) for i in range(50)]
    assert stacks._place(chain, 0)[1] == 2 * 1024       # the tensor being read and the one being written
    assert stacks._place(chain, 4)[1] == 6 * 1024
    assert stacks._place([], 0) == ([], 0)


@pytest.mark.parametrize("net", ["resnet18", "resnet50_bottlenecks", "vgg16", "mobilenetv2"])
def test_ops_follow_what_they_read_and_unread_ones_follow_at_once(net):
    ops = getattr(workloads, net)()
    readers = {}
    for j, op in enumerate(ops):
        readers.setdefault(op.src, []).append(j)
    order = stacks._order(ops, readers)
    assert sorted(order) == list(range(len(ops))) and order[-1] == len(ops) - 1
    at = {i: k for k, i in enumerate(order)}
    at[-1] = -1
    for i, op in enumerate(ops):
        assert at[i] > at[op.src]
        if not readers.get(i) and i < len(ops) - 1:
            assert at[i] == at[op.src] + 1
    kept = [i for i in range(len(ops)) if readers.get(i)]
    assert [i for i in order if i in kept] == kept          # the others keep their order


@pytest.mark.parametrize("keep", [False, True])
@pytest.mark.parametrize("compact", [False, True])
def test_rows_nobody_can_see_stay_unwritten(keep, compact):
    """Chained: an op that only convs read leaves its irrelevant rows; of the ops nobody reads, only those whose output the caller gets are
    zero-filled, and none of them is handed on as a list."""
    stack = object.__new__(stacks.ConvStack)
    stack.ops, stack.n, stack.h, stack.w, stack.dtype, stack.relu = workloads.resnet50_bottlenecks(), 2, 30, 40, B.BF16, True
    stack.sizes = {-1: (30, 40)}
    for i, op in enumerate(stack.ops):
        hi, wi = stack.sizes[op.src]
        stack.sizes[i] = B.out_dims(B.conv_desc(2, hi, wi, 1, 1, (op.k, op.k), (op.stride, op.stride), (op.pad, op.pad), (1, 1), B.F32))
    stack.pyramid_steps = stack._pyramid_steps()
    plan = stacks._Plan(stack, True, keep, True, compact)
    calls = [c for _, part in plan.parts for c in part]
    read = {op.src for op in stack.ops}
    returned = {i for i, _, _ in plan.returned}
    assert returned == (set(range(len(stack.ops))) if keep else {len(stack.ops) - 1})
    alone = [i for i in range(len(stack.ops)) if i not in read]
    assert len(alone) == 5                                   # the four projections and the last layer
    for i, call in zip(plan.order, calls):
        skipped = bool(call.desc.flags & B.SKIP_ZERO_FILL)
        assert skipped == (i in read or i not in returned)
        if i not in read:
            assert not call.desc.flags & B.COMPACT_OUT


# ---- fc_run_calls ----

ADDR = 0x1000


def _run(calls, slots):
    arr, tab = (B.Call * max(len(calls), 1))(*calls), (ctypes.c_void_p * max(len(slots), 1))(*slots)
    return B.lib().fc_run_calls(arr, len(calls), tab, len(slots), None, 0, None)


def _conv(**over):
    f = dict(kind=B.CALL_CONV, x=0, mask_in=-1, w=1, bias=-1, mask_out=-1, idx=-1, count=-1, out=2)
    f.update(over)
    desc = f.pop("desc", B.conv_desc(1, 8, 8, 16, 16))
    return B.Call(desc, *(f[k] for k in ("kind", "x", "mask_in", "w", "bias", "mask_out", "idx", "count", "out")))


@pytest.mark.parametrize("kind", [B.CALL_CONV, B.CALL_DWCONV, B.CALL_MAXPOOL])
def test_run_calls_refuses_slots_and_kinds_out_of_range(kind):
    slots = [ADDR, 2 * ADDR, 3 * ADDR]
    for field in ("x", "mask_in", "w", "bias", "mask_out", "idx", "count", "out"):
        assert _run([_conv(kind=kind, **{field: 3})], slots) == -6
        assert _run([_conv(kind=kind, **{field: 2 ** 31 - 1})], slots) == -6
    assert _run([_conv(kind=3)], slots) == -3 and _run([_conv(kind=-1)], slots) == -3
    # found before the sound call in front is enqueued (its addresses are nobody's memory)
    assert _run([_conv(kind=kind), _conv(out=3)], slots) == -6
    assert _run([_conv(kind=kind), _conv(kind=7)], slots) == -3


def test_run_calls_refuses_what_its_layers_refuse():
    slots = [ADDR, 2 * ADDR, 3 * ADDR, ADDR + 8]
    assert _run([], slots) == 0 and _run([], []) == 0
    assert B.lib().fc_run_calls(None, 0, (ctypes.c_void_p * 1)(), 1, None, 0, None) == -1
    assert B.lib().fc_run_calls((B.Call * 1)(_conv()), 1, None, 0, None, 0, None) == -1
    assert B.lib().fc_run_calls((B.Call * 1)(_conv()), -1, (ctypes.c_void_p * 1)(), 1, None, 0, None) == -2
    assert B.lib().fc_run_calls((B.Call * 1)(_conv()), 1, (ctypes.c_void_p * 1)(), -1, None, 0, None) == -2
    for field in ("x", "w", "out"):
        assert _run([_conv(**{field: -1})], slots) == -1                # a required slot left NULL
        assert _run([_conv(kind=B.CALL_DWCONV, **{field: -1})], slots) == -1
        assert _run([_conv(**{field: 3})], slots) == -4                 # not 16-byte aligned
    assert _run([_conv(kind=B.CALL_MAXPOOL, x=-1)], slots) == -1 and _run([_conv(kind=B.CALL_MAXPOOL, out=-1)], slots) == -1
    assert _run([_conv(x=-2 ** 31)], slots) == -1                       # any negative slot is NULL
    assert _run([_conv(desc=B.conv_desc(1, 8, 8, 0, 16))], slots) == -2
    assert _run([_conv(mask_in=0)], slots) == -5                        # a mask without a list needs a workspace
    assert _run([_conv(idx=0)], slots) == -1                            # a list without its count
