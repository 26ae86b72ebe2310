"""Waits that the compiler does not place: loads into LDS, and loads into registers written as inline assembly, are waited for by
hand.  The assembly of the kernels that have them is built for gfx950 and every path through it is walked; no GPU is needed."""
import concurrent.futures
import os
import re
import subprocess

import pytest

from paper_2207_10741_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CSRC = os.path.join(os.path.dirname(build.__file__), "csrc")


class Kernel:
    """A kernel's instructions in order; `after` gives the places control may go to from one."""

    def __init__(self, lines):
        self.code, self.by_hand, self.label = [], [], {}
        inside = False
        for line in lines:
            text = line.split(";", 1)[0].strip()
            if ";#ASMSTART" in line or ";#ASMEND" in line:
                inside = ";#ASMSTART" in line
            elif text.endswith(":"):
                self.label[text[:-1]] = len(self.code)
            elif text and not text.startswith("."):
                self.code.append(text)
                self.by_hand.append(inside)

    def after(self, at):
        op, _, rest = self.code[at].partition(" ")
        if op.startswith("s_endpgm"):
            return []
        if op == "s_branch":
            return [self.label[rest.strip()]]
        return [at + 1] + ([self.label[rest.strip()]] if op.startswith("s_cbranch") else [])


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{source: {kernel's mangled name: Kernel}}"""
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    tmp = tmp_path_factory.mktemp("asm")

    def assemble(source):
        out = str(tmp / (source + ".s"))
        subprocess.run([HIPCC, *build.HIPCC_FLAGS, "-w", "-I", os.path.join(build.ROOT, "include"), "-I", CSRC, "--cuda-device-only", "-S",
                        os.path.join(CSRC, source), "-o", out], check=True, stderr=subprocess.DEVNULL)
        found, name, lines = {}, None, []
        with open(out) as f:
            for line in f:
                start = re.match(r"(_Z\w+):", line)
                if start:
                    name, lines = start.group(1), []
                elif line.startswith(".Lfunc_end") and name:
                    found[name], name = Kernel(lines), None
                elif name:
                    lines.append(line)
        return found

    sources = ("fc_conv_small.hip", "fc_conv_reg.hip")
    with concurrent.futures.ThreadPoolExecutor(len(sources)) as pool:
        return dict(zip(sources, pool.map(assemble, sources)))


def _named(found, part):
    chosen = {name: k for name, k in found.items() if part in name}
    assert chosen
    return chosen


def _is_lds_load(text):
    return text.startswith("buffer_load") and text.endswith(" lds")


def test_lists_in_lds_lie_behind_a_barrier(kernels):
    """The lists of rows to clear lie where other waves' loads put weights: a wave waits for its own loads, and only the barrier after
    that for the others'.  (Words in LDS are lists' and a flag's; operands and sums are written by sixteen bytes.)"""
    for name, k in _named(kernels["fc_conv_small.hip"], "k_conv_small").items():
        loads = [at for at, text in enumerate(k.code) if _is_lds_load(text)]
        assert loads and any(t.startswith("ds_write_b32") for t in k.code), name
        seen, todo = set(), [n for at in loads for n in k.after(at)]
        while todo:
            at = todo.pop()
            if at in seen or k.code[at].startswith("s_barrier"):
                continue
            seen.add(at)
            assert not k.code[at].startswith("ds_write_b32"), "%s: `%s` while another wave's load may be on its way" % (name, k.code[at])
            todo += k.after(at)


def _registers(text):
    """Vector registers that an instruction names."""
    named = set()
    for first, last, one in re.findall(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b", text):
        named |= {int(one)} if one else set(range(int(first), int(last) + 1))
    return named


def _is_memory(text):
    return text.startswith(("buffer_load", "buffer_store", "buffer_atomic", "global_", "flat_", "scratch_"))


def _unwaited(k, at):
    """A place where the registers of the load at `at` are named, or the kernel ends, before a wait that covers the load; None if there is none."""
    written = _registers(k.code[at].split(",", 1)[0])
    seen, todo = set(), [(n, 0) for n in k.after(at)]       # (place, requests after the load)
    while todo:
        here = todo.pop()
        if here in seen:
            continue
        seen.add(here)
        place, later = here
        text = k.code[place]
        wait = re.search(r"vmcnt\((\d+)\)", text) if text.startswith("s_waitcnt") else None
        if wait and int(wait.group(1)) <= later:
            continue
        # (a multiply-add of 32 bits names a pair as its addend, whose high half is whatever lies there)
        spare = re.match(r"(v_mad_u64_u32 .*)v\[(\d+):\d+\]$", text)
        if text.startswith("s_endpgm") or _registers(spare.expand(r"\1v\2") if spare else text) & written:
            return text
        later = min(later + _is_memory(text), 63)
        todo += [(n, later) for n in k.after(place)]
    return None


@pytest.mark.parametrize("source,part,loads", [("fc_conv_small.hip", "k_conv_small_once", 9), ("fc_conv_reg.hip", "k_conv_f32_rounds", 9)])
def test_loads_written_by_hand_are_waited_for(kernels, source, part, loads):
    """The compiler does not know that the registers of such a load are still to be written: until a wait that covers it nothing may name
    them, on any path, and no path may end without one (there the compiler is free to use them for something else)."""
    for name, k in _named(kernels[source], part).items():
        by_hand = [at for at, text in enumerate(k.code) if k.by_hand[at] and _is_memory(text) and not _is_lds_load(text)]
        assert len(by_hand) == loads, name                  # entry, label, four of the bias, three of the mask
        for at in by_hand:
            found = _unwaited(k, at)
            assert found is None, "%s: `%s` after `%s`" % (name, found, k.code[at])
