"""Waits that the compiler does not place: loads into LDS, and loads into registers written as inline assembly, are waited for by
hand.  The assembly of the kernels that have them is built for gfx950 and every path through it is walked; scalars that such
instructions read are looked at in the whole built library.  No GPU is needed."""
import concurrent.futures
import os
import re
import struct
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


OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
_OPERANDS = re.compile(r",(?![^\[]*\])")


def _scalars(text):
    named = {"vcc"} if "vcc" in text else set()
    for first, last, one in re.findall(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b", text):
        named |= {int(one)} if one else set(range(int(first), int(last) + 1))
    return named


def _scalars_written(text):
    """Scalar registers that an instruction of the vector or the scalar unit writes."""
    op, _, rest = text.partition(" ")
    if op.startswith(("s_cmp", "s_bitcmp", "s_wait", "s_nop", "s_cbranch", "s_branch", "s_barrier", "s_endpgm", "s_set", "s_sleep")):
        return set()
    args = _OPERANDS.split(rest)
    carry = op.startswith(("v_mad_u64", "v_mad_i64", "v_add_co", "v_sub_co", "v_subrev_co", "v_addc", "v_subb", "v_div_scale"))
    return _scalars(",".join(args[:2] if carry else args[:1]))


def _device_code(library):
    """The gfx950 code objects bundled in a library."""
    with open(library, "rb") as f:
        data = f.read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            offset, size, length = struct.unpack_from("<QQQ", data, entry)
            if size and b"gfx950" in data[entry + 24:entry + 24 + length]:
                yield data[at + offset:at + offset + size]
            entry += 24 + length
        at = data.find(magic, at + 24)


def _early_scalars(listing):
    """Memory instructions that read a scalar register less than five wait states after the vector unit wrote it."""
    found, count, name, before = [], 0, "", []
    for line in listing.splitlines():
        if line.startswith("<"):
            name, before = line, []
        if not line.startswith("\t"):
            continue
        text = line.split("//", 1)[0].strip()
        if text.startswith(("buffer_", "global_", "flat_", "scratch_")):
            count += 1
            read, states = _scalars(text), 0
            for earlier in reversed(before):
                if states >= 5 or not read:
                    break
                if earlier.startswith(("v_", "s_")):
                    hit = _scalars_written(earlier) & read
                    if hit and earlier.startswith("v_"):
                        found.append("%s: `%s`, %d states, `%s`" % (name[:80], earlier, states, text))
                        break
                    read -= hit                             # (the scalar unit waits for the vector unit's write, and a read of its own for it)
                states += int(earlier.split()[1]) + 1 if earlier.startswith("s_nop") else 1
        before = before[-7:] + [text]
    return found, count


def test_scalars_of_memory_instructions_are_old_enough(tmp_path):
    """Five wait states lie between a vector instruction that writes a scalar register (v_readlane, which brings spilled ones back, among them) and a
    memory instruction that reads it.  The compiler sees to it for its own; those written by hand have to by themselves."""
    from paper_2207_10741_amd import binding
    if not (os.path.exists(OBJDUMP) and os.path.exists(binding.LIB_PATH)):
        pytest.skip("needs the built library and llvm-objdump")
    found, count = [], 0
    for i, code in enumerate(_device_code(binding.LIB_PATH)):
        path = str(tmp_path / ("%d.elf" % i))
        with open(path, "wb") as f:
            f.write(code)
        listing = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", path], check=True, capture_output=True, text=True).stdout
        early, seen = _early_scalars(listing)
        found, count = found + early, count + seen
    assert count > 1000                                     # (the listing is one)
    assert not found, "\n".join(found[:20])
