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
