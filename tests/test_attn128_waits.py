"""The wait states of the wide attention kernel's own MFMAs (csrc/attn128.hip: those that name accumulation registers), in the
assembly that the build's flags give.  The compiler does not know what is inside such an instruction, so that the order of the
code around it has to keep
  - two wait states between a vector instruction that writes one of its operands and the MFMA,
  - eleven between the MFMA (32x32x16, eight passes) and another instruction that reads or writes its result.
An instruction is one wait state, s_nop N is N + 1."""
import os
import re
import subprocess

import pytest

import __graft_entry__ as entry

BEFORE, AFTER = 2, 11


def _registers(text):
    """{"v12", "a3", ...} named in an operand."""
    out = set()
    for kind, one, first, last in re.findall(r"\b([va])(?:(\d+)|\[(\d+):(\d+)\])", text):
        lo, hi = (int(one), int(one)) if one else (int(first), int(last))
        out.update(f"{kind}{i}" for i in range(lo, hi + 1))
    return out


class Kernel:
    def __init__(self, asm):
        body = re.search(r"^\S*attn128_kernel\S*:.*?\n(.*?)^\.Lfunc_end", asm, re.S | re.M).group(1)
        self.code, self.labels = [], {}                       # instructions, label -> index of the next one
        for line in body.split("\n"):
            line = line.split(";")[0].strip()
            if line.endswith(":"):
                self.labels[line[:-1]] = len(self.code)
            elif line and not line.startswith("."):
                self.code.append(line)
        self.sources = {}                                     # index of a labelled instruction -> branches to it
        for i, line in enumerate(self.code):
            m = re.match(r"s_c?branch\S*\s+(\S+)", line)
            if m:
                self.sources.setdefault(self.labels[m.group(1)], []).append(i)
        parts = [re.match(r"(\S+)\s*(.*)", line).groups() for line in self.code]
        self.names = [p[0] for p in parts]
        operands = [p[1].split(", ") for p in parts]
        self.named = [_registers(p[1]) for p in parts]
        stores = ("ds_write", "global_store", "buffer_store", "v_cmp")
        self.written = [set() if n.startswith(stores) else _registers(o[0]) for n, o in zip(self.names, operands)]

    def before(self, i, states):
        """Instructions that may run fewer than `states` wait states in front of instruction i."""
        seen, todo = {}, [(i, 0)]
        while todo:
            at, passed = todo.pop()
            previous = list(self.sources.get(at, ()))
            if at > 0 and not re.match(r"s_branch|s_endpgm", self.names[at - 1]):
                previous.append(at - 1)
            for p in previous:
                if passed < seen.get(p, states):
                    seen[p] = passed
                    m = re.match(r"s_nop (\d+)", self.code[p])
                    todo.append((p, passed + (int(m.group(1)) + 1 if m else 1)))
        return [p for p in seen if self.names[p].startswith("v_")]

    def faults(self):
        own = [n.startswith("v_mfma") and any(r[0] == "a" for r in w) for n, w in zip(self.names, self.written)]
        assert sum(own) >= 64                                 # two halves of a tile twice, and the rest
        out = []
        for i, line in enumerate(self.code):
            if own[i]:
                out += [(self.code[p], line) for p in self.before(i, BEFORE) if not own[p] and self.written[p] & self.named[i]]
            elif any(r[0] == "a" for r in self.named[i]):
                out += [(self.code[p], line) for p in self.before(i, AFTER) if own[p] and self.written[p] & self.named[i]]
        return out


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "attn128.s")
    subprocess.run([entry.HIPCC] + entry.FLAGS + entry.VGPR_MFMA + ["--offload-device-only", "-S", os.path.join(entry.CSRC, "attn128.hip"),
                                                                    "-o", out], check=True, capture_output=True)
    with open(out) as f:
        return f.read()


def test_the_order_of_the_code_keeps_the_wait_states(assembly):
    assert Kernel(assembly).faults() == []


def test_a_copy_in_front_or_a_read_behind_is_found(assembly):
    """The check itself, on text that has the mistakes in it."""
    own = re.search(r"v_mfma_f32_32x32x16_bf16 (a\[(\d+):\d+\]), v\[(\d+):\d+\].*\n", assembly)
    first, operand = own.group(2), own.group(3)
    copy = assembly[:own.start()] + f"v_mov_b32_e32 v{operand}, v0\n\ts_nop 0\n\t" + assembly[own.start():]
    assert len(Kernel(copy).faults()) >= 1
    assert Kernel(copy.replace(f"v_mov_b32_e32 v{operand}, v0\n\ts_nop 0\n", f"v_mov_b32_e32 v{operand}, v0\n\ts_nop 1\n")).faults() == []
    read = assembly[:own.end()] + f"\ts_nop 9\n\tv_accvgpr_read_b32 v0, a{first}\n" + assembly[own.end():]
    assert len(Kernel(read).faults()) >= 1
    assert Kernel(read.replace("s_nop 9\n\tv_accvgpr", "s_nop 10\n\tv_accvgpr")).faults() == []
