"""Wait states of the compiled kernels: between some instructions the hardware
wants a number of others, and the compiler, which keeps them elsewhere, does not
look into inline assembly.  The assembly of each kernel file, compiled with the
library's flags, is searched along every path."""
import os
import re
import subprocess

import pytest

from paper_2002_03000_amd import build

LANE_OPS = ("v_readlane", "v_readfirstlane", "v_writelane")
TRANS = ("v_rcp", "v_rsq", "v_sqrt", "v_exp", "v_log", "v_sin", "v_cos")


def _registers(operand):
    operand = operand.strip().strip("|").lstrip("-").strip("|")
    m = re.fullmatch(r"([sv])(\d+)", operand)
    if m:
        return {(m[1], int(m[2]))}
    m = re.fullmatch(r"([sv])\[(\d+):(\d+)\]", operand)
    if m:
        return {(m[1], i) for i in range(int(m[2]), int(m[3]) + 1)}
    return {"vcc": {("s", "vcc_lo"), ("s", "vcc_hi")}, "exec": {("s", "exec")},
            "vcc_lo": {("s", "vcc_lo")}, "vcc_hi": {("s", "vcc_hi")}}.get(operand, set())


class _Instruction:
    def __init__(self, text, line):
        self.text, self.line = text, line
        parts = text.split(None, 1)
        self.op = parts[0]
        rest = parts[1] if len(parts) > 1 else ""
        self.operands = [o.strip().split()[0] for o in re.split(r",(?![^\[]*\])", rest) if o.strip()]
        self.vector = self.op.startswith("v_")
        self.written, self.read = set(), set()
        if not self.vector:
            for o in self.operands:
                self.read |= _registers(o)
            return
        outputs = 1
        if re.match(r"v_(add|sub|subrev|addc|subb|subbrev)_co_|v_div_scale|v_mad_[ui]64", self.op):
            outputs = 2
        if self.op.startswith("v_cmpx"):
            self.written = _registers("exec") | _registers("vcc")
            outputs = 1 if self.operands[0] in ("vcc", "exec") else 0
        for o in self.operands[:outputs]:
            self.written |= _registers(o)
        for o in self.operands[outputs:]:
            self.read |= _registers(o)

    def waits(self):
        return int(self.operands[0], 0) + 1 if self.op == "s_nop" else 1

    def rules(self):
        """(what a vector instruction before this one wrote, wait states it must be behind)"""
        if self.op.startswith(LANE_OPS):
            yield _registers("exec"), 4, False
            if not self.op.startswith("v_readfirst"):
                yield _registers(self.operands[2]), 4, False       # (the lane's number)
            if not self.op.startswith("v_write"):
                yield _registers(self.operands[1]), 1, False
        scalar = {r for r in self.read if r[0] == "s" and r[1] != "exec"}
        if self.vector:
            yield scalar, 2, False
            if not self.op.startswith(TRANS):
                yield {r for r in self.read if r[0] == "v"}, 1, True
        elif re.match(r"(global|buffer|flat|scratch)_", self.op):
            yield scalar, 5, False


def _short_waits(lines):
    code, labels = [], {}
    for number, line in enumerate(lines, 1):
        m = re.match(r"([.\w$]+):", line)
        if m:
            labels[m[1]] = len(code)
        text = line.split(";")[0].strip()
        if re.match(r"[sv]_|ds_|global_|buffer_|flat_|scratch_", text):
            code.append(_Instruction(text, number))
    before = {}                       # instructions that may run just before one
    for i, x in enumerate(code):
        if x.op not in ("s_branch", "s_endpgm", "s_setpc_b64"):
            before.setdefault(i + 1, []).append(i)
        if x.op == "s_branch" or x.op.startswith("s_cbranch"):
            before.setdefault(labels[x.operands[0]], []).append(i)
    short = []
    for i, x in enumerate(code):
        for registers, need, trans in x.rules():
            if not registers:
                continue
            todo, best = [(p, 0) for p in before.get(i, [])], {}
            while todo:
                j, waited = todo.pop()
                if waited >= need or best.get(j, need) <= waited:
                    continue
                best[j] = waited
                y = code[j]
                if y.vector and y.written & registers and (not trans or y.op.startswith(TRANS)):
                    short.append(f"{y.line}: {y.text}  ->  {x.line}: {x.text}  ({waited} of {need})")
                    continue
                todo += [(p, waited + y.waits()) for p in before.get(j, [])]
    return len(code), short


def test_the_search_finds_a_short_wait():
    lines = ["a:", "v_cmpx_lt_u32_e32 v1, v2", "ds_write_b32 v3, v4", "s_mov_b64 exec, -1", "s_cbranch_vccz b",
             "s_nop 0", "b:", "v_readlane_b32 s0, v5, s1"]
    assert len(_short_waits(lines)[1]) == 1            # (3 states over the branch, 4 past it)
    lines[2:2] = ["s_nop 0"]
    assert _short_waits(lines) == (7, [])
    assert len(_short_waits(["v_cmp_lt_u32_e64 s[2:3], v1, v2", "s_nop 0", "v_bcnt_u32_b32 v0, s3, 0"])[1]) == 1


@pytest.mark.parametrize("source", ["pperm_kernels.hip", "pperm_probe.hip"])
def test_kernels_keep_their_wait_states(source, tmp_path):
    out = tmp_path / "kernels.s"
    subprocess.run(["hipcc", "--offload-arch=gfx950", *build.FLAGS, "--cuda-device-only", "-S",
                    os.path.join(build.HERE, "csrc", source), "-o", str(out)],
                   check=True, capture_output=True, timeout=300)
    count, short = _short_waits(out.read_text().splitlines())
    assert count > 1000 and not short, short[:5]
