"""Products and lane reads written as assembly: the compiler sees neither them nor what they wait for, so every statement has to bring
its own wait states.  Checked in the assembly that the sources compile to, along every way through it, and not for the default
schedule alone: others put other instructions in front of such a statement."""
import os
import re
import subprocess

import pytest

from paper_2605_06046_amd.build import CSRC, FLAGS, HIPCC

# wait states: a vector instruction's result, before a product takes it as an operand, and before a lane of it is read;
# a product's sums, before anything but a product touches them (16 passes at most, and 3)
OPERAND, LANE, SUMS = 2, 1, 19
SCHEDULES = ["", "gcn-iterative-ilp", "ilpmax"]

_REG = re.compile(r"(?<![\w.])([av])(?:(\d+)|\[(\d+):(\d+)\])(?!\w)")


def _regs(text):
    return {f"{f}{k}" for f, one, lo, hi in _REG.findall(text) for k in (range(int(one), int(one) + 1) if one else range(int(lo), int(hi) + 1))}


class _Instruction:
    def __init__(self, text, by_hand):
        self.text, self.by_hand = text, by_hand
        self.op, _, rest = text.partition(" ")
        operands = [x.strip() for x in re.split(r",(?![^\[]*\])", rest)]
        self.product = self.op.startswith("v_mfma")
        self.vector = self.op.startswith("v_") and not self.product
        stores = "store" in self.op or self.op.startswith("ds_write") or "load_lds" in self.op
        self.writes = set() if stores else _regs(operands[0])
        self.reads = _regs(rest) if stores else _regs(",".join(operands[1:]))
        if "swap" in self.op:
            self.writes = self.reads = _regs(rest)
        self.states = 1 + (int(operands[0]) if self.op == "s_nop" else 0)
        self.next = []


def _kernels(assembly):
    """{kernel: its instructions, each with the indices of those that can follow it}."""
    out, code, labels, by_hand = {}, None, None, False
    for line in assembly.splitlines():
        line = line.strip()
        if line.startswith(";;#ASM"):
            by_hand = line.startswith(";;#ASMSTART")
            continue
        line = line.split(";")[0].strip()
        if line.startswith(".Lfunc_end"):
            code = None
        elif line.endswith(":"):
            if line.startswith("_Z"):
                code, labels = [], {}
                out[line[:-1]] = (code, labels)
            elif code is not None:
                labels[line[:-1]] = len(code)
        elif code is not None and re.match(r"[a-z]+_\w+", line):
            code.append(_Instruction(line, by_hand))
    for code, labels in out.values():
        for k, x in enumerate(code):
            if x.op not in ("s_endpgm", "s_branch"):
                x.next.append(k + 1)
            if x.op == "s_branch" or x.op.startswith("s_cbranch"):
                x.next.append(labels[x.text.split()[1]])
    return {name: code for name, (code, _) in out.items()}


def _within(code, k, states):
    """What can run behind instruction k with fewer than so many wait states between."""
    todo, seen = [(n, 0) for n in code[k].next], {}
    while todo:
        n, gone = todo.pop()
        if n < len(code) and gone < states and seen.get(n, states) > gone:
            seen[n] = gone
            yield code[n]
            todo += [(m, gone + code[n].states) for m in code[n].next]


def _too_early(code):
    for k, x in enumerate(code):
        if x.vector and x.writes:
            for y in _within(code, k, OPERAND):
                if y.by_hand and y.product and y.reads & x.writes:
                    yield x.text, y.text
            for y in _within(code, k, LANE):
                if y.by_hand and y.op.startswith("v_read") and y.reads & x.writes:
                    yield x.text, y.text
        if x.by_hand and x.product:
            for y in _within(code, k, SUMS):
                if not y.product and (y.reads | y.writes) & x.writes:
                    yield x.text, y.text


def _compile(source, schedule, path):
    options = [f for f in FLAGS if f not in ("-fPIC", "-shared")] + (["-mllvm", f"-misched={schedule}"] if schedule else [])
    return subprocess.Popen([HIPCC, *options, "--cuda-device-only", "-S", "-o", path, os.path.join(CSRC, source)], stderr=subprocess.DEVNULL)


def test_the_check_sees_what_comes_too_early():
    code = lambda *lines: _kernels("_Zk:\n" + "\n".join(lines) + "\ns_endpgm\n.Lfunc_end0:")["_Zk"]
    hand = lambda *lines: (";;#ASMSTART", *lines, ";;#ASMEND")
    product = "v_mfma_f32_16x16x32_bf16 a[0:3], v[8:11], v[0:3], a[0:3]"
    write = "v_mov_b32_e32 v2, v7"
    assert list(_too_early(code(write, *hand(product)))) and list(_too_early(code(write, "s_nop 0", *hand(product))))
    assert not list(_too_early(code(write, *hand("s_nop 1", product)))) and not list(_too_early(code(write, product)))
    assert list(_too_early(code(".L1:", *hand(product), write, "s_cbranch_scc1 .L1")))                    # around a loop
    read = "v_accvgpr_read_b32 v20, a3"
    assert list(_too_early(code(*hand(product), "s_nop 15", read))) and not list(_too_early(code(*hand(product, "s_nop 15", "s_nop 2"), read)))
    assert list(_too_early(code(write, *hand("v_readlane_b32 s64, v2, 0"))))


@pytest.mark.parametrize("source", ["fea_sweep_mfma.hip", "fea_hash.hip"])
def test_statements_wait_for_themselves(source, tmp_path):
    paths = {s: str(tmp_path / f"{s or 'default'}.s") for s in SCHEDULES}
    running = [_compile(source, s, p) for s, p in paths.items()]
    assert [r.wait(timeout=300) for r in running] == [0] * len(running)
    for schedule, path in paths.items():
        with open(path) as f:
            kernels = _kernels(f.read())
        assert any(x.by_hand and x.op.startswith(("v_mfma", "v_readlane")) for code in kernels.values() for x in code)
        for name, code in kernels.items():
            found = list(_too_early(code))
            assert not found, f"schedule {schedule or 'as by default'}, {name}: {found[:3]} and {len(found)} in all"
