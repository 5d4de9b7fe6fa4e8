"""The explicit waits of the weight-gradient kernels, checked on a model of their own
source: the statements from the first stage load to the end of the main loop are
executed here, with loads completing in issue order and LCVQ_WAIT_VM*(n) leaving at
most n of a wave's loads in flight.  A stage may be read for step s only after a
barrier before which its loads for s had completed (the other waves fill it too), and
refilled only after a barrier behind the last read of its old contents.  The compiler
may sink the prologue's register loads (used in the loop only) down to their first
use, so the waits have to hold with those loads in place and with them sunk."""
import os
import re

import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_10531_amd", "csrc",
                   "lcvq_gemm.hip")


def _body(kernel):
    """The statements of the kernel's prologue and main loop, as Python."""
    text = open(SRC).read()
    text = text[re.search(r"void %s\(" % kernel, text).start():]
    text = text[text.index("\n  issue(0"):text.index("\n  mfma_drain();")]
    text = re.sub(r"//[^\n]*|#pragma[^\n]*|__builtin_amdgcn_sched_barrier\(0\);", "", text)
    text = re.sub(r"auto (\w+) = \[&\]\(([^)]*)\) \{",
                  lambda g: "def %s(%s) {" % (g[1], ", ".join(p.split()[-1] for p in g[2].split(","))), text)
    out, pos = [], 0

    def space():
        nonlocal pos
        while pos < len(text) and text[pos] in " \n;":
            pos += 1

    def paren():  # the text inside the parentheses at pos
        nonlocal pos
        depth, start = 0, pos
        while True:
            depth += {"(": 1, ")": -1}.get(text[pos], 0)
            pos += 1
            if depth == 0:
                return text[start + 1:pos - 1]

    def expr(e):
        e = re.sub(r"\bint (\w+) =", r"\1 =", e.strip())
        e = re.sub(r"\+\+(\w+)|(\w+)\+\+", lambda g: "%s += 1" % (g[1] or g[2]), e)
        e = re.sub(r"\b(b0|b1)\[", r"\1_[", e)
        return e.replace("&&", " and ").replace("true", "True").replace("false", "False")

    def statement(ind):
        nonlocal pos
        space()
        pad = "  " * ind
        if text[pos] == "{":
            pos += 1
            space()
            while text[pos] != "}":
                statement(ind)
                space()
            pos += 1
            return
        head = re.match(r"(for|if) \(|def \w+\([^)]*\) ", text[pos:])
        if head and head[1] == "for":
            pos += 4
            init, cond, step = paren().split(";")
            if init.strip():
                out.append(pad + expr(init))
            out.append(pad + "while %s:" % expr(cond))
            statement(ind + 1)
            out.append(pad + "  " + expr(step))
        elif head and head[1] == "if":
            pos += 3
            out.append(pad + "if %s:" % expr(paren()))
            statement(ind + 1)
        elif head:
            out.append(pad + head[0].strip() + ":")
            pos += len(head[0])
            statement(ind + 1)
        else:
            end = text.index(";", pos)
            out.append(pad + re.sub(r"rd\([^,]*,", "rd(", expr(text[pos:end])).replace("\n", " "))
            pos = end + 1

    while True:
        space()
        if pos >= len(text):
            return "\n".join(out)
        statement(0)


class Model:
    """Loads of one wave in issue order (every wave runs the same program)."""

    def __init__(self, sunk):
        self.sunk, self.in_loop, self.held = sunk, False, []
        self.loads, self.done = [], 0             # issue order; the first `done` have completed
        self.ready = 0                            # loads complete before the last barrier
        self.stage, self.last_read = [None] * 4, [-1] * 4   # step a stage holds; barrier count at its last read
        self.barriers, self.faults = 0, []

    def load(self, what, count):
        if self.sunk and not self.in_loop and what[0] == "A":
            self.held.append((what, count))
        else:
            self.loads += [what] * count

    def issue(self, step, count):
        st = step % 4
        if self.last_read[st] >= self.barriers:
            self.faults.append("stage %d refilled for step %d with no barrier after its last read" % (st, step))
        self.stage[st] = step
        self.loads += [("B", step)] * count

    def wait(self, n):
        self.done = max(self.done, len(self.loads) - n)

    def barrier(self):
        self.barriers += 1
        self.ready = self.done

    def read(self, step):
        st = step % 4
        if self.stage[st] != step:
            self.faults.append("stage %d holds step %s, read for step %d" % (st, self.stage[st], step))
        if ("B", step) in self.loads[self.ready:]:
            self.faults.append("step %d read with its loads in flight" % step)
        self.last_read[st] = self.barriers

    def matrix(self, key):  # the instructions that use register load `key`
        self.in_loop = True
        for what, count in self.held:
            self.loads += [what] * count
        self.held = []
        last = max(i for i, what in enumerate(self.loads) if what == key)
        self.done = max(self.done, last + 1)      # the compiler's own wait


class Any:
    def __getitem__(self, i):
        return self


def _run(kernel, KBt, sunk, text):
    M = Model(sunk)
    env = dict(KBt=KBt, b0=Any(), b1=Any(), b0_=Any(), b1_=Any(), LCVQ_BARRIER=M.barrier, LCVQ_WAIT_VM=M.wait,
               LCVQ_WAIT_VM_LGKM0=M.wait)
    if kernel == "k_gemm_dw_half":
        env.update(issue=lambda kb: M.issue(kb, 4), load_a=lambda kk2, kb: M.load(("A", kk2, kb), 4),
                   rd=lambda kb, nb, kk2: M.read(kb))
        step = [0, 0]

        def half(kk2, b, nxt, rkb, rkk2):
            M.matrix(("A", kk2, step[kk2]))
            step[kk2] += 1
            M.read(rkb)
    else:
        state = dict(read=0)
        env.update(issue=lambda st, kb: (M.issue(kb, 8), None)[1] if st == kb % 4 else M.faults.append("stage"),
                   load_a=lambda buf, kk2, kb: M.load(("A", kk2, kb), 4),
                   rd=lambda st, nb, kk2: M.read(0))
        step = [0, 0]

        def half(buf, kk2, b, nxt, rst, rkk2):
            M.matrix(("A", kk2, step[kk2]))
            step[kk2] += 1
            s = step[kk2] - 1 + kk2               # reads the second half of its own step, or the first of the next
            if rst != s % 4:
                M.faults.append("stage")
            M.read(s)
    env["half"] = half
    exec(text, env)
    assert step == [KBt, KBt]
    assert M.done == len(M.loads), "loads in flight after the loop"
    return M.faults


@pytest.mark.parametrize("sunk", [False, True], ids=["in_place", "sunk"])
@pytest.mark.parametrize("KBt", [4, 8, 20])
@pytest.mark.parametrize("kernel", ["k_gemm_dw", "k_gemm_dw_half"])
def test_stages_are_complete_when_read(kernel, KBt, sunk):
    faults = _run(kernel, KBt, sunk, _body(kernel))
    assert not faults, faults[:4]


def test_the_model_sees_a_short_wait():
    """A wait that leaves the next step's loads in flight is found (mistake planted in the text)."""
    text = _body("k_gemm_dw")
    assert "LCVQ_WAIT_VM(20)" in text
    assert _run("k_gemm_dw", 8, False, text.replace("LCVQ_WAIT_VM(20)", "LCVQ_WAIT_VM(36)"))
