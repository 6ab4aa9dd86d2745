"""The LDS schedule of the fused head's product loop (nt_stream), on the CPU.

The loop's two wavefront groups read and refill the same LDS halves and are
ordered by workgroup barriers and waits alone, so a missing wait shows on the
GPU only when a read is late.  Here the loads, reads, waits and barriers are
taken from the source in their order, walked for both groups, and checked:

* a half is read only after every group's loads of that stage were waited for
  before a barrier that the reader has passed;
* a half is refilled with another stage only after a barrier that follows the
  wait of every read of it.

Operands that are read and waited for in one step (K-major ones) only finish
earlier than modelled.
"""
import os
import re

import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_05774_amd", "csrc",
                   "k_lmhead.hip")
WORDS = r"src\.load_[uv]|src\.first|src\.advance|read_[uv]\(|wait_lds|wait_loads|phase_barrier|__syncthreads|[uv]1 = "
LOADS_PER_HALF = 2  # instructions of one load_u / load_v


def _block(text, at):
    """The text between the brace at or after `at` and its partner, and the position past it."""
    i = text.index("{", at)
    depth = 0
    for j in range(i, len(text)):
        depth += {"{": 1, "}": -1}.get(text[j], 0)
        if depth == 0:
            return text[i + 1:j], j + 1
    raise AssertionError("unbalanced braces")


def _steps(text):
    text = re.sub(r"//[^\n]*", "", text)
    return [s.strip() for s in re.split(r"[;{}]", text) if re.search(WORDS, s)]


def _source():
    """(steps before the stage loop, of a stage, after the loop)"""
    text = open(SRC).read()
    body, _ = _block(text, text.index("void nt_stream("))
    body, _ = _block(body, body.index("if (nk > 0)"))
    tiles = body.index("for (int tile")
    loop, end = _block(body, tiles)
    stage, stage_end = _block(loop, loop.index("for (int k"))
    assert not _steps(loop[:loop.index("for (int k")]) and not _steps(loop[stage_end:])
    return _steps(body[:tiles]), _steps(stage), _steps(body[end:])


def _slot(where, p):
    """Half (buffer * 4 + U0, U1, V0, V1) that a load's destination names."""
    buf = 0
    if "p ^ 1" in where:
        buf = p ^ 1
    elif where.startswith("cur"):
        buf = p
    elif "kBufElems" in where:
        buf = 1
    m = re.search(r"(\d?)\s*\*?\s*kHalfElems", where)
    return buf * 4 + (0 if m is None else int(m.group(1) or 1))


class _Group:
    """One wavefront group's walk: loads and reads with the barriers passed when issued and when waited for."""

    def __init__(self, wr, stages):
        self.wr, self.stages, self.barriers = wr, stages, 0
        self.at = {"u1": 0, "u2": 0, "v1": 0, "v2": 0}
        self.loads, self.reads = [], []  # [slot, stage, issued, waited]

    def step(self, s, k, p):
        m = re.match(r"if \(wr == (\d)\) (.*)", s)
        if m:
            if int(m.group(1)) != self.wr:
                return
            s = m.group(2)
        if m := re.match(r"src\.load_([uv])\((\d), ([uv]\d), (.*)\)$", s):
            slot = _slot(m.group(4).replace("mine + ", ""), p)
            assert slot % 4 == (0 if m.group(1) == "u" else 2) + int(m.group(2)), s
            self.loads += [[slot, self.at[m.group(3)], self.barriers, None] for _ in range(LOADS_PER_HALF)]
        elif m := re.match(r"read_([uv])\((?:fv\d, )?(0|p|p \^ 1), (\d)\)$", s):
            buf = {"0": 0, "p": p, "p ^ 1": p ^ 1}[m.group(2)]
            stage = 0 if k is None else k + (m.group(2) == "p ^ 1")
            self.reads.append([buf * 4 + (0 if m.group(1) == "u" else 2) + int(m.group(3)), stage, self.barriers, None])
        elif m := re.match(r"wait_loads<(\d+)>\(\)$", s):
            for x in self.loads[:len(self.loads) - int(m.group(1))]:
                x[3] = self.barriers if x[3] is None else x[3]
        elif s == "wait_lds()":
            for x in self.reads:
                x[3] = self.barriers if x[3] is None else x[3]
        elif s in ("phase_barrier()", "__syncthreads()"):
            self.barriers += 1
        elif s == "src.advance(u2, v2)":
            self.at["u2"] = self.at["v2"] = min(self.at["u2"] + 1, self.stages - 1)
        elif m := re.match(r"(u)1 = u2$|(v)1 = v2$", s):
            self.at[s[:2]] = self.at[s[-2:]]
        else:
            assert re.match(r"src\.first\(u2, v2\)$", s), f"step not understood: {s}"


def _walk(wr, stages):
    before, stage, after = _source()
    g = _Group(wr, stages)
    for s in before:
        g.step(s, None, 0)
    for k in range(stages):
        for s in stage:
            g.step(s, k, k % 2)
    for s in after:
        g.step(s, stages, stages % 2)
    return g


def _faults(stages):
    groups = [_walk(0, stages), _walk(1, stages)]
    assert groups[0].barriers == groups[1].barriers, "the groups meet at different numbers of barriers"
    out = []
    for g in groups:
        for slot, stage, issued, waited in g.reads:
            if stage >= stages:  # past the last stage: read, never used
                continue
            for o in groups:
                own = [x for x in o.loads if x[0] == slot and x[1] == stage]
                if not any(x[3] is not None and x[3] < issued for x in own):
                    out.append(f"group {g.wr} reads half {slot} of stage {stage} before group {o.wr}'s loads landed")
                for _, other, at, _ in (x for x in o.loads if x[0] == slot and x[1] > stage):
                    if waited is None or at <= waited:
                        out.append(f"group {o.wr} refills half {slot} with stage {other} after barrier {at}, "
                                   f"group {g.wr} waits for its read of stage {stage} after barrier {waited}")
    return out


@pytest.mark.parametrize("stages", (1, 2, 3, 4, 9))
def test_every_read_is_between_its_loads_and_the_refill(stages):
    assert _faults(stages) == []


def test_a_missing_wait_is_found():
    """The check sees a wait that is not there: each one left out in turn, in a copy of the steps."""
    before, stage, after = _source()
    waits = [i for i, s in enumerate(stage) if s.startswith("wait")]
    assert len(waits) == 6
    for i in waits:
        cut = (before, stage[:i] + stage[i + 1:], after)
        with pytest.MonkeyPatch.context() as mp:
            mp.setitem(globals(), "_source", lambda cut=cut: cut)
            assert _faults(6), stage[i]
