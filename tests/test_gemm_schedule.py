"""The hand-written synchronisation of the GEMM main loop, checked on the host: the loop's own statements
are read from k_gemm.hip and played for both wavefront groups (wm = 0 and 1).  An epoch is the stretch
between two workgroup barriers; what one wavefront did is ordered before another's action only if it was
done in an earlier epoch."""
import os
import re

import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2608_16798_amd", "csrc",
                   "k_gemm.hip")


def _loop_source():
    text = open(SRC).read()
    text = text[text.index("// Main loop."):text.index("// the epilogues reuse the LDS of the pipeline")]
    text = re.sub(r"//[^\n]*", "", text)
    start = text.index("copy_half(true, 0, 0, 0);")  # behind step_b's definition
    body = text.index("auto slice = [&]")
    end = text.index("\n  };", body)
    return text[start:body], text[body:end]


def _statements(src):
    return [s.strip() for s in re.split(r"[;{]", src) if s.strip()]


def _play(nk, wm, k_major):
    """Events of one group: (epoch, kind, (operand, buffer, half), slice), kinds copy / landed / read / taken."""
    prologue, body = _loop_source()
    state = dict(epoch=0)
    events, in_flight, reading = [], [], []

    def copy(op, h, kt, buf):
        events.append((state["epoch"], "copy", (op, buf, h), kt))
        in_flight.append(((op, buf, h), kt))

    def wait_copies(n):  # all but the newest n half tiles
        while len(in_flight) > n:
            events.append((state["epoch"], "landed", *in_flight.pop(0)))

    def read(op, buf, h, kt):
        events.append((state["epoch"], "read", (op, buf, h), kt))
        reading.append(((op, buf, h), kt))

    def wait_reads():
        while reading:
            events.append((state["epoch"], "taken", *reading.pop(0)))

    def run(stmts, env, kt):
        for s in stmts:
            m = re.match(r"if \(wm == (\d)\) (.*)", s)
            if m:
                if int(m.group(1)) != wm:
                    continue
                s = m.group(2)
            call = re.match(r"(copy_half|step_b|read_a|wait_vmcnt<IN_FLIGHT>|wait_lgkm0|block_barrier|mma)\((.*)\)$", s)
            if not call:
                assert not re.search(r"copy_half|step_b|read_|wait_|barrier", s), f"statement not understood: {s}"
                continue
            name = call.group(1)
            a = [eval(x, {}, env) for x in call.group(2).split(",")] if call.group(2) else []
            if name == "copy_half":
                copy("B" if a[0] else "A", a[1], a[2], a[3])
            elif name == "read_a":
                read("A", a[0], a[1], kt)
            elif name == "step_b":
                rb, rh, cb, ch, ckt = a
                read("B", rb, rh, kt + (rb != kt % 2))  # the other buffer holds the next slice
                copy("B", ch, ckt, cb)
                wait_copies(5)
                if k_major:  # its one asm statement waits for its reads too
                    wait_reads()
            elif name == "wait_vmcnt<IN_FLIGHT>":
                wait_copies(5)
            elif name == "wait_lgkm0":
                wait_reads()
            elif name == "block_barrier":
                state["epoch"] += 1

    base = dict(c0=0, c1=1, true=True, false=False)
    run(_statements(prologue), base, 0)
    for kt in range(nk):
        run(_statements(body), dict(base, kt=kt, buf=kt % 2, cur=kt % 2, nxt=1 - kt % 2), kt)
    if wm == 0:
        state["epoch"] += 1
    return events, state["epoch"]


@pytest.mark.parametrize("k_major", [False, True])
@pytest.mark.parametrize("nk", [1, 2, 3, 6])
def test_half_tiles_are_not_overwritten_under_a_read(nk, k_major):
    groups = [_play(nk, wm, k_major) for wm in (0, 1)]
    assert groups[0][1] == groups[1][1], "the groups pass the same number of barriers"
    events = [e for g, _ in groups for e in g]
    copies = [e for e in events if e[1] == "copy"]
    for g, _ in groups:
        reads = [e for e in g if e[1] == "read"]
        taken = [e for e in g if e[1] == "taken"]
        assert len(taken) == len(reads) or len(reads) - len(taken) == 1  # the last read is of a slice past the end
        assert len(reads) == 4 * nk + 1
        for i, (epoch, _, half, kt) in enumerate(reads):
            if kt >= nk:
                continue
            done = taken[i]
            assert done[2] == half
            # the slice was copied, by both groups, and its copies had landed in an earlier epoch
            landed = [e for e in events if e[1] == "landed" and e[2] == half and e[3] == kt]
            assert len(landed) == 2 and all(e[0] < epoch for e in landed), (half, kt)
            # and whoever overwrites it does so in an epoch after the read was waited for
            over = [e for e in copies if e[2] == half and e[3] == kt + 2]
            assert all(e[0] > done[0] for e in over), (half, kt)
