"""Host-side replay of the few-token strips' pipeline (csrc/sq_thin.h): the
loader wave's counted waits over its LDS ring, the two operand buffers and the
register sets, for every strip the launcher can take.  Checked for each step s,
between the barrier of s and the next:

  (a) every copy of step s has completed under the wait before the barrier (a
      wait for n completes all but the n youngest);
  (b) the ring slot that a copy fills was last read before the barrier that
      precedes the copy;
  (c) the operands of s were written before the barrier of s, into a buffer
      whose last reader passed the barrier of s - 1;
  (d) all waves meet the same number of barriers, and no copy is in flight when
      the loader ends."""

import os
import re

import pytest

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_2609_04526_amd", "csrc")


def text(name):
    with open(os.path.join(CSRC, name)) as f:
        return f.read()


def launched():
    """(mode, MT, NT, KF, D, P) of every strip that the dispatch names."""
    found = re.findall(r"thin_go<kThin(Fwd|Dx), FMT, (\d+), (\d+), (\d+), (\d+), (\d+)>", text("sq_gemm.hip"))
    return sorted({(m, *map(int, v)) for m, *v in found})


def replay(MT, NT, KF, D, steps):
    PX = MT * KF
    assert D >= 3 and (D - 1) * PX <= 63
    landed, flight = set(), []                       # copies of a step, in issue order
    held = {}                                        # ring slot -> step
    read_step = {}                                   # slot -> interval (barrier index) of its last read
    issue_log = []

    def issue(step, slot, interval):
        prev = held.get(slot)
        if prev is not None:
            # (b) the step held before was read in interval `prev` (after barrier prev), which ends at barrier prev + 1
            assert read_step[prev] < interval, (step, prev)
        held[slot] = step
        flight.extend([step] * PX)
        issue_log.append(step)

    for d in range(D - 1):
        issue(d, d, -1)
    wr = D - 1
    for s in range(steps):
        keep = (D - 2) * PX                          # wait, then the barrier of s
        done = flight[:max(0, len(flight) - keep)]
        landed.update(done)
        del flight[:len(done)]
        assert s not in flight and s in landed, (s, flight)          # (a)
        assert held[s % D] == s
        read_step[s] = s                             # chains read slot s % D between barriers s and s + 1
        issue(s + D - 1, wr, s)
        wr = (wr + 1) % D
    flight.clear()                                   # (d) the last wait is for everything
    # (c) dequantising waves fill step s before barrier s, that is in interval s - 1; buffer s % 2 was read in interval s - 2
    for s in range(2, steps):
        assert (s - 2) < (s - 1) and (s - 2) % 2 == s % 2


@pytest.mark.parametrize("cfg", launched(), ids=str)
def test_ring_and_buffers(cfg):
    mode, MT, NT, KF, D, P = cfg
    for steps in range(1, 41):
        replay(MT, NT, KF, D, steps)
    # LDS of a workgroup, and its threads
    ops = NT * KF * (4 * (256 + 64) + 64) if mode == "Fwd" else 32 * KF * 32 * 2
    assert D * MT * KF * 1024 + 2 * ops <= 160 * 1024
    assert 64 * (NT + 1 + NT * KF // 2) <= 1024
    assert KF in (4, 8, 16) and P >= 2


def test_model_follows_the_kernel_source():
    """The waits, copies, reads and fills that the replay assumes, in their order."""
    src = text("sq_thin.h")
    body = src[src.index("__device__ __forceinline__ void thin_tile("):]
    loader = body[body.index("// ---- token rows"):body.index("// ---- weights")]
    seq = re.findall(r"issue\(d, d \* kSlot\)|thin_wait<[^;]*>\(\)|issue\(s \+ D - 1, wr\)", loader)
    assert seq == ["issue(d, d * kSlot)", "thin_wait<(D - 2) * PX, true>()", "issue(s + D - 1, wr)", "thin_wait<0, false>()"]
    chain = body[body.index("// ---- chains"):body.index("// ---- token rows")]
    step = chain[chain.index("auto step = "):]
    seq = re.findall(r"thin_wait<[^;]*>\(\)|read\(s, S\d\{\}|multiply\(", step[:step.index("slot = slot + kSlot")])
    assert seq == ["thin_wait<kThinAnyLoads, true>()", "read(s, S0{}", "multiply(", "read(s, S1{}", "multiply("]
    assert "ops + (s & 1) * kOps" in chain
    weights = body[body.index("// ---- weights"):]
    seq = re.findall(r"fill\(s, SET\)|load\(s \+ P, SET\)|thin_wait<[^;]*>\(\)", weights)
    assert seq == ["fill(s, SET)", "load(s + P, SET)", "thin_wait<kThinAnyLoads, true>()"]
    assert "ops + (s & 1) * kOps" in weights
    # the compiler may not move LDS accesses across a wait and its barrier
    wait = src[src.index("void thin_wait()"):src.index("constexpr int kThinAnyLoads")]
    assert re.search(r'asm volatile\("" ::: "memory"\);\s*wait_vm_lgkm0<n>\(\);\s*if \(BARRIER\) __builtin_amdgcn_s_barrier\(\);'
                     r'\s*asm volatile\("" ::: "memory"\);', wait)
