"""Exchanges between the two waves of a marching strip, on the CPU: the buffers
that csrc/march_order.hpp gives each exchange, replayed over every order in
which two waves can run that the barriers allow.  A wave must read what the
other wrote for the same exchange."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2502_16818_amd", "csrc")

PROGRAM = """
#include <cstdio>
#include "march_order.hpp"
int main() {
    using namespace cdbm;
    std::printf("%d %d\\n", MARCH_TAKE, MARCH_ONE);
    for (int it = 0; it < 40; ++it) std::printf("%d %d\\n", march_buffer(it, 0), march_buffer(it, 1));
}
"""


def _table(tmp_path):
    src, exe = tmp_path / "order.cpp", tmp_path / "order"
    src.write_text(PROGRAM)
    cxx = shutil.which("g++") or shutil.which("clang++")
    subprocess.run([cxx, "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True, timeout=120)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout
    rows = [tuple(map(int, line.split())) for line in out.splitlines()]
    return rows[0], rows[1:]


def _exchanges(take, one, rows, buffer):
    """Buffers of a piece's exchanges in order: pieces of `rows` rows run pairs
    of iterations, and stage 2 only for rows of the piece."""
    seq = [buffer(it, 0) for it in range(take, take + one)]
    it, row = take + one, 0
    while row < rows:
        for _ in range(2):
            seq.append(buffer(it, 0))
            if row < rows:
                seq.append(buffer(it, 1))
            it, row = it + 1, row + 1
    return seq


def _stale_reads(seq):
    """Exchanges of which a wave can read another's values.  A wave's steps: 3 e
    write its half of exchange e, 3 e + 1 meet at the barrier, 3 e + 2 read."""
    end = 3 * len(seq)

    def holds(steps, b):   # the exchange whose values a wave's half of buffer b has
        done = [e for e in range(len(seq)) if 3 * e < steps and seq[e] == b]
        return done[-1] if done else None

    stale, seen, todo = set(), set(), [(0, 0)]
    while todo:
        s = todo.pop()
        if s in seen:
            continue
        seen.add(s)
        if s[0] % 3 == 1 and s[0] == s[1]:   # both at the barrier
            todo.append((s[0] + 1, s[1] + 1))
            continue
        for w in (0, 1):
            if s[w] == end or s[w] % 3 == 1:
                continue
            if s[w] % 3 == 2:
                e = s[w] // 3
                if holds(s[1 - w], seq[e]) != e:
                    stale.add(e)
            todo.append((s[0] + 1, s[1]) if w == 0 else (s[0], s[1] + 1))
    assert (end, end) in seen
    return stale


@pytest.mark.parametrize("rows", [1, 2, 3, 4, 7, 16])
def test_every_order_reads_its_own_exchange(tmp_path, rows):
    (take, one), table = _table(tmp_path)
    assert not _stale_reads(_exchanges(take, one, rows, lambda it, stage: table[it][stage]))


def test_one_buffer_in_the_fill_is_found(tmp_path):
    """A planted order: the exchanges of stage 1 alone all through buffer 0."""
    (take, one), _ = _table(tmp_path)
    assert _stale_reads(_exchanges(take, one, 4, lambda it, stage: stage)) == set(range(one))
