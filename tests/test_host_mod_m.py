"""The reduction modulo m of the generic product (include/rlx_arith.hpp,
compiled for the host) on products that take its rare branch: a carry out of
word 16, a borrow out of word 8, a top word of all ones, and a value of the
second fold at or above 2^576.  A Python model of the folds counts how often
the operands reach each condition; the products themselves are compared with
plain integers."""
import random
import subprocess

import pytest

import oracle as O
from test_host_arith import from_words, harness, words  # noqa: F401  (fixture)

B32 = 1 << 32


def conditions(p):
    """Rare conditions of the reduction of p < 2^1152."""
    low, high = p % 2 ** 576, p >> 576
    t1 = low + (high << 240) - high
    lo, hi = t1 % 2 ** 576, t1 >> 576
    s = lo % 2 ** 544 + ((hi << 240) % 2 ** 544)
    carry = s >> 544
    borrow = lo % 2 ** 288 + ((hi << 240) % 2 ** 288) < hi or (s % 2 ** 288) < hi
    r17 = (lo >> 544) == B32 - 1
    return {"carry": carry != 0, "borrow": borrow, "top": r17, "overflow": lo + (hi << 240) - hi >= 2 ** 576}


def operands():
    m = O.M
    rng = random.Random(11)
    out = []

    def target(t):
        # random factor x and the y with x y = t (mod m)
        x = rng.randrange(1, m)
        out.append((x, t * pow(x, -1, m) % m))
    for _ in range(60):
        t = rng.randrange(m)
        target(t % 2 ** 544 + ((B32 - 1) << 544))            # top word of all ones
        target(m - 1 - rng.randrange(2 ** 200))
        target((t % 2 ** 256) + ((B32 - 1) << 256) + (t >> 288 << 288))   # word 8 all ones after a borrow
        target((t >> 544 << 544) + (t % 2 ** 500))           # word 16 zero after a carry
        target(rng.randrange(2 ** 240))
        target(rng.randrange(2 ** 16))
    # x 2^575 has the upper half H = x >> 1: H (2^240 - 1) just below a
    # multiple of 2^576, so the second fold passes 2^576
    for a in (1, 2, 7, 2 ** 40 + 1, 2 ** 200 + 5, 2 ** 238):
        h = ((a + 1) * 2 ** 576 - 1) // (2 ** 240 - 1)
        for x in (2 * h, 2 * h + 1, 2 * h - 2):
            if 0 < x < m:
                out.append((x, 2 ** 575))
    return out


def test_rare_branch_of_the_reduction(harness, tmp_path):  # noqa: F811
    ops = operands()
    hits = {"carry": 0, "borrow": 0, "top": 0, "overflow": 0}
    for x, y in ops:
        for k, v in conditions(x * y).items():
            hits[k] += v
    assert all(v >= 4 for v in hits.values()), hits
    src, dst = tmp_path / "in", tmp_path / "out"
    with open(src, "w") as f:
        f.write(" ".join("0" for _ in range(21 * 18)) + "\n")
        f.write(f"{len(ops)}\n")
        for x, y in ops:
            f.write(" ".join("%x" % w for w in words(x)) + " " + " ".join("%x" % w for w in words(y)) + "\n")
    subprocess.run([harness, str(src), str(dst)], check=True)
    lines = open(dst).read().splitlines()
    per = len(lines) // len(ops)
    for i, (x, y) in enumerate(ops):
        assert from_words(lines[i * per].split()) == x * y % O.M, (i, hex(x), hex(y))
