"""Exact division by one divisor for many dividends and the in-place difference
(host big integers of the gcd) against Python's integers, through a native
driver built with g++ (no GPU)."""

import os
import random
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def hx(v):
    return ("-" if v < 0 else "") + format(abs(v), "x")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("exact") / "driver")
    subprocess.run(["g++", "-O2", "-std=c++17", "-o", exe, os.path.join(HERE, "native", "exact_div_driver.cpp"),
                    os.path.join(os.path.dirname(HERE), "paper_1201_1548_amd", "csrc", "bigint.cpp")], check=True)
    return exe


@pytest.mark.parametrize("dbits", [1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 640])
def test_quotients_and_differences(driver, dbits):
    rng = random.Random(dbits)
    rows, want = [], []
    for k in range(120):
        d = (rng.getrandbits(dbits) | 1 << (dbits - 1)) << rng.choice([0, 0, 1, 31, 32, 63, 64, 65, 130])
        d *= rng.choice([1, -1])
        q = rng.choice([0, 1, (1 << rng.randint(1, 300)) - 1, rng.getrandbits(rng.randint(1, 700))]) * rng.choice([1, -1])
        a = d * q
        b = a + rng.choice([0, 1, -1, d // 2, 1 << rng.randint(0, abs(a).bit_length() + 2), rng.getrandbits(700)])
        c = rng.choice([a, -a, 0, b, rng.getrandbits(rng.randint(1, 900)), -rng.getrandbits(500)])
        rows.append("%s %s %s %s" % (hx(d), hx(a), hx(b), hx(c)))
        want.append((q, b // d if b % d == 0 else None, a - c))
    out = subprocess.run([driver], input="\n".join(rows) + "\n", capture_output=True, text=True, check=True).stdout
    for line, w in zip(out.split("\n"), want):
        assert [None if x == "inexact" else int(x, 16) for x in line.split(",")] == list(w)
