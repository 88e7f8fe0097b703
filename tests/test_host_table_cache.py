"""What the device tables' cache hands out, builds and lets go (native driver
built with g++, no GPU): sizes that grow in turn leave one table instead of a
row of outgrown ones, the limits hold, the least recently used go first, and a
table in use outlives its place in the cache."""

import os
import random
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
MIB = 1 << 20


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("tables") / "driver")
    subprocess.run(["g++", "-O1", "-std=c++17", "-o", exe, os.path.join(HERE, "native", "table_cache_driver.cpp")],
                   check=True)
    return exe


def run(driver, one, every, commands):
    out = subprocess.run([driver, str(one), str(every)], input="\n".join(commands) + "\n", capture_output=True,
                         text=True, check=True).stdout
    keys = ("a", "b", "built", "bytes", "alive", "went")
    return [dict(zip(keys, line.split())) for line in out.splitlines()]


def test_growing_sizes_never_run_out(driver):
    # the node tables' limits: at 4352 indices each step takes 182 MiB and more
    steps = [(4352, p) for p in range(32, 1025, 32)] + [(a, 704) for a in range(4608, 8193, 256)]
    got = run(driver, 512 * MIB, 1024 * MIB, ["get 0 %d %d 1" % s for s in steps])
    for s, g in zip(steps, got):
        assert g["a"] != "none" and int(g["a"]) >= s[0] and int(g["b"]) >= s[1]
        assert int(g["bytes"]) <= 1024 * MIB and int(g["alive"]) <= 1024 * MIB


def test_one_table_for_sizes_that_differ_in_turn(driver):
    got = run(driver, 512 * MIB, 1024 * MIB, ["get 0 256 704 1", "get 0 4352 32 1", "get 0 256 700 1", "get 0 4000 32 1"])
    assert [(g["a"], g["b"]) for g in got] == [("256", "704")] + [("4352", "704")] * 3
    assert got[-1]["built"] == "2" and int(got[-1]["bytes"]) == 76 * 4352 * 704


def test_least_recently_used_go_first(driver):
    size = 76 * 1000
    got = run(driver, size, 3 * size, ["get 1 1000 0 0", "get 2 1000 0 0", "get 3 1000 0 0", "look 1 1000 0",
                                       "get 4 1000 0 0", "look 1 1000 0", "look 2 1000 0", "look 3 1000 0"])
    assert [g["a"] for g in got[5:]] == ["1000", "none", "1000"]
    assert got[4]["went"] == "1" and int(got[-1]["bytes"]) == 3 * size


def test_a_table_in_use_outlives_its_place(driver):
    got = run(driver, MIB, MIB, ["get 0 10 10 1", "hold", "get 0 20 20 1", "drop"])
    assert int(got[2]["bytes"]) == 76 * 400 and got[2]["went"] == "1"
    got = run(driver, MIB, MIB, ["get 0 10 10 1", "hold", "clear", "get 0 20 20 1", "drop", "clear"])
    assert int(got[2]["bytes"]) == 0 and int(got[2]["alive"]) == 7600
    assert int(got[4]["alive"]) == 76 * 400 and int(got[5]["alive"]) == 0


def test_too_large_and_failed_builds_leave_the_rest(driver):
    got = run(driver, 76 * 100, 76 * 150, ["get 0 10 10 1", "get 0 11 10 1", "fail 1", "get 1 5 5 1", "look 0 10 10"])
    assert [g["a"] for g in got] == ["10", "none", "-", "none", "10"]


@pytest.mark.parametrize("seed", range(4))
def test_random_requests_keep_the_limits(driver, seed):
    rng = random.Random(seed)
    one, every = 76 * 4000, 76 * 10000
    req = [(rng.randint(0, 2), rng.randint(1, 120), rng.randint(1, 120), rng.randint(0, 1)) for _ in range(400)]
    for (tag, a, b, join), g in zip(req, run(driver, one, every, ["get %d %d %d %d" % r for r in req])):
        assert (g["a"] == "none") == (76 * a * b > one)
        if g["a"] != "none":
            assert int(g["a"]) >= a and int(g["b"]) >= b
        assert int(g["bytes"]) <= every and int(g["alive"]) <= every + one
