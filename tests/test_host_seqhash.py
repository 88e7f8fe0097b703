"""The signature under which a captured launch sequence is replayed: tables that
differ in any one field (the stored powers of the points among them) hash
apart, padding bytes do not count (native driver built with g++, no GPU)."""

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_every_table_field_is_part_of_the_signature(tmp_path):
    exe = str(tmp_path / "driver")
    subprocess.run(["g++", "-O1", "-std=c++17", "-o", exe, os.path.join(HERE, "native", "seqhash_driver.cpp")],
                   check=True)
    out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout
    sig = dict(line.split() for line in out.splitlines())
    assert sig.pop("padding") == sig["base"]
    assert {"pow_planes", "pow_nb", "qpow", "geo_D"} <= set(sig)
    assert len(set(sig.values())) == len(sig)
