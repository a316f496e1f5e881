"""The hand-over between workgroups in the clique search's first kernel, read
from the gfx950 assembly built from its source: every wave stores its roots'
counts, the workgroup meets, one thread releases them to the other XCDs and takes
a ticket, and the last workgroup to take one reads them all.  The barrier does not
wait for stores and the release waits for its own wave's only, so each wave has
to wait for its stores before that barrier."""
import os
import re
import subprocess

import pytest

from paper_2212_00574_amd import build

SOURCE = os.path.join(build.CSRC, "kz_clique.hip")


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("asm") / "kz_clique.s")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [build.HIPCC, *flags, "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "-S",
           "--cuda-device-only", "-o", out, SOURCE]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    with open(out) as f:
        return f.read()


def test_stores_land_before_the_release(asm):
    body = re.search(r"^_ZN\S*k_clique_alive\S*:\s.*?^\.Lfunc_end", asm, re.S | re.M).group(0)
    ops = [line.split(";")[0].strip() for line in body.split("\n")]
    ops = [op for op in ops if op]
    release = next(i for i, op in enumerate(ops) if op.startswith("buffer_wbl2"))
    assert any("global_atomic_add" in op for op in ops[release:]), "the ticket follows the release"
    barrier = max(i for i, op in enumerate(ops[:release]) if op.startswith("s_barrier"))
    store = max(i for i, op in enumerate(ops[:barrier]) if op.startswith("global_store"))
    # after the join behind the last store, on the path of every wave
    join = max(i for i, op in enumerate(ops[:barrier]) if op.endswith(":"))
    assert store < join
    waits = [op for op in ops[join:barrier] if op.startswith("s_waitcnt") and "vmcnt(0)" in op]
    assert waits, ops[join:barrier + 1]
