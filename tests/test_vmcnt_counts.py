"""The loader waves of the Gated DeltaNet state pass (gdn_state_roles_kernel) wait on
the vector-memory counter with a count derived from the kernel's own constants:
per chunk NL global_load_lds pieces, of which those of the next chunk may stay in
flight.  The count is only right if the compiler issues exactly those loads in
the loaders' chunk loop and no other vector-memory instruction (a register spill,
a split or merged load or an extra global load would shift it and the wait would
silently under-wait).  This test compiles the kernel source to gfx950 assembly
with the library's own flags and checks the loaders' loop of every instantiation
the library launches, on the CPU.
"""
import os
import re
import subprocess
import tempfile

import pytest

from paper_2606_01294_amd import build as B

C = 64


def expected(DK, NPR):
    """Loads of one loader wave and chunk: K, Tm, the V slice and the coefficients; a piece shared by
    several waves is one lane-masked load in each."""
    pieces = [C * DK * 2 // 1024, C * C * 2 // 1024, C * 16 * NPR * 2 // 1024]
    return sum((n + 3) // 4 for n in pieces) + 1


# the instantiations the library launches (template <DK, NPR, NG>)
INSTANCES = [(128, 1, 4), (128, 2, 4), (128, 4, 4), (128, 4, 2), (256, 1, 4), (256, 2, 4)]


@pytest.fixture(scope="module")
def roles_asm():
    src = os.path.join(B.CSRC, "ccq_gdn_roles.hip")
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "roles.s")
        cmd = [B._hipcc()] + B.COMMON + B.DEVICE + ["--cuda-device-only", "-S", src, "-o", out]
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            pytest.skip("hipcc unavailable for gfx950 here: " + res.stderr[-300:])
        return open(out).read()


@pytest.mark.parametrize("inst", INSTANCES, ids=lambda t: "dk%d-npr%d-ng%d" % t)
def test_state_pass_loop_issues_the_counted_vector_memory_ops(roles_asm, inst):
    sym = "_ZN3ccq22gdn_state_roles_kernelILi%dELi%dELi%dEEEvNS_7GdnArgsE" % inst
    assert ("\n" + sym + ":") in roles_asm, "instantiation %s not emitted" % sym
    body = roles_asm.split("\n" + sym + ":", 1)[1].split(".Lfunc_end", 1)[0].split("\n")
    assert not any(x.strip().startswith(("scratch_", "buffer_")) for x in body), "registers spilled"
    label = {m.group(1): i for i, x in enumerate(body) for m in [re.match(r"(\.LBB\d+_\d+):", x)] if m}
    loops = {}
    for i, x in enumerate(body):
        m = re.search(r"s_c?branch\w*\s+(\.LBB\d+_\d+)", x)
        if m and label[m.group(1)] <= i:
            loops[label[m.group(1)]] = max(i, loops.get(label[m.group(1)], 0))
    counts = []
    for h, e in loops.items():
        ins = [x.split(";")[0].split() for x in body[h:e + 1]]
        ins = [x[0] for x in ins if x and not x[0].startswith(".")]
        if not any("mfma" in x for x in ins):  # the loaders' loop
            vm = [x for x in ins if x.startswith(("global_", "buffer_", "scratch_", "flat_"))]
            counts.append((vm.count("global_load_lds_dwordx4"), len(vm)))
    n = expected(*inst[:2])
    assert (n, n) in counts, (n, counts)
