"""The passes over rows that are not 16-byte aligned take one element per lane and
row, and hide the latency by having the loads of several rows in flight.  A 16-bit
element that is converted under a branch is waited for there, so that one row is in
flight at a time: the compiled kernels are read for it."""
import os
import re
import subprocess

import pytest

from paper_2608_20818_amd import build as b


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    d = tmp_path_factory.mktemp("asm")

    def text(source):
        out = d / (source + ".s")
        if not out.exists():
            r = subprocess.run([b.hipcc(), *b.FLAGS, "--cuda-device-only", "-S", os.path.join(b.CSRC, source), "-o", str(out)],
                               capture_output=True, text=True, timeout=300)
            assert r.returncode == 0, r.stderr[-2000:]
        return out.read_text()
    return text


def in_flight(asm, kernel, load):
    """The most vector loads in flight at once in a kernel, from its first `load` to
    its last (a count of s_waitcnt vmcnt and of what it leaves in flight)."""
    i = asm.index("\n" + next(m for m in re.findall(r"\n(_Z\w+):", asm) if re.search(kernel, m)) + ":")
    lines = [s.strip() for s in asm[i:asm.index(".Lfunc_end", i)].splitlines()]
    at = [k for k, s in enumerate(lines) if s.startswith(load)]
    assert at
    now = most = 0
    for s in lines[at[0]:at[-1] + 1]:
        if s.startswith("global_load"):
            now += 1
            most = max(most, now)
        elif (m := re.match(r"s_waitcnt .*vmcnt\((\d+)\)", s)):
            now = min(now, int(m[1]))
    return most


def test_the_count():
    good = "\n_Zk:\n" + "global_load_ushort v1\n" * 8 + "s_waitcnt vmcnt(0)\n.Lfunc_end0:"
    bad = "\n_Zk:\n" + "global_load_ushort v1\nglobal_load_dword v2\ns_waitcnt vmcnt(1)\n" * 8 + ".Lfunc_end0:"
    assert in_flight(good, "_Zk", "global_load_ushort") == 8 and in_flight(bad, "_Zk", "global_load_ushort") == 3


# odd widths: <gradient, aligned> of the statistics; <weight, gradient, Nesterov,
# aligned, own norms, rows> of the apply
@pytest.mark.parametrize("kernel", ["rw_tall_stats_kernelILNS_5DTypeE1ELb0E", "rw_tall_apply_kernelILNS_5DTypeE1ELS1_1ELb0ELb0ELb0ELi16E",
                                    "rw_tall_apply_kernelILNS_5DTypeE1ELS1_0ELb0ELb0ELb0ELi16E",
                                    "rw_tall_apply_kernelILNS_5DTypeE0ELS1_1ELb1ELb0ELb0ELi16E"])
def test_rows_of_odd_tall_matrices(assembly, kernel):
    assert in_flight(assembly("rowwise.hip"), kernel, "global_load_ushort") >= 24


# <gradient, hi + lo>
@pytest.mark.parametrize("kernel", ["ns_prologue_kernelILNS_5DTypeE1ELb0E", "ns_prologue_kernelILNS_5DTypeE1ELb1E"])
def test_rows_of_the_refresh_prologue(assembly, kernel):
    assert in_flight(assembly("ns5.hip"), kernel, "global_load_ushort") >= 12


# widths that are multiples of 4: fp32 with Nesterov, norms from the finalize
def test_rows_of_aligned_tall_matrices_with_nesterov(assembly):
    kernel = "rw_tall_apply_kernelILNS_5DTypeE0ELS1_0ELb1ELb1ELb0ELi16E"
    assert in_flight(assembly("rowwise.hip"), kernel, "global_load_dwordx4") >= 20


# ragged rows, a block of 256 threads with four chunks of 8 elements per thread
@pytest.mark.parametrize("types", ["1ELS1_1", "1ELS1_0", "0ELS1_1", "0ELS1_0"])
def test_pieces_of_ragged_rows(assembly, types):
    kernel = f"rw_wide_kernelILi256ELi256ELi4ELNS_5DTypeE{types}ELb0E"
    assert in_flight(assembly("rowwise.hip"), kernel, "global_load_dwordx4") >= 20
