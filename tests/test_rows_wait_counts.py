"""The multi-row decode kernel that takes X through LDS waits by count: vmcnt(9) leaves the nine youngest loads (one register
set of W and its gain) in flight, which is right only if at least nine ordinary loads follow every request that writes
LDS, in the prologue and around the loop.  Compiled to assembly here and checked; runs on the CPU."""
import importlib.util
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2604_15272_amd")


def loads_after_requests(asm_text):
    """{kernel symbol: (N of its hand-written vmcnt(N), N > 0, ordinary loads between the last LDS request before it and the
    wait, ordinary loads between the last LDS request after it and the branch that closes the loop)}"""
    out, name, in_asm, since, wait = {}, None, False, 0, None
    for line in asm_text.split("\n"):
        m = re.match(r"^(_ZN5prism18decode_rows_kernelI\S*Lb0ELi[24]ELb1E\S+):", line)
        if m:
            name, in_asm, since, wait = m.group(1), False, 0, None
        elif name is None:
            continue
        elif "s_endpgm" in line:
            name = None
        elif "#ASMSTART" in line:
            in_asm = True
        elif "#ASMEND" in line:
            in_asm = False
        elif re.search(r"\b(buffer|global)_load", line):
            since = 0 if re.search(r"\blds\b", line) else since + 1
        elif in_asm and wait is None and (w := re.search(r"s_waitcnt vmcnt\(([1-9]\d*)\)", line)):
            wait = (int(w.group(1)), since)
        elif wait is not None and name not in out and re.search(r"\bs_cbranch", line):
            out[name] = wait + (since,)
    return out


def test_checker_sees_a_request_that_is_too_young():
    k = "_ZN5prism18decode_rows_kernelIxLb0ELi2ELb1ELb0EEEv"
    req, ld = " buffer_load_dwordx4 v1, s[0:3], 0 offen lds", " buffer_load_dwordx4 v[2:5], v1, s[0:3], 0 offen"
    asm = [k + ":", req, ld, ld, ";;#ASMSTART", " s_waitcnt vmcnt(2)", ";;#ASMEND", ld, req, ld, " s_cbranch_scc1 .L", " s_endpgm"]
    assert loads_after_requests("\n".join(asm)) == {k: (2, 2, 1)}


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    spec = importlib.util.spec_from_file_location("_prism_build_for_test", os.path.join(PKG, "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    out = str(tmp_path_factory.mktemp("asm") / "rows.s")
    cmd = [b.hipcc_path()] + [f for f in b.HIPCC_FLAGS if f not in ("-shared", "-fPIC")] + [
        "-S", "--cuda-device-only", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
        os.path.join(PKG, "csrc", "decode_rows_kernel.hip"), "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    return open(out).read()


def test_the_counted_wait_covers_every_request_of_x(assembly):
    found = loads_after_requests(assembly)
    assert len(found) == 8, sorted(found)  # 32 and 64 rows, one and several row blocks, two storage formats
    for name, (n, before, around) in found.items():
        assert n == 9 and before >= n and around >= n, (name, n, before, around)


def test_the_kernel_does_not_ask_for_the_grid(assembly):
    """The grid's size is a load that the first addresses of W would wait for; the host passes what depends on it."""
    assert "decode_rows_kernel" in assembly and "hidden_block_count" not in assembly
