"""Loads that write LDS are inline assembly, which the compiler adds no wait states to: in the assembly of the kernels built on
them, no vector instruction writes a scalar register within five wait states of such a load that reads it, and nothing but the
loads uses m0."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1807_02037_amd", "csrc")
WAIT_STATES = 5


def sgprs(operand):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.fullmatch(r"s(\d+)", operand)
    return {int(m[1])} if m else set()


def scan(text):
    """(number of LDS-writing loads, offending instructions)"""
    loads, bad, before = 0, [], []        # before: (wait states, scalar registers written by a vector instruction)
    for line in text.splitlines():
        line = line.split(";")[0].strip()
        if not line or line.startswith(".") or line.endswith(":"):
            continue
        op, *args = [t.strip(",") for t in line.split()]
        if op.startswith("buffer_load") and "lds" in args:
            loads += 1
            reads, distance = sgprs(args[1]) | sgprs(args[2]), 0
            for states, written in reversed(before):
                if distance >= WAIT_STATES:
                    break
                if written & reads:
                    bad.append(line)
                distance += states
        elif "m0" in args and op != "s_mov_b32":
            bad.append(line)
        written = set()
        if op.startswith("v_"):           # results come first; carries and the flags of a scaled division second
            written = sgprs(args[0]) | (sgprs(args[1]) if "_co_" in op or "div_scale" in op else set())
        before = (before + [(int(args[0], 0) + 1 if op == "s_nop" else 1, written)])[-WAIT_STATES - 1:]
    return loads, bad


def test_the_scan_finds_a_missing_wait_state():
    head, load = "v_readfirstlane_b32 s7, v1\n", "s_mov_b32 m0, s2\ns_nop 0\nbuffer_load_dwordx4 v3, s[4:7], s9 offen lds\n"
    assert scan(head + load) == (1, ["buffer_load_dwordx4 v3, s[4:7], s9 offen lds"])
    assert scan(head + "s_nop 2\n" + load) == (1, [])
    assert scan("v_readlane_b32 s9, v1, 3\n" + load)[1] and not scan("v_readlane_b32 s8, v1, 3\n" + load)[1]


def test_wait_states_of_the_built_kernels(tmp_path):
    def assembly(name):
        out = str(tmp_path / (name + ".s"))
        subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-Xclang", "-target-feature",
                        "-Xclang", "-packed-fp32-ops", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "--cuda-device-only", "-S",
                        os.path.join(CSRC, name), "-o", out], check=True, capture_output=True)
        return open(out).read()

    names = [f for f in sorted(os.listdir(CSRC)) if f.endswith(".hip") and "conv_dma.hpp" in open(os.path.join(CSRC, f)).read()]
    assert len(names) >= 4
    with ThreadPoolExecutor(4) as pool:
        for name, text in zip(names, pool.map(assembly, names)):
            loads, bad = scan(text)
            assert loads > 0 and not bad, (name, bad[:3])
