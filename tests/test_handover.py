"""The hand-over of data between workgroups of a launch (csrc/handover.h), in
the intermediate code that the compiler makes of it for gfx950: the data's
stores, a release fence, the wait, a release fence, then the flag; and behind
the flag's load an acquire fence before the data's loads."""
import os
import re
import subprocess

import pytest

from paper_1906_08125_amd import build as B

KERNELS = """
#include "handover.h"
__global__ void put(fp::EmitSlot* p, fp::EmitSums v, int flag) { fp::sums_put(p, v, flag); }
__global__ void get(const fp::EmitSlot* p, fp::EmitSums* v, int flag) {
  fp::EmitSums s;
  if (fp::sums_get(p, s, flag)) *v = s;
}
"""


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    d = tmp_path_factory.mktemp("handover")
    src = d / "k.hip"
    src.write_text(KERNELS)
    out = d / "k.ll"
    subprocess.run([B.hipcc(), *B.FLAGS, f"-I{B.CSRC}", "--cuda-device-only", "-S", "-emit-llvm",
                    str(src), "-o", str(out)], check=True, capture_output=True, timeout=120)
    bodies = {}
    for name in ("put", "get"):
        m = re.search(r"define[^\n]*@_Z\d+%s\S*\([^\n]*\{\n(.*?)\n\}" % name, out.read_text(), re.S)
        ops = []
        for line in m.group(1).splitlines():
            if "atomic" in line and "store" in line:
                ops.append("store " + re.search(r"(i32|i64|double)", line).group(1))
            elif "atomic" in line and "load" in line:
                ops.append("load " + re.search(r"(i32|i64|double)", line).group(1))
            elif re.search(r"\bfence\b", line):
                ops.append("release" if "release" in line else "acquire" if "acquire" in line
                           else line.strip())
            elif "waitcnt" in line and "call" in line:
                ops.append("wait")
        bodies[name] = ops
    return bodies


def test_put(code):
    assert code["put"] == ["store i64"] * 5 + ["release", "wait", "release", "store i32"]


def test_get(code):
    """(the wait's loop may lie around the rest in the text)"""
    ops = code["get"]
    assert ops[0] == "load i32"
    assert [o for o in ops if o != "load i32"] == ["acquire"] + ["load i64"] * 5
