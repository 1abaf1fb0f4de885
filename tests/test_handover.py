"""The hand-over of data between workgroups of a launch (csrc/handover.h).  In
the intermediate code that the compiler makes of it for gfx950: the data's
stores, a release fence, the wait, a release fence, then the flag; and behind
the flag's load an acquire fence before the data's loads.  On the host, in a
build of its own: what a step injects by its sums, none when a trip was lost."""
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
  fp::sums_get(p, s, flag);
  *v = s;
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
    assert code["put"] == ["store i64"] * 6 + ["release", "wait", "release", "store i32"]


def test_get(code):
    """(the wait's loop may lie around the rest in the text)"""
    ops = code["get"]
    assert ops[0] == "load i32"
    assert [o for o in ops if o != "load i32"] == ["acquire"] + ["load i64"] * 6


END = """
#include <cstdio>
#include "handover.h"
int main() {
  const long long cases[][4] = {  // offset, lost, base, capacity
      {5, 0, 10, 100}, {5, 0, 97, 100}, {5, 0, 100, 100}, {0, 0, 0, 100}, {5, 0, 101, 100},
      {5, 1, 10, 100}, {5, 1, 99, 100}, {0, 1, 0, 100}};
  for (const auto& c : cases) {
    fp::EmitSums s{};
    s.offset = c[0];
    s.lost = c[1];
    const fp::EmitEnd e = fp::emit_end(s, c[2], c[3]);
    std::printf("%lld %lld %d\\n", e.total, e.fit, (int)e.status);
  }
}
"""


def test_what_is_injected(tmp_path):
    from paper_1906_08125_amd import pic
    src, exe = tmp_path / "end.hip", tmp_path / "end"
    src.write_text(END)
    subprocess.run([B.hipcc(), "-O1", "-std=c++17", f"--offload-arch={B.ARCH}", f"-I{B.CSRC}",
                    str(src), "-o", str(exe)], check=True, capture_output=True, timeout=120)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60)
    got = [tuple(map(int, line.split())) for line in out.stdout.splitlines()]
    ok, full, dev = pic.PIC_OK, pic.PIC_E_CAPACITY, pic.PIC_E_DEVICE
    assert got == [(5, 5, ok), (5, 3, full), (5, 0, full), (0, 0, ok), (5, 0, full),
                   (0, 0, dev), (0, 0, dev), (0, 0, dev)]
