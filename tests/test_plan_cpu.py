"""The dense search's planner on the CPU: a small host program over the library's own planning
functions checks the limits that its kernels rely on."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2608_08340_amd")
ROCM = "/opt/rocm"

pytestmark = pytest.mark.skipif(not shutil.which("g++") or not os.path.isdir(ROCM), reason="g++ or ROCm not available")

HEAD = r"""
#include "oprag_internal.h"
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>
using namespace oprag;
constexpr int kCus = 256;
#define CHECK(c, ...) if (!(c)) { printf("failed: " #c "  " __VA_ARGS__); printf("\n"); return 1; }
int main() {
"""


def _run(tmp_path, body: str) -> None:
    import paper_2608_08340_amd as P

    P.library()  # built if it was not
    src, exe = str(tmp_path / "t.cpp"), str(tmp_path / "t")
    with open(src, "w") as f:
        f.write(HEAD + body + "\n  return 0;\n}\n")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", f"-I{PKG}/csrc", src,
                        "-o", exe, os.path.join(PKG, "liboprag.so"), f"-Wl,-rpath,{PKG}", f"-L{ROCM}/lib", "-lamdhip64",
                        f"-Wl,-rpath,{ROCM}/lib"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]


def test_chunk_rows_fit_a_queued_hit(tmp_path):
    """A queued hit keeps its row offset in the chunk in 24 bits: rows of few bytes (fp32, d = 4 to
    12) must not fill a chunk up to the byte limit alone."""
    _run(tmp_path, r"""
  for (int d : {4, 8, 12, 16, 128})
    for (long long rows : {1000ll, 100000000ll, 268000000ll, 2147483646ll})
      for (int nq : {1, 65, 2049, 4096}) {
        const DensePlan p = plan_dense_dump(kDtypeF32, d, rows, nq, kCus);
        // chunks differ by one tile of at most 256 rows
        CHECK((rows + p.n_chunks - 1) / p.n_chunks <= (1 << 24), "d %d rows %lld nq %d: %d chunks", d, rows, nq, p.n_chunks)
      }
""")
