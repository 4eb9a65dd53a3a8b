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


def test_workspace_bound_holds_and_stays_small(tmp_path):
    """A workspace sized for a batch, k and capacity serves every smaller batch, k and row count, and
    group maxima never take more than 24 MiB of it for up to 64 queries (with the coarse ones less than the
    32 MiB of the fixed array) nor 256 MiB for more, however long the index."""
    _run(tmp_path, r"""
  std::mt19937_64 g(7);
  auto log_int = [&](double lo, double hi) {
    return (long long)std::exp(std::uniform_real_distribution<double>(std::log(lo), std::log(hi))(g));
  };
  for (int i = 0; i < 300000; ++i) {
    const int dtype = (int)(g() % 3);
    const int d = dtype == kDtypeF32 ? 4 * (int)log_int(1, 2048) : 128 * (int)log_int(1, 64);
    const long long cap = std::min<long long>(log_int(1, 2147483646), 288000000000ll / (d * (dtype == kDtypeF32 ? 4 : 2)));
    const long long rows = g() % 4 ? std::min(cap, log_int(1, (double)cap + 1)) : cap;
    const int nq_ws = (int)log_int(1, 4096), nq = g() % 2 ? nq_ws : (int)log_int(1, nq_ws + 1);
    const int k_ws = (int)log_int(1, 128), k = g() % 2 ? k_ws : (int)log_int(1, k_ws + 1);
    const size_t bound = dense_workspace_bound(dtype, d, cap, nq_ws, k_ws, kCus);
    // as the host runtime splits a batch
    auto need = [&](int n) { return dense_workspace_bytes(plan_dense(dtype, d, rows, n, k, kCus), dtype, d, n, rows, k); };
    int parts = 1, part = nq;
    for (; std::max(need(part), need(nq - (nq - 1) / part * part)) > bound; part = (nq + parts - 1) / parts) {
      CHECK(part > 64, "dtype %d d %d cap %lld rows %lld nq %d/%d k %d/%d: %zu > %zu", dtype, d, cap, rows, nq, nq_ws, k, k_ws,
            need(part), bound)
      parts += std::max(1, parts / 4);
    }
    CHECK(parts <= 4, "%d parts: dtype %d d %d rows %lld nq %d k %d", parts, dtype, d, rows, nq, k)
    if (nq <= 64 && k <= 16) CHECK(need(nq) <= (size_t)OPRAG_SCRATCH, "%zu bytes: dtype %d d %d rows %lld nq %d k %d", need(nq), dtype, d, rows, nq, k)
    if (k_ws <= 16) CHECK(bound <= (nq_ws <= 64 ? 27u : 290u) << 20, "%zu bytes: d %d cap %lld nq %d k %d", bound, d, cap, nq_ws, k_ws)
  }
""".replace("OPRAG_SCRATCH", "(32u << 20)"))


def test_levels_are_spread_over_the_index(tmp_path):
    """The threshold levels' tiles: each level's pitch a multiple of the next one's, the last level's
    tiles the whole index, and the first level's rows spread over the index and within it."""
    _run(tmp_path, r"""
  for (int dtype : {kDtypeF32, kDtypeBF16})
    for (int d : {128, 1024, 8192})
      for (long long rows : {32769ll, 99999ll, 393217ll, 8450000ll, 500000000ll})
        for (int nq : {1, 64, 65, 1000, 4096})
          for (int k : {10, 17, 128}) {
            const DensePlan p = plan_dense(dtype, d, rows, nq, k, kCus);
            if (p.kind != DensePlan::kFilter) continue;
            CHECK(p.n_levels >= 2 && (p.level_pitch[p.n_levels - 1] == 128 || p.level_pitch[p.n_levels - 1] == 256), "rows %lld", rows)
            for (int l = 2; l < p.n_levels; ++l)
              CHECK(p.level_pitch[l - 1] == (k <= 16 ? 8 : 4) * p.level_pitch[l], "rows %lld level %d", rows, l)
            CHECK(p.level_rows[0] >= 3840 && p.level_rows[0] <= 32000, "rows %lld: %lld", rows, p.level_rows[0])
            // tiles of 128 or 256 rows: the last one's last row, and how much of the index is spanned
            int found = 0;
            for (int bm : {128, 256}) {
              const long long tiles = p.level_rows[0] / bm, last = (tiles - 1) * p.level_pitch[0] + (bm - 1) * (long long)p.row_pitch0;
              if (p.level_pitch[0] != rows / tiles) continue;  // tiles of the other length
              ++found;
              CHECK(p.row_pitch0 >= 1 && last < rows, "rows %lld: the first level ends at %lld", rows, last)
              CHECK((long long)bm * p.row_pitch0 * d * (dtype == kDtypeF32 ? 4 : 2) <= 1ll << 30, "rows %lld", rows)
            }
            CHECK(found > 0, "rows %lld: pitch %lld", rows, p.level_pitch[0])
          }
""")
