"""The library's host-side choices (csrc/attn_plan.cpp): key ranges, item size and plan of packed and
chunk calls, accesses of device copies; compiled with g++ under ASan and UBSan with a driver that walks
random and extreme shapes."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_19271_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

DRIVER = r"""
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include "attn_launch.h"
using namespace tsattn;
static int bad = 0;
#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); ++bad; } } while (0)
int main() {
  uint64_t r = 12345;
  auto rnd = [&](int64_t n) { r = r * 6364136223846793005ull + 1442695040888963407ull; return (int64_t)(r >> 33) % n; };
  const int32_t big[] = {0, 1, 63, 64, 65, 255, 256, 257, 32760, 8388607};
  for (int i = 0; i < 200000; ++i) {
    struct { int32_t nseq, total_q, max_k, H, d; } c;
    c.nseq = 1 + (int32_t)(rnd(3) ? rnd(70) : rnd(100000));
    c.total_q = rnd(4) ? (int32_t)rnd(200000) : big[rnd(10)];
    c.max_k = rnd(4) ? (int32_t)rnd(100000) : big[rnd(10)];
    c.H = 1 + (int32_t)rnd(128);
    c.d = rnd(2) ? 64 : 128;
    const int32_t n = auto_splits(c.total_q, c.max_k, c.H, c.d, 256);
    const int64_t tiles = ((int64_t)c.max_k + key_tile(c.d) - 1) / key_tile(c.d);
    CHECK(n >= 1 && n <= 16 && (n == 1 || tiles / n >= 4));
    // the fewest rounds of key tiles, then the fewest ranges; grids that fill the GPU stay whole
    const int64_t q_items = (int64_t)c.H * ((c.total_q + 255ll) / 256);
    auto rounds = [&](int64_t m) { return (q_items * m + 255) / 256 * ((tiles + m - 1) / m); };
    if (q_items == 0 || q_items >= 256 || tiles < 8) CHECK(n == 1);
    else
      for (int32_t m = 1; m <= 16 && tiles / m >= 4; ++m) CHECK(m < n ? rounds(m) > rounds(n) : rounds(m) >= rounds(n));
    // the launch grid holds every item, whatever the lengths: equal ones, and all but one empty
    const int32_t tile = rnd(2) ? kSmallTile : kQueryTile;
    const int64_t per = (int64_t)c.H * n, t = tile;
    const int64_t even = c.total_q / c.nseq, more = c.total_q % c.nseq;
    const int64_t items = per * ((c.nseq - more) * ((even + t - 1) / t) + more * ((even + t) / t));
    CHECK(packed_items(c.total_q, c.nseq, c.H, n, tile) >= items);
    CHECK(packed_items(c.total_q, c.nseq, c.H, n, tile) >= per * ((c.total_q + t - 1) / t));
    CHECK(packed_items(c.total_q, c.nseq, c.H, n, kQueryTile) <= packed_grid_bound(c.total_q, c.nseq, c.H, n));
  }
  // a call that fills the GPU for many rounds is not split; one 24-item call over 512 tiles is
  CHECK(auto_splits(32760, 32760, 40, 128, 256) == 1);
  CHECK(auto_splits(500, 32760, 12, 128, 256) > 4);
  // equal sessions, single chunks, and uneven ones: total queries, longest cache, heads, d -> ranges
  const int32_t known[][5] = {{1024, 1536, 4, 64, 3}, {768, 2816, 12, 128, 7}, {3072, 4608, 12, 128, 12}, {1024, 5120, 16, 128, 4},
                              {1280, 5120, 12, 64, 4}, {512, 5120, 16, 128, 8}, {1560, 32760, 12, 128, 3}, {768, 2304, 4, 64, 4}};
  for (const auto& w : known) CHECK(auto_splits(w[0], w[1], w[2], w[3], 256) == w[4]);
  CHECK(!small_items(257, 4096, 256) && small_items(256, 4096, 256) && !small_items(1, 64, 256));
  // the waves' own plan: at most 96 segments x rounds of items, one segment always
  CHECK(wave_plan(1, 1 << 23, 256) && wave_plan(64, 1, 256) && wave_plan(64, 384, 256) && !wave_plan(64, 385, 256));
  CHECK(!wave_plan(65, 1, 256) && !wave_plan(64, 2560, 256) && !wave_plan(32, 1280, 256) && !wave_plan(48, 1920, 256));
  CHECK(wave_plan(8, 1280, 256) && wave_plan(2, 12288, 256) && !wave_plan(2, 12289, 256) && !wave_plan(64, 1 << 23, 256));
  // device copies: plain accesses as long as the Infinity Cache holds what is read and written
  CHECK(!bypass_caches(40ll << 20) && !bypass_caches(128ll << 20) && bypass_caches((128ll << 20) + 1));
  printf("failures %d\n", bad);
  return bad != 0;
}
"""


def test_split_choice(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "driver.cpp", str(tmp_path / "driver")
    src.write_text(DRIVER)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=all", "-Wall", "-Wextra", "-Werror", "-D__HIP_PLATFORM_AMD__",
                        "-I" + os.path.join(ROCM, "include"), "-I" + CSRC, str(src),
                        os.path.join(CSRC, "attn_plan.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "failures 0" in r.stdout, r.stdout + r.stderr
