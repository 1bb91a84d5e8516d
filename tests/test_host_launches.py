"""CPU checks of what the library's host side launches: small programs linked
against libkk.so and a stand-in for the HIP runtime (host_runtime.hpp), which
records every kernel launch and runs none."""
import os
import subprocess

import pytest

from paper_1309_4349_amd import kk

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1309_4349_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _run(tmp_path, program):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    kk.load()  # builds the library if nothing is built
    src, exe = tmp_path / "p.cpp", tmp_path / "p"
    src.write_text('#include "host_runtime.hpp"\n#include "kk.h"\n' + program)
    lib = os.path.dirname(kk.LIB_PATH)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-O1", "-w", "-rdynamic",
                    *(f"-I{d}" for d in (os.path.join(ROOT, "tests"), os.path.join(ROOT, "include"), CSRC)),
                    str(src), "-o", str(exe), f"-L{lib}", "-l:" + os.path.basename(kk.LIB_PATH), f"-Wl,-rpath,{lib}",
                    "-Wl,--allow-shlib-undefined"], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.stdout + r.stderr)[-2000:]


# The lanes of a whole ring's phase waves stay, in every class, before the words where other waves store the draws, and
# the ring, two buffers of draws and 128 class orders fit the LDS next to what the kernel holds there besides (under 1 KiB).
RING = r"""
#include "kk_tri.hpp"
using namespace kk;
int main() {
  int rings = 0, most = 0;
  for (int L = 4; L <= 13568; L += 8)
    for (int H = 4; (size_t)L * H <= kTriResidentMaxBytes; H += 4) {
      const int B = (int)ring_segments(L, H);
      if (B == 0) continue;
      ++rings;
      const int W = L * H / (16 * B);
      REQUIRE(W * 16 * B == L * H && W <= kRingStride && 16 * W >= 2 * L);
      REQUIRE(ring_lds_bytes(L, H) + 1024 <= 160 * 1024);
      most = W > most ? W : most;
      const int lanes = (W + 63) / 64 * 64;
      REQUIRE(15 * kRingStride + lanes <= kRingWords && kRingWords % 2 == 0);
      REQUIRE(ring_lds_bytes(L, H) >= 4u * kRingWords + 12u * 16u * W * 4u + 128u * 8u);
    }
  REQUIRE(rings > 1000 && most == kRingMaxWords);
  return 0;
}
"""


def test_every_lane_of_a_whole_ring_stays_off_the_draws(tmp_path):
    _run(tmp_path, RING)


# Every tile that kk_set_tile accepts can be launched, for a single sweep and for two.
SET_TILE = r"""
int main() {
  for (unsigned L : {1024u, 1036u}) {
    kk_sim* h = nullptr;
    REQUIRE(kk_create_ex(&h, L, 0.5, 0.5, 1, L % 32 ? KK_LAYOUT_INT8 : KK_LAYOUT_BITPACKED, nullptr) == KK_OK);
    int accepted = 0;
    for (unsigned words = 1; words <= 32; ++words)
      for (unsigned rows = 2; rows <= 1200; rows += 2)
        for (unsigned units = 1; units <= 2; ++units) {
          if (kk_set_tile(h, words, rows, units) != KK_OK) continue;
          ++accepted;
          for (unsigned n = 1; n <= 2; ++n)
            if (kk_sweep(h, n) != KK_OK) {
              printf("tile %u x %u at %u units, %u sweeps: %s\n", words, rows, units, n, kk_last_error());
              return 1;
            }
        }
    REQUIRE(accepted > 2000);
    REQUIRE(kk_set_tile(h, 1, 996, 2) == KK_OK && kk_set_tile(h, 1, 998, 2) == KK_EINVAL);  // 1536 units, and 1539
    kk_destroy(h);
  }
  return 0;
}
"""


def test_every_accepted_tile_can_be_launched(tmp_path):
    _run(tmp_path, SET_TILE)


# Each pass of a cluster histogram has the workgroups to work on all tiles (64 x 64 sites) of a small lattice at once.
HIST = r"""
int main() {
  for (unsigned L : {64u, 256u, 400u, 640u}) {
    kk_sim* h = nullptr;
    REQUIRE(kk_create_ex(&h, L, 0.5, 0.5, 1, KK_LAYOUT_INT8, nullptr) == KK_OK);
    g_launches.clear();
    size_t n = 0;
    REQUIRE(kk_cluster_hist(h, 1, nullptr, 0, &n) == KK_OK);
    const unsigned tiles = ((L + 63) / 64) * ((L + 63) / 64);
    size_t seen = 0;
    for (const Launch& l : g_launches)
      for (const char* pass : {"ccl_tile", "ccl_sizes", "ccl_hist"})
        if (l.kernel.find(pass) != std::string::npos) {
          REQUIRE(l.blocks == tiles);
          ++seen;
        }
    REQUIRE(seen == 3);
    kk_destroy(h);
  }
  return 0;
}
"""


def test_histogram_passes_take_all_tiles_at_once(tmp_path):
    _run(tmp_path, HIST)


# Whole rings of a batch of fewer than 64 share one launch; a replica whose handle was given another tile since, and one
# that is no ring, run their own.
FEW_RINGS = r"""
int main() {
  std::vector<kk_tri_replica> reps;
  for (unsigned i = 0; i < 12; ++i) {
    const unsigned L = i % 3 == 0 ? 100u : 140u;
    reps.push_back(kk_tri_replica{L, L, KK_TRI_CLASSES, KK_START_RANDOM, 0.5, 0.5, i, 3 + i % 2});
  }
  reps.push_back(kk_tri_replica{101, 84, KK_TRI_MPKK, KK_START_RANDOM, 0.5, 0.5, 1, 3});
  kk_tri_batch* b = nullptr;
  REQUIRE(kk_tri_batch_create(&b, reps.data(), reps.size(), nullptr) == KK_OK);
  g_launches.clear();
  REQUIRE(kk_tri_batch_run(b) == KK_OK);
  REQUIRE(launched("ring_sweeps") == 1 && launched("mpkk") == 3);
  for (const Launch& l : g_launches) REQUIRE(l.kernel.find("ring_sweeps") == std::string::npos || l.blocks == 12);
  kk_sim* h = nullptr;
  REQUIRE(kk_tri_batch_sim(b, 1, &h) == KK_OK && kk_tri_set_tile(h, 16, 16) == KK_OK);
  g_launches.clear();
  REQUIRE(kk_tri_batch_run(b) == KK_OK);
  REQUIRE(launched("ring_sweeps") == 1 && launched("hex_sweep") == 4);
  for (const Launch& l : g_launches) REQUIRE(l.kernel.find("ring_sweeps") == std::string::npos || l.blocks == 11);
  uint64_t sweeps = 0, attempts = 0;
  REQUIRE(kk_stats(h, &sweeps, &attempts, nullptr) == KK_OK && sweeps == 8 && attempts == 8 * 140 * 140);
  kk_tri_batch_destroy(b);
  return 0;
}
"""


def test_few_whole_rings_share_a_launch(tmp_path):
    _run(tmp_path, FEW_RINGS)


# kk_autotune times the tile the handle has and the untuned default, also once another tile is the default of the process,
# and ranks by launches of two sweeps whatever the number of trial sweeps.
AUTOTUNE = r"""
#include "kk_kernels.hpp"
static unsigned fast[2];  // words and rows of the tile that is quicker than all others
static double cost(const Launch& l) {
  if (l.kernel.find("halo_kernel") == std::string::npos && l.kernel.find("sweep_kernel") == std::string::npos &&
      l.kernel.find("pipe_kernel") == std::string::npos)
    return 0.0;
  const kk::SweepParams& p = *static_cast<const kk::SweepParams*>(l.args[0]);
  return (p.nsweeps == 1 ? 50.0 : p.nsweeps) * ((unsigned)p.tww == fast[0] && (unsigned)p.th == fast[1] ? 0.5 : 1.0);
}
int main() {
  g_cost = cost;
  for (unsigned L : {300u, 400u, 1036u, 2048u}) {
    const unsigned layout = L % 32 ? KK_LAYOUT_INT8 : KK_LAYOUT_BITPACKED;
    kk_sim *h = nullptr, *g = nullptr, *f = nullptr;
    uint32_t words, rows, units;
    double us = 0.0;
    REQUIRE(kk_create_ex(&h, L, 0.5, 0.5, 1, layout, nullptr) == KK_OK);
    uint32_t untuned[3];
    REQUIRE(kk_get_tile(h, &untuned[0], &untuned[1], &untuned[2]) == KK_OK);
    fast[0] = 8, fast[1] = 96;  // one of the list
    REQUIRE(kk_autotune(h, 1, &words, &rows, &units, &us) == KK_OK && words == 8 && rows == 96 && us == 500.0);
    fast[0] = untuned[0], fast[1] = untuned[1];  // only the rule's; the process's default is the list's now
    REQUIRE(kk_create_ex(&g, L, 0.5, 0.5, 1, layout, nullptr) == KK_OK);
    REQUIRE(kk_autotune(g, 5, &words, &rows, &units, &us) == KK_OK);
    REQUIRE(words == untuned[0] && rows == untuned[1] && units == untuned[2] && us == 500.0);
    fast[0] = 8, fast[1] = 100;  // only the handle's
    REQUIRE(kk_create_ex(&f, L, 0.5, 0.5, 1, layout, nullptr) == KK_OK && kk_set_tile(f, 8, 100, 1) == KK_OK);
    REQUIRE(kk_autotune(f, 4, &words, &rows, &units, nullptr) == KK_OK && words == 8 && rows == 100 && units == 1);
    for (kk_sim* s : {h, g, f}) kk_destroy(s);
  }
  return 0;
}
"""


def test_autotune_times_the_tile_it_replaces(tmp_path):
    _run(tmp_path, AUTOTUNE)


# Sweeps in pairs where that takes no more rounds of workgroups, as for every default tile; one per launch on tiles that
# fill the device several times over, or would with twice the threads.
PAIRS = r"""
int main() {
  for (unsigned L = 4; L <= 8192; L += L < 512 ? 4 : (L < 4096 ? 92 : 512))
    for (unsigned layout : {KK_LAYOUT_INT8, KK_LAYOUT_BITPACKED}) {
      kk_sim* h = nullptr;
      if (layout == KK_LAYOUT_BITPACKED && L % 32) continue;
      REQUIRE(kk_create_ex(&h, L, 0.5, 0.5, 1, layout, nullptr) == KK_OK);
      g_launches.clear();
      REQUIRE(kk_sweep(h, 9) == KK_OK);
      if (g_launches.size() != (launched("halo_kernel") ? 5 : 1)) {
        printf("%u: %zu launches\n", L, g_launches.size());
        return 1;
      }
      kk_destroy(h);
    }
  kk_sim* h = nullptr;
  REQUIRE(kk_create_ex(&h, 4096, 0.5, 0.5, 1, KK_LAYOUT_BITPACKED, nullptr) == KK_OK);
  const unsigned tiles[][4] = {{16, 128, 2, 5}, {8, 256, 2, 5}, {8, 64, 1, 9}, {8, 16, 1, 9}, {2, 32, 1, 9}, {16, 40, 1, 9}};
  for (const auto& t : tiles) {
    REQUIRE(kk_set_tile(h, t[0], t[1], t[2]) == KK_OK);
    g_launches.clear();
    uint64_t launches = 0;
    REQUIRE(kk_sweep_timed(h, 9, nullptr, &launches) == KK_OK);
    if (launches != t[3] || launched("halo_kernel") != t[3]) {
      printf("%u x %u: %zu launches\n", t[0], t[1], (size_t)launches);
      return 1;
    }
  }
  kk_destroy(h);
  return 0;
}
"""


def test_sweeps_in_pairs_where_they_pay(tmp_path):
    _run(tmp_path, PAIRS)
