"""Checked at compile time: the LDS layout that the selection kernels and their launch sizes share, for every capacity, where
the kernel with the caller's top-k list reads that list, and which steps with that list gather its fixed rows beside their second phase."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_05688_amd", "csrc")

CHECK = r"""
#include "vatt_select.h"
using namespace vatt;
// every place follows the one before it with room for what it holds, at 16-byte boundaries where bitmaps are cleared
template <int NT, bool TWO>
constexpr bool in_order(int n) {
  const HeadLds l = head_lds<NT, TWO>(n);
  const uint32_t words = (uint32_t)bitmap_words(n);
  const uint32_t maps[] = {l.bm_f, l.taken0, l.taken1, l.scratch0, l.scratch1, l.wpre, l.mail0};
  if (words * 32 < (uint32_t)n || l.cand * 4 < sizeof(typename HeadOps<NT>::HeadSmem) || l.cand % 4 || l.bm_f % 4 || words % 4) return false;
  if (l.qual - l.cand < 2 * kCandCap || l.bm_f - l.qual < kCandCap) return false;
  for (int i = 0; i < 6; ++i)
    if (maps[i + 1] - maps[i] != (i == 3 && !TWO ? 0 : words)) return false;
  return l.mail1 - l.mail0 == (TWO ? kMailSlots : 0) && l.lists - l.mail1 == kMailSlots;
}
constexpr bool all() {
  for (int n = 1; n <= kCapacityMax; n += n < 4100 ? 1 : 509)
    if (!in_order<512, false>(n) || !in_order<512, true>(n) || !in_order<1024, false>(n) ||
        // a capacity that either form of the scored path's kernel takes is one the kernel with the caller's list takes
        head_lds<512, false>(n).lists > head_lds<1024, false>(n).lists || head_lds<512, false>(n).lists > head_lds<512, true>(n).lists)
      return false;
  return true;
}
static_assert(all(), "layout");
static_assert(sizeof(uint32_t) * head_lds<1024, false>(kCapacityMax).lists + sizeof(TopkSmem) + 64 <= 160 * 1024, "end");
// loads of the caller's top-k list stay inside it, and an empty one, which may have no memory, is not touched
constexpr int32_t lists[8] = {}, other[1] = {};
constexpr bool inside() {
  for (int count = 1; count <= 3; ++count)
    for (int t = 0; t < 9; ++t)
      if (list_or(lists, 4, count, other) != lists + 4 || list_entry(t, count) != (t < count ? t : count - 1)) return false;
  for (int t = 0; t < 9; ++t)
    if (list_or(nullptr, 1 << 20, 0, other) != other || list_entry(t, 0) != 0) return false;
  return true;
}
static_assert(inside(), "list");
static_assert(kCapacityMax <= kMailTokens * (int)kMailSlots, "a slot's tokens");
"""

BESIDE = r"""
#include "vatt_internal.h"
using namespace vatt;
constexpr Plan plan(int heads, int q_len, int n, int rows, double eps, int target = VATT_TARGET_D, int d = 128) {
  Plan p{};
  p.num_cus = 256;
  p.vbatch = heads;
  p.p.n_q_heads = 1;
  p.q_len = q_len;
  p.p.n_max = n;
  p.k_max = rows;
  p.p.target = target;
  p.p.head_dim = d;
  p.z_half = 1.96;
  p.eps = eps;
  p.split_cap = (32 * 256 + heads - 1) / heads;
  p.split_cap = p.split_cap < 1 ? 1 : p.split_cap > 32 ? 32 : p.split_cap;
  p.given_splits = (16 * 256 + heads - 1) / heads;
  p.given_splits = p.given_splits < 1 ? 1 : p.given_splits > 16 ? 16 : p.given_splits;
  if (p.given_splits > p.split_cap) p.given_splits = p.split_cap;
  return p;
}
constexpr int fixed(int heads, int q_len, int n, int rows, double eps = 0.05, int target = VATT_TARGET_D) {
  return given_fixed_splits(plan(heads, q_len, n, rows, eps, target));
}
// calls that were slower with the rows beside the phase: short lists, a sample that is most of the residual, targets N and SDPA, more
// heads than the phases have compute units
static_assert(fixed(192, 1, 600, 271) == 0 && fixed(192, 1, 3000, 331) == 0 && fixed(32, 1, 4000, 356) == 0 && fixed(32, 1, 900, 526) == 0, "lists");
static_assert(fixed(192, 1, 9000, 481, 0.005) == 0 && fixed(512, 16, 9000, 481, 0.01) == 0, "budgets");
static_assert(fixed(128, 1, 9000, 481, 0.05, VATT_TARGET_SDPA) == 0 && fixed(128, 1, 9000, 481, 0.05, VATT_TARGET_N) == 0, "targets");
static_assert(fixed(512, 1, 32768, 1075) == 0 && fixed(960, 3, 32768, 1075) == 0 && fixed(512, 16, 1500, 556) == 0, "heads");
// calls that gain, with the workgroups that they gained most with
static_assert(fixed(192, 1, 12000, 556) == 3 && fixed(256, 1, 30000, 1006) == 2 && fixed(128, 1, 131072, 1950) == 4 && fixed(32, 1, 100000, 2756) == 6, "apart");
static_assert(fixed(512, 16, 9000, 481) == 2 && fixed(512, 16, 32768, 6809) == 7, "query tokens");
// a partial sum for every workgroup, one of them behind the phase at least, and no workgroup without a row in the longest list
constexpr bool sound() {
  for (int heads = 1; heads <= 1100; heads += 13)
    for (int rows = 1; rows < 40000; rows += rows < 3000 ? 111 : 3001)
      for (int given = 1; given <= 32; given += given < 3 ? 1 : 7)
        for (int d = 64; d <= 128; d += 64) {
          Plan p = plan(heads, 4, 131072, rows, 0.05, VATT_TARGET_D, d);
          if (given <= p.split_cap) p.given_splits = given;
          const int f = given_fixed_splits(p), t = given_tail_splits(p);
          if (f < 0 || t < 1 || (f > 0 && f + t > given_part_slots(p)) || (f > 0 && (f - 1) * fixed_step_rows(d) >= rows)) return false;
          if (t > p.given_splits || (f == 0 && t != p.given_splits) || f + t > 64) return false;
        }
  return true;
}
static_assert(sound(), "splits");
"""


def _compiles(tmp_path, text):
    src = tmp_path / "check.hip"
    src.write_text(text)
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", "--cuda-host-only", "-std=c++17", "-fsyntax-only", "-Wno-unused-function",
                        "-fconstexpr-steps=20000000", "-I", CSRC, str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]


def test_lds_places_and_list_reads(tmp_path):
    _compiles(tmp_path, CHECK)


def test_which_steps_gather_the_fixed_set_beside_the_second_phase(tmp_path):
    _compiles(tmp_path, BESIDE)
