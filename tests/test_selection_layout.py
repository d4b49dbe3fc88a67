"""Checked at compile time: the LDS layout that the selection kernels and their launch sizes share, for every capacity, and where
the kernel with the caller's top-k list reads that list."""
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



def test_lds_places_and_list_reads(tmp_path):
    src = tmp_path / "layout.hip"
    src.write_text(CHECK)
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", "--cuda-host-only", "-std=c++17", "-fsyntax-only", "-Wno-unused-function",
                        "-fconstexpr-steps=20000000", "-I", CSRC, str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
