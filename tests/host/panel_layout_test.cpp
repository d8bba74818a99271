// LDS layouts of the bitmap build over every bitmap length, brick counts around each limit and panel
// sizes with and without staging.  Every fault prints a line; the exit status says whether there was one.
#include "panel_layout.h"

#include <cstdio>

int main() {
  using namespace spmm;
  int faults = 0;
  for (uint32_t words = 64; words <= 32768; words *= 2)
    for (uint32_t bricks = 1; bricks <= 13000; ++bricks)
      for (uint32_t entries : {0u, 1u, 2047u, 2048u, 2049u, 50000u}) {
        const PanelBuildLayout l = panel_build_layout(words, bricks, entries);
        // patterns, bitmap, rank table of one more entry than groups, value offsets, staged words and order
        auto counted = [&](uint32_t group, uint32_t staged) {
          return (size_t)bricks * 8 + words * 4 + (words / group + 1) * 4 + (size_t)bricks * 4 + staged * 6;
        };
        const bool fits = counted(kGroupWords, 0) <= kPanelMaxLds;
        bool ok = fits == (l.bytes != 0);
        if (l.bytes)
          ok = ok && l.bytes == counted(l.group, l.stage_cap) && l.bytes <= kPanelMaxLds &&
               (l.group == 1 || l.group == kGroupWords) && l.stage_cap % 2 == 0;
        if (!ok && faults++ < 5)
          std::printf("words %u bricks %u entries %u: %zu bytes, group %u, %u staged\n", words, bricks,
                      entries, l.bytes, l.group, l.stage_cap);
      }
  if (faults) std::printf("%d faults\n", faults);
  return faults != 0;
}
