// LDS of k_panel_build (host code only).
#ifndef SPMM_PANEL_LAYOUT_H_
#define SPMM_PANEL_LAYOUT_H_

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace spmm {

constexpr uint32_t kGroupWords = 8;                 // bitmap words per entry of the coarse rank table
constexpr uint32_t kPanelFineWords = 2048;          // bitmaps with a rank per word (16 KiB with it)
constexpr uint32_t kPanelStageMax = 2048;           // entries of a panel staged in LDS (12 KiB)
constexpr size_t kPanelMaxLds = 150 * 1024;         // of the 160 KiB of a CU

struct PanelBuildLayout {
  uint32_t group = 0;       // bitmap words per entry of the rank table: 1 or kGroupWords
  uint32_t stage_cap = 0;   // entries staged
  size_t bytes = 0;         // dynamic LDS, at most kPanelMaxLds; 0: the panels do not fit
};

// bytes for a bitmap of words_cap words, panels of up to nb_cap bricks, rank table entries every
// `group` words and up to stage_cap staged entries
inline size_t panel_build_bytes(uint32_t words_cap, uint32_t nb_cap, uint32_t group, uint32_t stage_cap) {
  return (size_t)nb_cap * 8 + ((size_t)words_cap + words_cap / group + 1 + nb_cap) * 4 +
         (size_t)stage_cap * 6;
}

// A rank per word of the bitmap while that is short (no walk through a group of words for every
// entry) and LDS has room for it; staging for panels of up to kPanelStageMax entries, likewise.
inline PanelBuildLayout panel_build_layout(uint32_t words_cap, uint32_t nb_cap, uint32_t max_nnz) {
  PanelBuildLayout l;
  if (words_cap == 0 || panel_build_bytes(words_cap, nb_cap, kGroupWords, 0) > kPanelMaxLds) return l;
  const bool fine = words_cap <= kPanelFineWords && panel_build_bytes(words_cap, nb_cap, 1, 0) <= kPanelMaxLds;
  l.group = fine ? 1 : kGroupWords;
  l.stage_cap = (std::min(max_nnz, kPanelStageMax) + 1) & ~1u;
  if (panel_build_bytes(words_cap, nb_cap, l.group, l.stage_cap) > kPanelMaxLds) l.stage_cap = 0;
  l.bytes = panel_build_bytes(words_cap, nb_cap, l.group, l.stage_cap);
  return l;
}

}  // namespace spmm
#endif  // SPMM_PANEL_LAYOUT_H_
