// Tags of the panels' exchange words: the rule alone, without device code
// (constexpr, so that the kernels and host tests share it).
#pragma once
#include <stdint.h>

namespace ozp {

constexpr uint32_t PANEL_TAGS = 1024;  // a panel has at most 512 columns

// The word `end` of a handle marks the last range of tags that its
// factorisations used, 0 at first.  The next one takes PANEL_TAGS for each of
// its panels; where they would pass 2^32 the exchange words are cleared and
// the ranges start over, so that no word can hold a tag that comes again.
struct TagRange {
  uint32_t end;
  bool clear;
};
constexpr TagRange next_tags(uint32_t end, uint32_t panels) {
  const uint64_t e = (uint64_t)end + (uint64_t)PANEL_TAGS * panels;
  return e + PANEL_TAGS > 0xffffffffull ? TagRange{PANEL_TAGS * panels, true}
                                        : TagRange{(uint32_t)e, false};
}

// tag of column 0 of a factorisation's panel (never 0, which cleared words hold)
constexpr uint32_t panel_tag0(uint32_t end, uint32_t panel) { return end - PANEL_TAGS * panel + 1u; }

}  // namespace ozp
