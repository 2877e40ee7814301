// The texts of bounded verification: which stretch of a bin's bases is aligned,
// and in which parts. Plain integer code, shared by the kernels and its CPU test.
#pragma once

#include <cstdint>

namespace grim {

// A span [x, y) of a text, as 32-bit offsets from its start. y = kWholeText
// stands for all of the text, however long; a span that ends there by itself
// does not occur (texts of 2^32 - 1 bases and more always get the mark).
constexpr uint32_t kWholeText = 0xFFFFFFFFu;
constexpr uint32_t kPart = 192;      // columns of a part
constexpr uint32_t kTextParts = 64;  // parts of a text, at most

// Parts of a span for a read of L bases: all but the last end one step of columns
// after the one before. A span is cut where that saves its length by half; whole
// texts that the sift could not look through are not. 0: nothing to align.
// Offsets may be as large as 2^32 - 2, so no sum is formed before a division.
constexpr uint32_t span_parts(uint32_t x, uint32_t y, uint32_t L) {
  if (x >= y) return 0;
  const uint32_t len = y - x, reach = 2 * L;  // L + E, E < L
  if (y == kWholeText || len < 2 * (kPart + reach)) return 1;
  const uint32_t n = (len - 1) / kPart + 1;
  return n < kTextParts ? n : kTextParts;
}

// Columns between the ends of np parts.
constexpr uint32_t part_step(uint32_t x, uint32_t y, uint32_t np) { return (y - x - 1) / np + 1; }

// Part u of np of span [x, y) of the text [lo, hi), and the `back` columns before
// it that an alignment ending there can reach; widened to whole 16-byte loads.
struct TextPart {
  uint64_t lo, hi;
};
constexpr TextPart text_part(uint64_t lo, uint64_t hi, uint32_t x, uint32_t y, uint32_t np, uint32_t u, uint32_t back) {
  if (y == kWholeText) return {lo, hi};
  const uint64_t step = part_step(x, y, np), before = u * step;
  const uint64_t end = x + before + step < y ? x + before + step : y;
  const uint64_t from = (lo + x + (before > back ? before - back : 0)) & ~15ull, to = (lo + end + 15) & ~15ull;
  return {from > lo ? from : lo, to < hi ? to : hi};
}

}  // namespace grim
