// CPU checks of the texts of bounded verification (verify_text.h): a span's parts
// leave no column out, up to texts at and beyond 32-bit lengths. Prints "OK".
#include <cstdio>
#include <cstdlib>
#include <random>

#include "verify_text.h"

using namespace grim;

#define CHECK(c)                                                          \
  do {                                                                    \
    if (!(c)) {                                                           \
      std::fprintf(stderr, "CHECK failed line %d: %s (x %u y %u L %u lo %llu)\n", __LINE__, #c, x, y, L, \
                   (unsigned long long)lo);                               \
      std::exit(1);                                                       \
    }                                                                     \
  } while (0)

// Every alignment that ends in (x, y] of the text and starts at most `back` before
// its end lies in one of the parts.
static void check_span(uint64_t lo, uint32_t x, uint32_t y, uint32_t L, uint32_t E, uint64_t text) {
  const uint32_t np = span_parts(x, y, L), back = L + E;
  const uint64_t hi = lo + text;
  CHECK(np >= 1 && np <= kTextParts);
  uint64_t done = lo + x;  // ends up to here are covered
  for (uint32_t u = 0; u < np; ++u) {
    const TextPart p = text_part(lo, hi, x, y, np, u, back);
    CHECK(p.lo >= lo && p.hi <= hi && p.lo < p.hi);
    CHECK(p.lo <= lo + x || p.lo + back <= done);
    CHECK(p.hi > done);
    CHECK(np == 1 || p.hi - p.lo <= uint64_t(part_step(x, y, np)) + back + 46);  // and no part is much longer
    done = p.hi;
  }
  CHECK(done >= lo + (y == kWholeText ? text : y));
}

int main() {
  std::mt19937_64 rng(11);
  using u64 = unsigned long long;
  const u64 top = 0xFFFFFFFFull;
  for (uint32_t L : {13u, 26u, 100u, 192u, 193u, 250u, 512u}) {
    for (uint32_t E : {0u, 1u, L / 13 - 1}) {
      for (u64 lo : {0ull, 2048ull, 16ull * 77777 + 5, (1ull << 33) + 3}) {
        for (u64 len : {1ull, 15ull, 383ull, 384ull, 385ull, 1000ull, 2300ull, 12287ull, 12288ull, 12289ull, 100000ull,
                             1ull << 31, (1ull << 31) + 1, top - 4096, top - 192, top - 191, top - 190, top - 64, top - 63,
                             top - 1}) {
          check_span(lo, 0, (uint32_t)len, L, E, len);
          for (u64 x : {1ull, 190ull, 4000ull, len / 2})
            if (x < len) check_span(lo, (uint32_t)x, (uint32_t)len, L, E, len + rng() % 100);
        }
        for (u64 text : {1ull, 2300ull, top - 1, top, top + 1, top + 1000, 2 * top}) {
          const uint32_t x = 0, y = kWholeText;
          check_span(lo, x, y, L, E, text);
          const TextPart p = text_part(lo, lo + text, x, y, 1, 0, L + E);
          CHECK(p.lo == lo && p.hi == lo + text);
        }
      }
    }
  }
  for (int i = 0; i < 200000; ++i) {
    const uint32_t y = (uint32_t)((rng() % (top - 1)) >> (rng() % 32)) + 1, x = (uint32_t)(rng() % y);
    const uint32_t L = 13 + rng() % 500;
    check_span(rng() >> 30, x, y, L, L / 13 - 1, y + rng() % 50);
  }
  if (span_parts(0, 0, 100) != 0 || span_parts(7, 7, 100) != 0) return 1;
  std::puts("OK");
}
