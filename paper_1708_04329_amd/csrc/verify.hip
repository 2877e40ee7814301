// Verification of filtered locations: the alignment step that follows the
// filter in a seed-and-extend mapper (paper Section 1, step 5; Section 5
// counts a passing location that yields no mapping against the filter).
//
// For a (read, bin) pair the result is the smallest Levenshtein distance
// between the whole read and any substring of the bases bin x's tokens cover,
// [x*B, min(x*B + B + O + q - 1, G)). It is computed with Myers' bit-vector
// algorithm (G. Myers, "A fast bit-vector algorithm for approximate string
// matching based on dynamic programming", J. ACM 46(3), 1999): one column of
// the dynamic-programming matrix is held as vertical +1/-1 difference bits,
// 32 rows per uint32 word, and each reference base advances every word with
// a dozen bitwise operations and one add. Reads longer than 32 bases use
// Myers' block form: word w hands its top row's horizontal difference to
// word w + 1. Row 0 has horizontal difference 0 in every column, so an
// alignment may start anywhere in the text, and the distance is the minimum
// over all columns of the last row.
//
// The read's match masks are kept as two code bit planes and a validity
// plane, so a text base selects its mask with two three-input operations
// per word; 16-byte text chunks holding a byte other than A, C, G, T (N
// runs) take a checked step that masks it out.
//
// Work split: one lane per pair. A first pass counts the pairs to align per
// class (words per read, 1..16) and writes the outputs of the pairs it skips; a
// prefix over chunks of reads turns the counts into list positions (no global
// atomics, which would serialise on a few class counters); a second pass lists
// the pairs class by class, so that one launch per class runs lanes with equal
// word counts in lock step.
//
// The bounded form first looks for the pairs that can map at all (k_verify_sift):
// of E + 1 disjoint pieces of a read, E edits leave one untouched, so a bin
// that holds none of them exactly is further than E. Only the others, and of
// their bins only the stretch around the pieces found, are aligned. Reads whose
// pieces would be too short have classes of their own, and their bins are aligned
// whole as in the exact form.

#include <algorithm>
#include <cstdlib>

#include "grim_internal.h"
#include "verify_text.h"

namespace grim {
namespace {

constexpr uint32_t kSkipped = 0xFFFFu;
constexpr int kGroups = 16;

// Selection of pair k: a valid bin, and the mask (if any) set.
__device__ __forceinline__ bool selected(const VerifyArgs& a, int32_t x, uint8_t m) {
  return x >= 0 && (uint64_t)x < a.nb && (!a.verify_mask || m);
}

// Bin ids and mask bytes of kGroups consecutive 64-pair groups from k0, all
// loads issued before the first wait (past the end: the read's last pair,
// ignored by the caller).
__device__ __forceinline__ void load_groups(const VerifyArgs& a, int64_t k0, int64_t c1, uint32_t lane,
                                            int32_t (&x)[kGroups], uint8_t (&m)[kGroups]) {
#pragma unroll
  for (int u = 0; u < kGroups; ++u) x[u] = a.cand_bin[min(k0 + u * 64 + (int64_t)lane, c1 - 1)];
  if (a.verify_mask) {
#pragma unroll
    for (int u = 0; u < kGroups; ++u) m[u] = a.verify_mask[min(k0 + u * 64 + (int64_t)lane, c1 - 1)];
  } else {
#pragma unroll
    for (int u = 0; u < kGroups; ++u) m[u] = 1;
  }
}

// Pieces of a read of L bases that the sift looks for, of which E edits leave one
// untouched (see k_verify_sift); 0 where it cannot.
constexpr uint32_t kMinPiece = 13;
constexpr uint32_t kMaxPieces = 32;
__device__ __forceinline__ uint32_t sift_pieces(int64_t E, uint32_t L) {
  return E >= 0 && E < (int64_t)kMaxPieces && L / (uint32_t)(E + 1) >= kMinPiece ? (uint32_t)E + 1 : 0u;
}

// Work list of read r; 0: it has no bases or too many.
__device__ __forceinline__ uint32_t list_class(const VerifyArgs& a, uint64_t r) {
  const uint64_t L = (uint64_t)(a.offsets[r + 1] - a.offsets[r]);
  if (L == 0 || L > kVerifyMaxLen) return 0u;
  const uint32_t words = (uint32_t)((L + 31) / 32);
  if (!a.bounded) return words;
  // E_r from the threshold, which is at least -2^30
  const int32_t E = ((int32_t)L - (int32_t)a.q + 1 - a.thr[r]) / (int32_t)a.q;
  return sift_pieces(E, (uint32_t)L) ? words : words + kVerifyWords;
}

// First pass, one workgroup of 16 wavefronts per chunk of reads, a wavefront
// per read: count the read's selected pairs (read_sel, with its class), write the outputs of the
// pairs it skips, and sum the counts per class (list_class) for the chunk
// (chunk_sum[class][chunk]). No global atomics: the list positions come from
// a prefix over chunks. Bound by the lists' bytes (5 in, 3 out per pair).
__global__ __launch_bounds__(1024) void k_verify_count(VerifyArgs a) {
  __shared__ unsigned long long csum[kVerifyBuckets];
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  if (threadIdx.x < kVerifyBuckets) csum[threadIdx.x] = 0;
  __syncthreads();
  const bool rejected = a.status[0] & ~(uint32_t)(ST_BAD_BIN | ST_BAD_CAND_OFF | ST_VERIFY_LONG);
  const uint64_t r_lo = (uint64_t)blockIdx.x * a.chunk;
  const uint64_t r_hi = min(a.n_reads, r_lo + a.chunk);
  for (uint64_t r = r_lo + wave; r < r_hi && !rejected; r += 16) {
    const int64_t c0 = a.cand_off[r], c1 = a.cand_off[r + 1];
    if (c0 < 0 || c1 < c0 || (uint64_t)c1 > a.n_cand || c1 - c0 > 0xFFFFFFFFll) {
      if (lane == 0) {
        atomicOr(a.status, ST_BAD_CAND_OFF);
        a.read_sel[r] = make_uint2(0, 0);
      }
      continue;
    }
    const uint32_t cls = list_class(a, r);
    uint32_t n_sel = 0;
    for (int64_t k0 = c0; k0 < c1; k0 += kGroups * 64) {
      int32_t x[kGroups];
      uint8_t m[kGroups];
      load_groups(a, k0, c1, lane, x, m);
#pragma unroll
      for (int u = 0; u < kGroups; ++u) {
        const int64_t k = k0 + u * 64 + lane;
        bool sel = false;
        if (k < c1) {
          if (x[u] < 0 || (uint64_t)x[u] >= a.nb) atomicOr(a.status, ST_BAD_BIN);
          sel = selected(a, x[u], m[u]);
          if (!sel) {
            a.dist_out[k] = (uint16_t)kSkipped;
            a.match_out[k] = 0;
          }
        }
        n_sel += (uint32_t)__popcll(__ballot(sel));
      }
    }
    if (lane == 0) {
      a.read_sel[r] = make_uint2(n_sel, cls);
      if (n_sel) {
        if (cls == 0) atomicOr(a.status, ST_VERIFY_LONG);
        else atomicAdd(&csum[cls], (unsigned long long)n_sel);
      }
    }
  }
  __syncthreads();
  if (threadIdx.x < kVerifyBuckets) a.chunk_sum[(uint64_t)threadIdx.x * gridDim.x + blockIdx.x] = csum[threadIdx.x];
}

// One wavefront per class, 16 to a workgroup (class 0 holds no pairs): a scan over
// the chunks, 512 at a time (8 per lane, loaded together), turns
// chunk_sum[class][chunk] into the pairs of that class in the chunks before;
// bucket[class] gets the class's pair count (the host launches one alignment per
// class). Classes follow each other in the list in increasing order.
__device__ __forceinline__ uint64_t shfl_up64(uint64_t v, uint32_t d) {
  const uint32_t lo = (uint32_t)__shfl_up((int)(uint32_t)v, d), hi = (uint32_t)__shfl_up((int)(v >> 32), d);
  return ((uint64_t)hi << 32) | lo;
}

__global__ __launch_bounds__(1024) void k_verify_prefix(VerifyArgs a, uint64_t n_chunks) {
  constexpr uint32_t kPer = 8;
  const uint32_t lane = threadIdx.x & 63u, c = 1 + kVerifyWords * blockIdx.x + (threadIdx.x >> 6);
  uint64_t* sums = a.chunk_sum + (uint64_t)c * n_chunks;
  unsigned long long acc = 0;
  for (uint64_t k0 = 0; k0 < n_chunks; k0 += 64 * kPer) {
    const uint64_t k = k0 + lane * kPer;
    uint64_t v[kPer], sum = 0;
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) v[j] = k + j < n_chunks ? sums[k + j] : 0;
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) sum += v[j];
    uint64_t incl = sum;
#pragma unroll
    for (uint32_t d = 1; d < 64; d <<= 1) {
      const uint64_t t = shfl_up64(incl, d);
      if (lane >= d) incl += t;
    }
    uint64_t run = acc + incl - sum;
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
      if (k + j < n_chunks) sums[k + j] = run;
      run += v[j];
    }
    acc += ((uint64_t)(uint32_t)__shfl((int)(incl >> 32), 63) << 32) | (uint32_t)__shfl((int)(uint32_t)incl, 63);
  }
  if (lane == 0) a.bucket[c] = acc;
  if (c == 1 && lane == 0) a.bucket[0] = 0;
}

// Second pass, same chunks: each wavefront claims its read's slots in the
// read's class (a cursor per class in LDS; reads of a class may come in any
// order) and lists the read's selected pairs in pair order. The first pass has
// checked every bin, so the mask alone selects. Handing out the slots with one
// thread per class over chunks of 2048 reads took 400 us whatever the size.
__global__ __launch_bounds__(1024) void k_verify_scatter(VerifyArgs a) {
  __shared__ unsigned long long cur[kVerifyBuckets];
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const uint64_t r_lo = (uint64_t)blockIdx.x * a.chunk;
  const uint64_t r_hi = min(a.n_reads, r_lo + a.chunk);
  if (wave == 0) {  // the pairs of the classes before, and of the class in the chunks before
    const bool used = lane >= 1 && lane <= (a.bounded ? 2 * kVerifyWords : kVerifyWords);
    const uint64_t pairs = used ? a.bucket[lane] : 0;
    const uint64_t before = used ? a.chunk_sum[(uint64_t)lane * gridDim.x + blockIdx.x] : 0;
    uint64_t incl = pairs;
#pragma unroll
    for (uint32_t d = 1; d < 64; d <<= 1) {
      const uint64_t t = shfl_up64(incl, d);
      if (lane >= d) incl += t;
    }
    if (used) cur[lane] = incl - pairs + before;
  }
  __syncthreads();
  for (uint64_t r = r_lo + wave; r < r_hi; r += 16) {
    const uint32_t n_sel = a.read_sel[r].x, cls = a.read_sel[r].y;
    if (n_sel == 0 || cls == 0) continue;
    const int64_t c0 = a.cand_off[r], c1 = a.cand_off[r + 1];
    unsigned long long claim = 0;
    if (lane == 0) claim = atomicAdd(&cur[cls], (unsigned long long)n_sel);
    uint64_t pos0 = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(claim >> 32)) << 32) |
                    (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)claim);
    if (a.verify_mask && (int64_t)n_sel * 8 < c1 - c0) {
      // few of many: 16 mask bytes per lane, then only the selected are touched
      for (int64_t k0 = c0; k0 < c1; k0 += 1024) {
        const int64_t k = k0 + 16 * (int64_t)lane;
        uint32_t v[4] = {0, 0, 0, 0};
        if (k + 16 <= c1) {
          __builtin_memcpy(v, a.verify_mask + k, 16);
        } else {
          for (int64_t i = k; i < c1; ++i) v[(i - k) >> 2] |= (uint32_t)a.verify_mask[i] << (8 * ((i - k) & 3));
        }
        uint32_t mine = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {  // bit 7 of each byte that is not zero
          v[i] = (((v[i] & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | v[i]) & 0x80808080u;
          mine += (uint32_t)__popc(v[i]);
        }
        uint32_t incl = mine;
        for (int d = 1; d < 64; d <<= 1) {
          const uint32_t y = (uint32_t)__shfl_up((int)incl, d);
          if ((int)lane >= d) incl += y;
        }
        uint64_t pos = pos0 + incl - mine;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          for (uint32_t b = v[i]; b; b &= b - 1) {
            a.item_pair[pos] = (uint64_t)(k + 4 * i + (__ffs((int)b) - 1) / 8);
            a.item_read[pos++] = (uint32_t)r;
          }
        pos0 += (uint32_t)__shfl((int)incl, 63);
      }
      continue;
    }
    for (int64_t k0 = c0; k0 < c1; k0 += kGroups * 64) {
      uint8_t m[kGroups];
#pragma unroll
      for (int u = 0; u < kGroups; ++u)
        m[u] = a.verify_mask ? a.verify_mask[min(k0 + u * 64 + (int64_t)lane, c1 - 1)] : (uint8_t)1;
#pragma unroll
      for (int u = 0; u < kGroups; ++u) {
        const int64_t k = k0 + u * 64 + lane;
        const bool sel = k < c1 && m[u];
        const uint64_t bal = __ballot(sel);
        if (sel) {
          const uint64_t pos = pos0 + (uint64_t)__popcll(bal & ((1ull << lane) - 1ull));
          a.item_pair[pos] = (uint64_t)k;
          a.item_read[pos] = (uint32_t)r;
        }
        pos0 += (uint64_t)__popcll(bal);
      }
    }
  }
}

// Myers' column step for W words. The read is held as bit planes: bit i of
// word w of r0 / r1 is bit 0 / bit 1 of the code of read base 32w + i, and
// va marks the bases that are A, C, G or T; so the match mask of text code c
// is va & ~(r0 ^ c0) & ~(r1 ^ c1) with c0, c1 the bits of c spread to all
// 32 positions, two three-input operations per word. pv/mv: vertical +1/-1
// bits of the current column; `top` is the read's last row within word
// W - 1, whose distance `score` tracks. The W words are one long integer: the
// addition's carry runs through them (add with carry), which is what a -1
// entering a word from below does in the block form, without that form's two
// operations per word: 12 operations per word and column, 16.3 before (975910
// pairs of 100 bp and 2.3 kbp 2.9 ms, 3.7 before; bound by VALU issue).
// CHECKED steps also accept text bytes other than 0..3 (they match nothing).
template <int W>
struct Column {
  uint32_t r0[W], r1[W], va[W];
  uint32_t pv[W], mv[W];
  uint32_t top;
  int32_t score, best;

  template <bool CHECKED>
  __device__ __forceinline__ void step(uint32_t c) {
    const uint32_t c0 = 0u - (c & 1u), c1 = 0u - ((c >> 1) & 1u);
    const uint32_t valid = (!CHECKED || c < 4u) ? 0xFFFFFFFFu : 0u;
    // the previous word's unshifted horizontal +1/-1 bits, whose top bits enter
    // this word's bottom row (0 below word 0)
    uint32_t php = 0, mhp = 0, carry = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      // truth tables of bitop3 over (src0, src1, src2) = 0xF0, 0xCC, 0xAA
      uint32_t eq = __builtin_amdgcn_bitop3_b32(va[w], r0[w], c0, 0x90);  // va & ~(r0 ^ c0)
      eq = __builtin_amdgcn_bitop3_b32(eq, r1[w], c1, 0x90);              //    & ~(r1 ^ c1)
      if (CHECKED) eq &= valid;
      const uint32_t xv = eq | mv[w];
      const uint32_t sum = __builtin_addc(eq & pv[w], pv[w], carry, &carry);
      const uint32_t xh = __builtin_amdgcn_bitop3_b32(sum, pv[w], eq, 0xBE);  // (sum ^ pv) | eq
      const uint32_t ph = __builtin_amdgcn_bitop3_b32(mv[w], xh, pv[w], 0xF1);  // mv | ~(xh | pv)
      const uint32_t mh = pv[w] & xh;
      if (w == W - 1)
        score += (int32_t)__builtin_amdgcn_ubfe(ph, top, 1u) + (int32_t)__builtin_amdgcn_sbfe((int)mh, top, 1u);
      // shift up one row, the entering difference moving into row 0
      const uint32_t phs = __builtin_amdgcn_alignbit(ph, php, 31);
      const uint32_t mhs = __builtin_amdgcn_alignbit(mh, mhp, 31);
      pv[w] = __builtin_amdgcn_bitop3_b32(mhs, xv, phs, 0xF1);  // mhs | ~(xv | phs)
      mv[w] = phs & xv;
      php = ph;
      mhp = mh;
    }
    best = min(best, score);
  }
};

// A pair's read and bin: the read's bases and budget, the bases bin x's tokens
// cover, text [lo, hi).
struct Pair {
  const uint8_t* rd;
  uint32_t L;
  int64_t E;  // the read's error budget, recovered from its threshold
  uint64_t lo, hi;
};

__device__ __forceinline__ Pair pair_of(const VerifyArgs& a, uint32_t r, uint32_t x) {
  Pair p;
  const int64_t o0 = a.offsets[r];
  p.rd = a.bases + o0;
  p.L = (uint32_t)(a.offsets[r + 1] - o0);
  p.E = ((int64_t)p.L - (int64_t)a.q + 1 - (int64_t)a.thr[r]) / (int64_t)a.q;
  const uint64_t starts_end = a.G >= a.q ? a.G - a.q + 1 : 0;
  p.lo = (uint64_t)x * a.B;
  p.hi = p.lo + a.B + a.O;
  if (p.hi > starts_end) p.hi = starts_end;
  if (p.lo > p.hi) p.lo = p.hi;
  p.hi = p.hi > p.lo ? p.hi + a.q - 1 : p.lo;
  return p;
}

// The smallest distance of pair p's read to a part of text [lo, hi) within its bin.
template <int W>
__device__ __forceinline__ int32_t align_text(const VerifyArgs& a, const Pair& p, uint64_t lo, uint64_t hi) {
  Column<W> col;
  const uint32_t L = p.L;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    // four bases at a time: codes in bits 0-1 of each byte, a letter compared
    // with the one its code names, and one bit per base gathered by a dot product
    uint32_t b0 = 0, b1 = 0, ok = 0;
#pragma unroll
    for (uint32_t b = 0; b < 32; b += 4) {
      const uint32_t l = read4(p.rd, (uint32_t)w * 32 + b, L) | 0x20202020u;
      const uint32_t c = ((l >> 1) ^ (l >> 2)) & 0x03030303u;
      const uint32_t d = __builtin_amdgcn_perm(0u, 0x74676361u, c) ^ l;  // byte k: "acgt"[c_k] ^ base k
      const uint32_t good = ~((((d & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | d) >> 7) & 0x01010101u;
      b0 |= __builtin_amdgcn_udot4(c & 0x01010101u, 0x08040201u, 0u, false) << b;
      b1 |= __builtin_amdgcn_udot4((c >> 1) & 0x01010101u, 0x08040201u, 0u, false) << b;
      ok |= __builtin_amdgcn_udot4(good, 0x08040201u, 0u, false) << b;
    }
    col.r0[w] = b0;
    col.r1[w] = b1;
    col.va[w] = ok;
    col.pv[w] = 0xFFFFFFFFu;  // column 0: row i holds distance i
    col.mv[w] = 0;
  }
  col.top = (L - 1) & 31u;
  col.best = col.score = (int32_t)L;

  const uint8_t* txt = a.ref;
  uint64_t j = lo;
  const uint64_t aligned = min(hi, (lo + 15) & ~15ull);
  for (; j < aligned; ++j) col.template step<true>(txt[j]);
  uint4 next = make_uint4(0, 0, 0, 0);
  if (j + 16 <= hi) next = *reinterpret_cast<const uint4*>(txt + j);
  for (; j + 16 <= hi; j += 16) {
    const uint4 v = next;
    if (j + 32 <= hi) next = *reinterpret_cast<const uint4*>(txt + j + 16);
    const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
    if (((v.x | v.y | v.z | v.w) & 0xFCFCFCFCu) == 0) {  // A, C, G, T only (the common case)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
        for (int by = 0; by < 4; ++by) col.template step<false>((wv[q4] >> (8 * by)) & 0xFFu);
    } else {
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
        for (int by = 0; by < 4; ++by) col.template step<true>((wv[q4] >> (8 * by)) & 0xFFu);
    }
  }
  for (; j < hi; ++j) col.template step<true>(txt[j]);
  return col.best;
}

__device__ __forceinline__ void write_distance(const VerifyArgs& a, uint64_t k, int32_t best, int64_t E) {
  uint32_t d = (uint32_t)min(best, (int32_t)0xFFFE);
  if (a.bounded && (int64_t)d > E) d = (uint32_t)min<int64_t>(E + 1, 0xFFFE);  // the bounded output
  a.dist_out[k] = (uint16_t)d;
  a.match_out[k] = (int64_t)d <= E ? 1 : 0;
}

// The whole text of every listed pair, a lane each: all pairs in the exact form, in
// the bounded form those of reads that the sift cannot look through. These have
// lists of their own: cut to a workgroup of k_verify_left they ended unevenly (2M
// pairs of 100 bp reads at E = 10: 8.7 ms for the call). The full column serves
// them too: with Ukkonen's cutoff, which the add with carry does not allow, 200000
// such pairs took 1.43 ms, with it 1.10.
template <int W>
__global__ __launch_bounds__(256) void k_verify_align(VerifyArgs a, uint64_t first, uint64_t count) {
  const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= count) return;
  const uint64_t k = a.item_pair[first + t];
  const Pair p = pair_of(a, a.item_read[first + t], (uint32_t)a.cand_bin[k]);
  write_distance(a, k, align_text<W>(a, p, p.lo, p.hi), p.E);
}

// ---------------------------------------------------------------------------
// The bounded form's sift. A pair within E edits holds one of E + 1 disjoint
// pieces of its read unedited, so a bin without an occurrence of a piece is
// further than E: its result is E + 1 without an alignment. With pieces of
// p = min(16, L / (E + 1)) bases, at least kMinPiece, chance occurrences in a
// 2.3 kbp bin are rare (5% error rates give p = 16).
//
// A wavefront takes 64 listed pairs, four at a time on 16 lanes each. The 16
// lanes read 256 consecutive bytes of the bin per step and pack 16 bases to a
// word. An occurrence of a piece covers, at one of its four phases, p - 3 bases
// that start at a multiple of four of the text, so a lane looks up four windows
// per 16 bases (the next lane's word supplies their ends) in a bitmap of 2^13
// bits in LDS, which holds the first 13 bits of the windows' codes for every
// piece and phase. What is found there is looked up by its last 13 bits in a
// second one, then the p bases at its four phases in a third, hashed: chance
// occurrences, like a base other than A, C, G, T (read as some base here), only
// let a pair through. About 45 operations per 16 bases and lane whatever the
// number of pieces (comparing each window with every code took 190), against
// 12 per 32 rows and base in the alignment. Bound by the bins' bytes, each read
// for one pair: 752065 pairs of the 3.1 Gbp reference (100003 reads of 100-250
// bp) take 0.61 ms, 2.8 TB/s, and the alignments of what is left 0.94 ms; without
// the sift the alignments took 5.1 ms.
// ---------------------------------------------------------------------------
constexpr uint32_t kMapBits = 13, kMapWords = (1u << kMapBits) / 32;

// 16 text or read bases of code bytes (bits 0-1), the first most significant.
__device__ __forceinline__ uint32_t pack16(const uint4& v) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  uint32_t q = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) q = __builtin_amdgcn_udot4(w[i] & 0x03030303u, 0x01041040u, q << 8, false);
  return q;
}

// Per pair in flight: bitmaps of the first (0) and last (1) 13 bits of its
// read's window codes and of its pieces (2, hashed), and the packed read while
// they are made.
struct SiftLds {
  uint32_t map[3][kMapWords];
  uint32_t words[kVerifyMaxLen / 16 + 2];
  uint32_t pad[2];
};
static_assert(sizeof(SiftLds) % 16 == 0, "16-byte stores");

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The bit of window code t (left-justified) in a bitmap indexed by t >> shift.
__device__ __forceinline__ uint32_t map_bit(const uint32_t* map, uint32_t t, uint32_t shift) {
  const uint32_t i = t >> shift;
  return map[(i >> 5) & (kMapWords - 1)] >> (i & 31u);
}

__device__ __forceinline__ uint32_t piece_hash(uint32_t code) { return code * 0x9E3779B1u; }

// Sifts items [0, count): item_span[t] = the part of the pair's text, as offsets
// from its start, that an alignment within the budget lies in: what one that
// touches a found piece can cover. Empty (0, 0) where none was found, and then
// the pair's outputs are written here. Texts too long for the offsets get all of
// theirs, (0, kWholeText).
__global__ __launch_bounds__(256) void k_verify_sift(VerifyArgs a, uint64_t count) {
  __shared__ __attribute__((aligned(16))) SiftLds lds_all[4][4];
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, sub = lane >> 4, j = lane & 15u;
  const uint64_t t0 = ((uint64_t)blockIdx.x * 4 + wave) * 64, t = t0 + lane;
  if (t0 >= count) return;
  // every lane looks its own pair up; the 16 lanes that sift it get the values
  // by shuffles (looked up by each step, the chain of loads took longer than
  // the step)
  uint64_t my_pair = 0;
  uint32_t my_read = 0, my_np = 0, my_L = 0, my_blocks = 0;
  uint64_t my_rd = 0, my_txt = 0;
  Pair mine{};
  if (t < count) {
    my_pair = a.item_pair[t];
    my_read = a.item_read[t];
    mine = pair_of(a, my_read, (uint32_t)a.cand_bin[my_pair]);
    my_np = sift_pieces(mine.E, mine.L);
    my_L = mine.L;
    my_rd = (uint64_t)(mine.rd - a.bases);
    my_txt = mine.lo & ~15ull;
    // the bin's blocks and one more, in which the last block's windows are looked up
    if (mine.hi > mine.lo) my_blocks = (uint32_t)min<uint64_t>((mine.hi - my_txt + 15) / 16 + 1, 0xFFFFFFF0ull);
  }
  const bool my_sift = my_np != 0;
  uint32_t my_lo = 0, my_hi = 0;  // blocks with a piece (see below)
  SiftLds& lds = lds_all[wave][sub];
  // shift to a window's last 13 bits, mask of a piece's code, the read that the bitmaps hold
  uint32_t last = 0, piece = 0, have = 0xFFFFFFFFu;
  // step s takes lanes 16 sub .. 16 sub + 15's own s-th items, which mostly share
  // their read; the next step's read bases and first block come in meanwhile
  struct Next {
    uint32_t r, np, L, blocks;
    const uint8_t* rd;
    const uint4* txt;
    uint32_t w[4];  // the read's bases 16 j .. 16 j + 15
    uint4 text;
  };
  auto take = [&](uint32_t s) {
    Next x;
    const int src = (int)(16 * sub + (s & 15u));
    auto from = [&](uint32_t v) { return (uint32_t)__shfl((int)v, src); };
    auto from64 = [&](uint64_t v) { return ((uint64_t)from((uint32_t)(v >> 32)) << 32) | from((uint32_t)v); };
    x.r = from(my_read);
    x.np = from(my_np);
    x.L = from(my_L);
    x.blocks = x.np ? from(my_blocks) : (from(my_blocks), 0u);
    x.rd = a.bases + from64(my_rd);
    x.txt = reinterpret_cast<const uint4*>(a.ref + from64(my_txt));
    x.text = make_uint4(0, 0, 0, 0);
    for (uint32_t i = 0; i < 4; ++i) x.w[i] = 0;
    if (s < 16 && x.np) {
      if (j < x.blocks) x.text = x.txt[j];
      if (16 * j < x.L)
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) x.w[i] = read4(x.rd, 16 * j + 4 * i, x.L);
    }
    return x;
  };
  Next ahead = take(0);
  for (uint32_t s = 0; s < 16; ++s) {
    const Next p = ahead;
    ahead = take(s + 1);
    const uint32_t r = p.r;
    const bool live = p.np != 0;
    if (!__any(live)) continue;
    if (__any(live && r != have)) {
      if (live) {
        uint4* m = reinterpret_cast<uint4*>(&lds.map[0][0]);
#pragma unroll
        for (uint32_t i = 0; i < 3 * kMapWords / 4; i += 16) m[i + j] = make_uint4(0, 0, 0, 0);
        for (uint32_t w = j; 16 * w < p.L; w += 16) {
          uint32_t q = 0;
#pragma unroll
          for (uint32_t i = 0; i < 4; ++i) {
            const uint32_t l = w == j ? p.w[i] : read4(p.rd, 16 * w + 4 * i, p.L);
            q = __builtin_amdgcn_udot4(((l >> 1) ^ (l >> 2)) & 0x03030303u, 0x01041040u, q << 8, false);
          }
          lds.words[w] = q;
        }
      }
      wave_lds_sync();
      if (live) {
        const uint32_t np = p.np, len = min(16u, p.L / np);
        last = 32 - 2 * (len - 3);
        piece = 0xFFFFFFFFu << (32 - 2 * len);
        for (uint32_t i = j; i < 4 * np; i += 16) {  // piece i / 4 at phase i % 4
          const uint32_t b = (i >> 2) * len + (i & 3u);
          const uint64_t two = ((uint64_t)lds.words[b >> 4] << 32) | lds.words[(b >> 4) + 1];
          const uint32_t code = (uint32_t)((two << (2 * (b & 15u))) >> 32);
          const uint32_t i0 = code >> (32 - kMapBits), i1 = code >> last;
          atomicOr(&lds.map[0][i0 >> 5], 1u << (i0 & 31u));
          atomicOr(&lds.map[1][(i1 >> 5) & (kMapWords - 1)], 1u << (i1 & 31u));
          if ((i & 3u) == 0) {
            const uint32_t h = piece_hash(code & piece) >> (32 - kMapBits);
            atomicOr(&lds.map[2][h >> 5], 1u << (h & 31u));
          }
        }
        have = r;
      }
      wave_lds_sync();
    }
    const uint32_t n_blocks = p.blocks;
    uint32_t hit_lo = 0xFFFFFFFFu, hit_hi = 0;
    uint32_t before = 0, before2 = 0;  // lane 0's previous blocks: lanes 15's and 14's of the step before
    uint4 next = p.text;
    for (uint32_t n = j; __any(n < n_blocks); n += 16) {
      const uint4 v = next;
      if (n + 16 < n_blocks) next = p.txt[n + 16];
      const uint32_t q = pack16(v);
      const uint32_t ror = (uint32_t)__builtin_amdgcn_mov_dpp((int)q, 0x121, 0xF, 0xF, false);  // lane j - 1's, cyclic
      const uint32_t prev = j == 0 ? before : ror;
      before = ror;
      const uint32_t ror2 = (uint32_t)__builtin_amdgcn_mov_dpp((int)prev, 0x121, 0xF, 0xF, false);
      const uint32_t prev2 = j == 0 ? before2 : ror2;
      before2 = ror2;
      uint32_t w[4], first[4];
      w[0] = prev;
#pragma unroll
      for (int f = 1; f < 4; ++f) w[f] = __builtin_amdgcn_alignbit(prev, q, 32 - 8 * f);
#pragma unroll
      for (int f = 0; f < 4; ++f) first[f] = map_bit(lds.map[0], w[f], 32 - kMapBits);
      const bool in = n < n_blocks;
      if (__any(in && ((first[0] | first[1] | first[2] | first[3]) & 1u))) {
        bool hit = false;
#pragma unroll
        for (int f = 0; f < 4; ++f) {
          const bool both = in && (first[f] & map_bit(lds.map[1], w[f], last) & 1u);
          if (!__any(both)) continue;
          uint32_t found = 0;
#pragma unroll
          for (int ph = 0; ph < 4; ++ph) {
            constexpr uint32_t kShift = 32 - kMapBits;
            const int o = 4 * f - ph;  // a piece starts here, from the start of block n - 1
            const uint32_t c = o == 0  ? prev
                               : o > 0 ? __builtin_amdgcn_alignbit(prev, q, 32 - 2 * o)
                                       : __builtin_amdgcn_alignbit(prev2, prev, -2 * o);
            found |= map_bit(lds.map[2], piece_hash(c & piece), kShift);
          }
          hit |= both && (found & 1u);
        }
        if (hit) {  // block n - 1, counted from 1 so that block -1 is 0
          hit_lo = min(hit_lo, n);
          hit_hi = max(hit_hi, n);
        }
      }
    }
    if (__any(hit_lo != 0xFFFFFFFFu)) {
      for (int d = 1; d < 16; d <<= 1) {
        hit_lo = min(hit_lo, (uint32_t)__shfl_xor((int)hit_lo, d));
        hit_hi = max(hit_hi, (uint32_t)__shfl_xor((int)hit_hi, d));
      }
    }
    if (j == s && my_sift) {  // the lane that holds the pair
      my_lo = hit_lo;
      my_hi = hit_hi;
    }
  }
  if (t >= count) return;
  uint2 span = make_uint2(0, kWholeText);
  if (my_sift && my_lo > my_hi) {
    span = make_uint2(0, 0);
    write_distance(a, my_pair, 0xFFFE, mine.E);
  } else if (my_sift) {
    const int64_t reach = (int64_t)mine.L + mine.E, off = (int64_t)(mine.lo & 15u), len = (int64_t)(mine.hi - mine.lo);
    if (len < (int64_t)kWholeText)
      span = make_uint2((uint32_t)max<int64_t>(0, 16 * ((int64_t)my_lo - 1) - off - reach),
                        (uint32_t)min<int64_t>(len, 16 * ((int64_t)my_hi + 1) - off + reach));
  }
  a.item_span[t] = span;
}

// Alignment of the sifted pairs. A workgroup cuts the text of those of `per`
// listed pairs that are left into parts of kPart columns and the L + E before
// them that an alignment ending there can reach back, orders the parts by
// length, so that a wavefront's lanes end together, and aligns them a lane
// each. (With whole texts in list order a wavefront ran to its longest of 64
// lanes, five times the mean, and a whole bin of 2.3 kbp alone took 0.5 ms.)
// Bound by the chain of a lane's columns, so every class of read lengths is in
// one launch, that as many workgroups as fit are there to hide it: for 752065
// listed pairs of 100-250 bp reads, launches by class (512, 512 and 358
// workgroups one after the other) took 1.47 ms, one 1.07 with 1024 workgroups and
// parts of 384 columns, 0.94 with 2048 and 192 (96 columns 0.96, 4096 workgroups
// 0.96: more columns before the parts, fewer parts to order).
constexpr uint32_t kMostLeft = 2048;
constexpr uint32_t kMostParts = 4096;
constexpr uint64_t kLeftBlocks = 2048;

struct LeftLds {
  uint32_t part[kMostParts];  // item | part << 11
  uint32_t best_of[kMostLeft];
  uint32_t cur[64];
  uint32_t n_parts;
};
static_assert(kMostLeft == 1u << 11, "item bits of a part");

// Items [t0, t0 + n), reads of W words, by one workgroup.
template <int W>
__device__ __forceinline__ void left_items(const VerifyArgs& a, uint64_t t0, uint32_t n, LeftLds& lds) {
  uint32_t* const part = lds.part;
  uint32_t* const best_of = lds.best_of;
  uint32_t* const cur = lds.cur;
  uint32_t& n_parts = lds.n_parts;
  const uint32_t t = threadIdx.x;
  if (t < 64) cur[t] = 0;
  for (uint32_t i = t; i < n; i += 256) best_of[i] = 0xFFFFFFFFu;
  // parts of an item's text; the read's length is looked up only where it may be cut
  auto parts_of = [&](uint2 sp, uint32_t item) -> uint32_t {
    if (sp.y - sp.x < 2 * kPart) return sp.x < sp.y ? 1u : 0u;
    const uint32_t r = a.item_read[t0 + item];
    return span_parts(sp.x, sp.y, (uint32_t)(a.offsets[r + 1] - a.offsets[r]));
  };
  auto bucket = [](uint2 sp, uint32_t np) {
    const uint32_t len = np == 1 ? sp.y - sp.x : part_step(sp.x, sp.y, np) + kPart;
    return 63u - min(len / 64u, 63u);
  };
  __syncthreads();
  for (uint32_t i = t; i < n; i += 256) {
    const uint2 sp = a.item_span[t0 + i];
    const uint32_t np = parts_of(sp, i);
    if (np) atomicAdd(&cur[bucket(sp, np)], np);
  }
  __syncthreads();
  if (t < 64) {
    const uint32_t v = cur[t];
    uint32_t x = v;
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = (uint32_t)__shfl_up((int)x, d);
      if ((int)t >= d) x += y;
    }
    cur[t] = x - v;
    if (t == 63) n_parts = x;
  }
  __syncthreads();
  const bool whole = n_parts > kMostParts;  // more parts than the table holds: texts as they are
  for (uint32_t i = t; i < n; i += 256) {
    const uint2 sp = a.item_span[t0 + i];
    const uint32_t np = parts_of(sp, i);
    if (whole) {
      part[i] = np ? i : 0xFFFFFFFFu;
    } else if (np) {
      const uint32_t at = atomicAdd(&cur[bucket(sp, np)], np);
      for (uint32_t u = 0; u < np; ++u) part[at + u] = i | u << 11;
    }
  }
  __syncthreads();
  const uint32_t m = whole ? n : n_parts;
  for (uint32_t i = t; i < m; i += 256) {
    if (part[i] == 0xFFFFFFFFu) continue;
    const uint32_t item = part[i] & (kMostLeft - 1), u = part[i] >> 11;
    const Pair p = pair_of(a, a.item_read[t0 + item], (uint32_t)a.cand_bin[a.item_pair[t0 + item]]);
    const uint2 sp = a.item_span[t0 + item];
    const uint32_t np = whole ? 1u : parts_of(sp, item);
    const TextPart text = text_part(p.lo, p.hi, sp.x, sp.y, np, u, p.L + (uint32_t)p.E);
    atomicMin(&best_of[item], (uint32_t)align_text<W>(a, p, text.lo, text.hi));
  }
  __syncthreads();
  for (uint32_t i = t; i < n; i += 256) {
    if (best_of[i] == 0xFFFFFFFFu) continue;
    const uint32_t r = a.item_read[t0 + i];
    const int64_t L = a.offsets[r + 1] - a.offsets[r];
    write_distance(a, a.item_pair[t0 + i], (int32_t)best_of[i], (L - (int64_t)a.q + 1 - (int64_t)a.thr[r]) / (int64_t)a.q);
  }
}

// The classes of reads of W0 .. W0 + 7 words in one launch: block[c] .. block[c + 1]
// are the workgroups of words W0 + 7 - c (the longest alignments start first).
struct LeftPlan {
  uint32_t block[9];
  uint32_t per;
  uint64_t first[8], count[8];
};

template <int W0>
__global__ __launch_bounds__(256) void k_verify_left(VerifyArgs a, LeftPlan plan) {
  __shared__ LeftLds lds;
  uint32_t c = 0;
  while (blockIdx.x >= plan.block[c + 1]) ++c;
  const uint64_t at = (uint64_t)(blockIdx.x - plan.block[c]) * plan.per, t0 = plan.first[c] + at;
  const uint32_t n = (uint32_t)min<uint64_t>(plan.per, plan.count[c] - at);
  switch (c) {
    case 0: left_items<W0 + 7>(a, t0, n, lds); break;
    case 1: left_items<W0 + 6>(a, t0, n, lds); break;
    case 2: left_items<W0 + 5>(a, t0, n, lds); break;
    case 3: left_items<W0 + 4>(a, t0, n, lds); break;
    case 4: left_items<W0 + 3>(a, t0, n, lds); break;
    case 5: left_items<W0 + 2>(a, t0, n, lds); break;
    case 6: left_items<W0 + 1>(a, t0, n, lds); break;
    default: left_items<W0>(a, t0, n, lds); break;
  }
}

template <int W0>
hipError_t launch_left(const VerifyArgs& a, const uint64_t* first, const uint64_t* count, hipStream_t s) {
  uint64_t total = 0, blocks = 0;
  for (int c = 0; c < 8; ++c) total += count[W0 + c];
  if (total == 0) return hipSuccess;
  LeftPlan plan;
  // part of the pairs are left after the sift, so a workgroup takes several for
  // each of its lanes, where that leaves some for every CU
  plan.per = (uint32_t)std::min<uint64_t>(kMostLeft, std::max<uint64_t>(256, total / kLeftBlocks));
  for (int c = 0; c < 8; ++c) {
    const int w = W0 + 7 - c;
    plan.block[c] = (uint32_t)blocks;
    plan.first[c] = first[w];
    plan.count[c] = count[w];
    blocks += (count[w] + plan.per - 1) / plan.per;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidConfiguration;
  }
  plan.block[8] = (uint32_t)blocks;
  hipLaunchKernelGGL((k_verify_left<W0>), dim3((unsigned)blocks), dim3(256), 0, s, a, plan);
  return hipGetLastError();
}

template <int W>
hipError_t launch_align_w(const VerifyArgs& a, uint64_t first, uint64_t count, hipStream_t s) {
  const uint64_t blocks = (count + 255) / 256;
  if (blocks > 0x7FFFFFFFull) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL((k_verify_align<W>), dim3((unsigned)blocks), dim3(256), 0, s, a, first, count);
  return hipGetLastError();
}

}  // namespace

// Reads per workgroup of the list passes: whole rounds of its 16 wavefronts, as
// few as keep the chunks, which one workgroup scans, within 2048. At a fixed
// 2048 reads, 20000 reads were listed by 10 workgroups (313 + 450 us).
uint32_t verify_chunk_reads(uint64_t n_reads) {
  return (uint32_t)std::max<uint64_t>(16, (n_reads + 2047) / 2048 + 15 & ~15ull);
}
uint64_t verify_chunks(uint64_t n_reads) {
  const uint64_t c = verify_chunk_reads(n_reads);
  return (n_reads + c - 1) / c;
}

hipError_t launch_verify_count(const VerifyArgs& a, hipStream_t s) {
  const uint64_t chunks = verify_chunks(a.n_reads);
  if (chunks == 0) return hipSuccess;
  if (chunks > 0x7FFFFFFFull) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL(k_verify_count, dim3((unsigned)chunks), dim3(1024), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_verify_prefix, dim3(a.bounded ? 2 : 1), dim3(1024), 0, s, a, chunks);
  return hipGetLastError();
}

hipError_t launch_verify_scatter(const VerifyArgs& a, hipStream_t s) {
  const uint64_t chunks = verify_chunks(a.n_reads);
  if (chunks == 0) return hipSuccess;
  hipLaunchKernelGGL(k_verify_scatter, dim3((unsigned)chunks), dim3(1024), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_verify_sift(const VerifyArgs& a, uint64_t count, hipStream_t s) {
  // one thread per item, and a launch holds fewer than 2^32 (GRIM_VERIFY_SLICE: fewer items, for tests)
  uint64_t most = 1ull << 31;
  if (const char* e = std::getenv("GRIM_VERIFY_SLICE")) most = std::min<uint64_t>(most, std::max(1ll, std::atoll(e)));
  for (uint64_t at = 0; at < count; at += most) {
    VerifyArgs b = a;
    b.item_pair += at;
    b.item_read += at;
    b.item_span += at;
    const uint64_t n = std::min(count - at, most);
    hipLaunchKernelGGL(k_verify_sift, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, b, n);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_verify_left(const VerifyArgs& a, const uint64_t* first, const uint64_t* count, hipStream_t s) {
  const hipError_t e = launch_left<1>(a, first, count, s);
  return e == hipSuccess ? launch_left<9>(a, first, count, s) : e;
}

hipError_t launch_verify_align(const VerifyArgs& a, uint32_t words, uint64_t first, uint64_t count,
                               hipStream_t s) {
  if (count == 0) return hipSuccess;
  switch (words) {
    case 1: return launch_align_w<1>(a, first, count, s);
    case 2: return launch_align_w<2>(a, first, count, s);
    case 3: return launch_align_w<3>(a, first, count, s);
    case 4: return launch_align_w<4>(a, first, count, s);
    case 5: return launch_align_w<5>(a, first, count, s);
    case 6: return launch_align_w<6>(a, first, count, s);
    case 7: return launch_align_w<7>(a, first, count, s);
    case 8: return launch_align_w<8>(a, first, count, s);
    case 9: return launch_align_w<9>(a, first, count, s);
    case 10: return launch_align_w<10>(a, first, count, s);
    case 11: return launch_align_w<11>(a, first, count, s);
    case 12: return launch_align_w<12>(a, first, count, s);
    case 13: return launch_align_w<13>(a, first, count, s);
    case 14: return launch_align_w<14>(a, first, count, s);
    case 15: return launch_align_w<15>(a, first, count, s);
    case 16: return launch_align_w<16>(a, first, count, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace grim
