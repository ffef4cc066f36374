// Piece starts from bitmaps of the window (Sec. 4.1: the run-local rules; Sec.
// 4.2 lists decode, classify, runs, predicate and scans as stages over
// characters).
//
// The block classifies its window and turns the classes into bitmaps: one bit
// per byte position, one bitmap per class, 64 words of 32 positions.  One wave
// then holds the whole window, a word per lane, and every rule is a few bitwise
// operations for all 2,048 positions at once: the class of the character before
// a position is the class bitmap shifted by one (classes spread over the
// continuation bytes of their characters first, when there are any), and a
// property of a whole run is carried along it by an integer addition over the
// bitmap, 64 lanes wide, with the carries between lanes resolved by one scalar
// addition.  The same wave numbers the units.
//
// GPT-2- and cl100k-style: evaluating the rules per character in every thread,
// with a block-wide segmented scan for cl100k, took 13.6 us of a tile in
// multilingual text (scan and carries 6.4, rules 7.2) and 5.3 us under GPT-2
// (with the wait for the slowest wave), most of it instruction issue by eight
// waves and up to nine block barriers; one wave and one barrier take 2.2 and
// 1.0 us.  Whole device-resident calls: 1M multilingual characters 66.1 -> 47.5
// us, 100K of code and prose 24.4 -> 18.6, a 16M corpus 351 -> 309 us.
// o200k- and DeepSeek-style: walking the alternatives piece by piece between
// synchronizing positions, one lane per stretch, took 17.6 and 15.0 us of a tile
// (46 and 32 in the slowest) and made tiles wait for the piece that enters
// them; the bitmaps take 3.1 and 2.4 us (8.4 and 3.4).  1M multilingual
// characters under o200k 82.4 -> 46.4 us, spans of 200K under DeepSeek, host to
// host, 113 -> 98 us.
#pragma once

#include "tt_bpe.h"
#include "tt_internal.h"

namespace tt {

// Bitmaps of the window; a position's bit k in its classification word is at
// 4 (k % 8) + (position & 3) (bitmaps 8 and up, which only the o200k- and
// DeepSeek-style patterns have, are in a second word).
enum { BM_L = 0, BM_N = 1, BM_O = 2, BM_WS = 3, BM_NL = 4, BM_SP = 5, BM_APO = 6, BM_CUT = 7 };
enum { BM2_U = 0, BM2_LO = 6, BM2_X = 8, BM2_M = 9, BM2_APO = 10, BM2_SLASH = 11 };   // o200k (with N, O, WS, NL, SP)
enum { BMD_AL = 0, BMD_L = 6, BMD_AP = 2, BMD_PS = 8, BMD_O = 9, BMD_KL = 10, BMD_KP = 11, BMD_KO = 12 };  // DeepSeek
constexpr int BM_STRIDE = 72;  // words between bitmaps: the 64 words a wave stores at once lie in 64 banks
constexpr int BM_WORDS = PT_WIN / 32;
static_assert(BM_WORDS == 64, "one word of a bitmap per lane");

// A lane holds bit 4 k + j for bitmap k and position 4 lane + j.  Returns, in
// the lane with number k in its group of eight, the group's 32 positions of
// bitmap k: a transposition of lane bits 2, 1, 0 with word bits 4, 3, 2.
__device__ __forceinline__ uint32_t to_bitmaps(uint32_t e, int lane) {
#define TT_DPP(x, ctrl) ((uint32_t)__builtin_amdgcn_update_dpp(0, (int)(x), ctrl, 0xF, 0xF, true))
  auto exchange = [](uint32_t x, uint32_t y, bool hi, uint32_t low, uint32_t s) -> uint32_t {
    const uint32_t keep = hi ? ~low : low;
    return (x & keep) | (__builtin_amdgcn_alignbit(y, y, hi ? s : 32u - s) & ~keep);
  };
  const uint32_t x7 = TT_DPP(e, 0x141);                                            // row_half_mirror: lane ^ 7
  e = exchange(e, TT_DPP(x7, 0x1B), (lane & 4) != 0, 0x0000FFFFu, 16u);            // quad_perm 3,2,1,0: lane ^ 4
  e = exchange(e, TT_DPP(e, 0x4E), (lane & 2) != 0, 0x00FF00FFu, 8u);              // quad_perm 2,3,0,1: lane ^ 2
  e = exchange(e, TT_DPP(e, 0xB1), (lane & 1) != 0, 0x0F0F0F0Fu, 4u);              // quad_perm 1,0,3,2: lane ^ 1
#undef TT_DPP
  return e;
}

// Four bits per lane, as one bitmap: the last lane of each group of eight
// stores the group's word (no atomics, and no clearing beforehand).
__device__ __forceinline__ void store_nibbles(uint32_t* words, int pos, int lane, uint32_t nib) {
  int x = (int)(nib << (pos & 31));
  x |= __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);  // row_shr:1
  x |= __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);  // row_shr:2
  x |= __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);  // row_shr:4
  if ((lane & 7) == 7) words[pos >> 5] = (uint32_t)x;
}

// ---- operations on bitmaps held one word per lane ---------------------------
// position q takes the bit of position q - 1 (q + 1); zero comes in at the ends
__device__ __forceinline__ uint32_t bm_shl1(uint32_t x) {
  const uint32_t p = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x138, 0xF, 0xF, true);  // wave_shr:1
  return __builtin_amdgcn_alignbit(x, p, 31);
}
__device__ __forceinline__ uint32_t bm_shr1(uint32_t x) {
  const uint32_t n = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x130, 0xF, 0xF, true);  // wave_shl:1
  return __builtin_amdgcn_alignbit(n, x, 1);
}
// The sum of two bitmaps as 2,048-bit integers: a lane's word generates a carry
// or passes one on, and adding the two lane masks resolves all of them.
__device__ __forceinline__ uint64_t bm_carries(uint64_t gen, uint64_t pass) { return ((gen << 1) + pass) ^ pass; }
__device__ __forceinline__ uint32_t bm_add(uint32_t a, uint32_t b) {
  const uint32_t s = a + b;
  const uint64_t c = bm_carries(__ballot(s < a), __ballot(s == 0xFFFFFFFFu));
  return s + (__builtin_amdgcn_inverse_ballot_w64(c) ? 1u : 0u);
}
// The same from the last position to the first.
__device__ __forceinline__ uint32_t bm_add_rev(uint32_t a, uint32_t b) {
  const uint32_t ra = __builtin_bitreverse32(a), s = ra + __builtin_bitreverse32(b);
  const uint64_t c = bm_carries(__builtin_bitreverse64(__ballot(s < ra)), __builtin_bitreverse64(__ballot(s == 0xFFFFFFFFu)));
  return __builtin_bitreverse32(s + (__builtin_amdgcn_inverse_ballot_w64(__builtin_bitreverse64(c)) ? 1u : 0u));
}
// Word `lane` of the bitmap of positions [lo, hi).
__device__ __forceinline__ uint32_t bm_range(int lo, int hi, int lane) {
  const int a = max(lo - 32 * lane, 0), b = min(hi - 32 * lane, 32);
  if (a >= b) return 0u;
  return (0xFFFFFFFFu << a) & (0xFFFFFFFFu >> (32 - b));
}
// The last set position of a bitmap, or -1 (the same in every lane).
__device__ __forceinline__ int bm_last(uint32_t x) {
  const uint64_t m = __ballot(x != 0u);
  if (m == 0ull) return -1;
  const int l = 63 - __builtin_clzll(m);
  return 32 * l + 31 - __builtin_clz((uint32_t)__builtin_amdgcn_readlane((int)x, l));
}
__device__ __forceinline__ bool bm_test(uint32_t x, int pos) {  // 0 <= pos < PT_WIN, wave-uniform
  return ((uint32_t)__builtin_amdgcn_readlane((int)x, pos >> 5) >> (pos & 31)) & 1u;
}

// A window's bitmaps in one wave.
struct RunBits {
  uint32_t L, N, O, WS, NL, SP, APO;  // first bytes of the characters of a class
  uint32_t D;                         // document starts
  uint32_t C;                         // first bytes of characters
  uint32_t K;                         // continuation bytes
  bool multi;                         // there are continuation bytes (wave-uniform)

  // the positions of a class's characters, continuation bytes included
  __device__ __forceinline__ uint32_t fill(uint32_t x) const {
    if (!multi) return x;
    const uint32_t a = bm_shl1(x) & K, b = bm_shl1(a) & K, c = bm_shl1(b) & K;
    return x | a | b | c;
  }
  // positions whose preceding character (in the same document) is in x (filled)
  __device__ __forceinline__ uint32_t after(uint32_t filled) const { return bm_shl1(filled) & ~D; }
  // first bytes whose following character (in the same document) is in x
  __device__ __forceinline__ uint32_t before(uint32_t x) const {
    uint32_t g = bm_shr1(x & ~D), r = g;
    if (multi) {
      g = bm_shr1(g & K);
      r |= g;
      g = bm_shr1(g & K);
      r |= g;
      g = bm_shr1(g & K);
      r |= g;
    }
    return r;
  }
};

// Strict UTF-8 decode from bytes in registers, with selects only: the length
// of the sequence that starts with b0 (0 if it is invalid or longer than
// `avail`) and its code point.
__device__ __forceinline__ uint32_t decode_sel(uint32_t b0, uint32_t b1, uint32_t b2, uint32_t b3, uint32_t avail,
                                               uint32_t& cp) {
  const uint32_t len = b0 < 0x80u ? 1u : b0 < 0xC2u ? 0u : b0 < 0xE0u ? 2u : b0 < 0xF0u ? 3u : b0 < 0xF5u ? 4u : 0u;
  const uint32_t lo = b0 == 0xE0u ? 0xA0u : b0 == 0xF0u ? 0x90u : 0x80u;
  const uint32_t hi = b0 == 0xEDu ? 0x9Fu : b0 == 0xF4u ? 0x8Fu : 0xBFu;
  const bool ok1 = len < 2u || (b1 >= lo && b1 <= hi);
  const bool ok2 = len < 3u || (b2 & 0xC0u) == 0x80u;
  const bool ok3 = len < 4u || (b3 & 0xC0u) == 0x80u;
  const uint32_t c2 = ((b0 & 0x1Fu) << 6) | (b1 & 0x3Fu);
  const uint32_t c3 = ((b0 & 0x0Fu) << 12) | ((b1 & 0x3Fu) << 6) | (b2 & 0x3Fu);
  const uint32_t c4 = ((b0 & 0x07u) << 18) | ((b1 & 0x3Fu) << 12) | ((b2 & 0x3Fu) << 6) | (b3 & 0x3Fu);
  cp = len <= 1u ? b0 : len == 2u ? c2 : len == 3u ? c3 : c4;
  return (len != 0u && len <= avail && ok1 && ok2 && ok3) ? len : 0u;
}

// The first of the characters text[0, end) whose class `in` does not hold: its
// class, or ~0 when there is none, or invalid input (reported elsewhere) before
// it.  ASCII bytes for which plain() holds are in the set.  text may begin inside
// a character, which is left out.  One wave, 16 bytes per lane per step; every
// lane has the same answer.
// A step first looks for bytes that are not plain, and only when there are some
// decodes the characters that begin in each lane's bytes.  (Decoding one character
// per step instead took 97 ms for 100 KB of U+3000 after a line break and 109 ms
// for 100 KB of Cyrillic capitals; now 0.65 and 0.94 ms.)
template <class Plain, class In, class ClassOf>
__device__ __forceinline__ uint32_t first_outside(const uint8_t* text, uint32_t end, int lane, Plain plain, In in,
                                                  ClassOf class_of) {
#pragma unroll 1
  for (uint32_t pos = 0;; pos += 16u * 64u) {
    const uint32_t p0 = pos + 16u * (uint32_t)lane;
    uint32_t k = 16u;
#pragma unroll 4
    for (int i = 15; i >= 0; --i) {
      const uint32_t p = p0 + (uint32_t)i;
      if (!(p < end && plain((uint32_t)text[p]))) k = (uint32_t)i;  // (the end counts as a stop)
    }
    if (__ballot(k < 16u) == 0ull) continue;
    uint32_t c = ~0u;
    bool stop = false;
#pragma unroll 1
    while (k < 16u) {
      const uint32_t p = p0 + k;
      const uint32_t avail = p < end ? min(end - p, 4u) : 0u;
      auto at = [&](uint32_t i) -> uint32_t { return i < avail ? (uint32_t)text[p + i] : 0u; };
      const uint32_t b0 = at(0);
      ++k;
      if (avail != 0u && (b0 & 0xC0u) == 0x80u) continue;  // (of a character that begins before)
      uint32_t cp = 0;
      const uint32_t len = decode_sel(b0, at(1), at(2), at(3), avail, cp);
      c = len != 0u ? class_of(cp) : ~0u;
      stop = len == 0u || !in(c);
      if (stop) break;
      k += len - 1u;
    }
    const uint64_t m = __ballot(stop);
    if (m != 0ull) return (uint32_t)__builtin_amdgcn_readlane((int)c, __builtin_ctzll(m));
  }
}

// The suffix of a contraction whose apostrophe is at window position a: its
// bytes (1 or 2, 0 for none).  GPT-2: lower-case; else folded, and U+017F
// counts as s.
template <int PAT>
__device__ __forceinline__ uint32_t suffix_bytes(const uint8_t* buf, const uint8_t* dstart, int a) {
  const uint8_t* p = buf + PT_PAD + a + 1;  // (staged up to 16 bytes past the window)
  uint32_t c1 = p[0], c2 = p[1], len = 0;
  const bool split = dstart != nullptr && dstart[PT_PAD + a + 2] != 0;  // (a document starts at c2)
  if (PAT != TT_PATTERN_GPT2) {
    if (c1 == 0xC5u && c2 == 0xBFu) len = 2;  // U+017F
    c1 |= 0x20u;
    c2 |= 0x20u;
  }
  if (c1 == 's' || c1 == 't' || c1 == 'm' || c1 == 'd') len = 1;
  if (!split && ((c2 == 'e' && (c1 == 'r' || c1 == 'v')) || (c1 == 'l' && c2 == 'l'))) len = 2;
  return len;
}

// Contractions: an apostrophe that no symbol and no U+0020 precedes begins one
// when a suffix letter (or two) follows.  No piece starts at the suffix, and
// one starts after it when the letters go on.  `starts` is edited in place.
template <int PAT>
__device__ __forceinline__ void contractions(const RunBits& b, uint32_t pO, uint32_t pSP, const uint8_t* buf,
                                             const uint8_t* dstart, int lane, uint32_t& starts) {
  const uint32_t letter = b.L & ~b.D;
  uint32_t cand = b.APO & ~pO & ~pSP & bm_shr1(letter);
  if (__ballot(cand != 0u) == 0ull) return;
  uint64_t clear = 0, set = 0;  // this lane's positions, and spilling into the next lane's
  while (cand) {
    const int a = __builtin_ctz(cand);
    cand &= cand - 1u;
    const uint32_t len = suffix_bytes<PAT>(buf, dstart, 32 * lane + a);
    if (len) {
      clear |= 2ull << a;
      set |= 2ull << (a + (int)len);
    }
  }
  auto spread = [&](uint64_t x) -> uint32_t {
    return (uint32_t)x | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), 0x138, 0xF, 0xF, true);
  };
  starts = (starts & ~spread(clear)) | (spread(set) & letter);
}

// GPT-2-style piece starts (valid at the tile's own positions).
__device__ __forceinline__ uint32_t gpt2_starts(const RunBits& b, const uint8_t* buf, const uint8_t* dstart, int lane) {
  const uint32_t pW = b.after(b.fill(b.WS) | b.NL), pL = b.after(b.fill(b.L)), pN = b.after(b.fill(b.N)),
                 pO = b.after(b.fill(b.O)), pSP = b.after(b.SP);
  const uint32_t solid = b.L | b.N | b.O;
  // whitespace: the head of its run, and its last character before something else;
  // other runs: the head, unless U+0020 (which then starts the piece) precedes
  uint32_t st = ((b.WS | b.NL) & (~pW | b.before(solid))) | (((b.L & ~pL) | (b.N & ~pN) | (b.O & ~pO)) & ~pSP);
  contractions<TT_PATTERN_GPT2>(b, pO, pSP, buf, dstart, lane, st);
  return st;
}

// ---- what runs carry from tile to tile --------------------------------------
// Every tile publishes what the text up to its last byte would bring into the
// next one; a later tile asks only when the 32 bytes of its context do not tell
// and its own rules depend on it.
//   number runs: the characters of the trailing run in the tile, mod 3 (bits 1..2);
//   tail: cl100k- and DeepSeek-style, a symbol precedes the trailing CR/LF run
//     (bit 3);
//   state (bits 4..7): o200k-style, what the last character is part of (below);
//     DeepSeek-style, ST_LOW when trailing ASCII letters belong to the symbol
//     before them.
// Bits 8..10: the tile adds nothing of its own to number, tail, state (one run
// covers it): ask the tile before.
enum : uint32_t { SUM_TAIL = 8u, SUM_N_ALL = 256u, SUM_TAIL_ALL = 512u, SUM_STATE_ALL = 1024u };
constexpr int SUM_STATE_SHIFT = 4;
// What the last character of a tile is part of (o200k-style).
enum : uint32_t {
  ST_NONE = 0,   // nothing that reaches on: whitespace, a number, CR/LF of no tail
  ST_UP = 1,     // letters, none of them lower-case since the piece's start
  ST_LOW = 2,    // letters, with a lower-case one
  ST_LONE = 3,   // a symbol that starts a piece
  ST_RUN = 4,    // a symbol run
  ST_TAIL = 5,   // the CR/LF and slashes after a symbol run
  ST_SUFFIX = 6  // a contraction that ends with the tile (7, 8: one or two bytes after it)
};
struct RunCarry {
  uint32_t n;
  bool tail;
  uint32_t state;
};
static_assert(PT_HALO == 32, "the context before the tile is one bitmap word");

// Whether lane 0 (the context before the tile) has every bit set.
__device__ __forceinline__ bool covers_context(uint32_t x) { return (__ballot(x == 0xFFFFFFFFu) & 1ull) != 0ull; }
// Whether every character of the tile is in x.
__device__ __forceinline__ bool covers_tile(const RunBits& b, uint32_t own, uint32_t x) {
  return __ballot((b.C & own & ~x) != 0u) == 0ull;
}
// In lane 0, the bytes before the window's first character: the end of a character
// that begins outside, whose class is not in the bitmaps.
__device__ __forceinline__ uint32_t cut_bytes(const RunBits& b, int lane) {
  return lane == 0 ? (b.C & (0u - b.C)) - 1u : 0u;
}
// Bits of m reached from the bits of s by runs of m, towards later positions
// (s within m; several bits of s may lie in one run).
__device__ __forceinline__ uint32_t bm_flood(uint32_t m, uint32_t s) { return ((bm_add(m, s) ^ m) | s) & m; }

// Number runs: what the tile publishes, and the starts of the groups of three.
struct NumberRuns {
  uint32_t heads;   // first characters of number runs
  uint32_t breaks;  // characters that begin or end one
};
__device__ __forceinline__ NumberRuns number_runs(const RunBits& b, bool first_tile, int lane) {
  NumberRuns r;
  r.heads = b.N & ~b.after(b.fill(b.N));
  // (what precedes the window's first character is not known)
  if (!first_tile && lane == 0) r.heads &= ~(b.C & (0u - b.C)) | b.D;
  r.breaks = (b.C & ~b.N) | r.heads;
  return r;
}
__device__ __forceinline__ bool number_enters(const RunBits& b, const NumberRuns& r) {
  return (__ballot(b.N != 0u && r.breaks == 0u) & 1ull) != 0ull;
}
__device__ __forceinline__ uint32_t number_summary(const RunBits& b, const NumberRuns& r, uint32_t own, int lane) {
  const int h = bm_last(r.breaks & own);
  const uint32_t c = (uint32_t)__popc(b.N & own & bm_range(max(h, 0), PT_WIN, lane));
  const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_sum(c), 63);
  return (h < 0 ? SUM_N_ALL : 0u) | ((total % 3u) << 1);
}

// CR/LF runs: whether the trailing one is a symbol piece's tail.
__device__ __forceinline__ uint32_t nl_summary(const RunBits& b, uint32_t own, uint32_t nl_heads, uint32_t sym) {
  const int last = bm_last(b.C & own);
  if (last < 0) return SUM_TAIL_ALL;
  if (!bm_test(b.NL, last)) return 0u;
  const int h = bm_last(nl_heads & own);  // (the last head of a CR/LF run is the trailing run's)
  if (max(h, bm_last(b.C & ~b.NL & own)) < 0) return SUM_TAIL_ALL;
  return h >= 0 && bm_test(sym, h) ? SUM_TAIL : 0u;
}

// Starts of the groups of three inside number runs: `off` characters of the
// run lie before this lane's word.
__device__ __forceinline__ uint32_t number_starts(uint32_t N, uint32_t heads, uint32_t off) {
  uint32_t st = 0, x = N;
  while (x) {
    const uint32_t a = (uint32_t)__builtin_ctz(x);
    if ((heads >> a) & 1u) off = 0;
    // the one-byte characters from a on, up to the next run (a longer
    // character ends the stretch; the count goes on after it)
    const uint32_t stop = (~x | (heads & ~(1u << a))) >> a;
    const uint32_t s = stop ? (uint32_t)__builtin_ctz(stop) : 32u - a;
    const uint32_t seg = (0xFFFFFFFFu >> (32u - s)) << a;
    st |= ((0x49249249u << (off ? 3u - off : 0u)) << a) & seg;
    const uint32_t t = off + s;
    off = t - 3u * ((t * 43u) >> 7);  // mod 3 (t < 35)
    x &= ~seg;
  }
  return st;
}

__device__ __forceinline__ uint32_t number_part(const RunBits& b, const NumberRuns& r, uint32_t entering, int lane) {
  if (__ballot(b.N != 0u) == 0ull) return 0u;
  // characters of the trailing number run of every word, summed over words
  // that one run covers (top bit: something else is in the word)
  constexpr uint32_t RESET = 0x80000000u;
  const uint32_t br = r.breaks ? 31u - (uint32_t)__builtin_clz(r.breaks) : 0u;
  uint32_t v = r.breaks ? (RESET | (uint32_t)__popc(b.N >> br)) : (uint32_t)__popc(b.N);
  if (lane == 0 && r.breaks == 0u) v = RESET | entering;
  auto comb = [](uint32_t p, uint32_t c) -> uint32_t { return (c & RESET) ? c : p + c; };
#define TT_COMB(ctrl, rows) v = comb((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xF, true), v)
  TT_COMB(0x111, 0xF);  // row_shr:1, 2, 4, 8
  TT_COMB(0x112, 0xF);
  TT_COMB(0x114, 0xF);
  TT_COMB(0x118, 0xF);
  TT_COMB(0x142, 0xA);  // row_bcast:15 into rows 1, 3
  TT_COMB(0x143, 0xC);  // row_bcast:31 into rows 2, 3
#undef TT_COMB
  const uint32_t before = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xF, 0xF, true) & ~RESET;
  return number_starts(b.N, r.heads, before % 3u);
}

// Whitespace as cl100k, o200k and the last DeepSeek splitter have it
// (\s*[\r\n]+, \s+(?!\S), \s+), where `sym` are the positions after a symbol
// character and `tail` those after the CR/LF (or slash) tail of a symbol
// piece; `solid` is what the lookahead stops at.  beyond() tells whether the
// whitespace stretch that reaches the window's end is the last of its run.
template <class Beyond>
__device__ __forceinline__ uint32_t whitespace_starts(const RunBits& b, uint32_t solid, uint32_t sym, uint32_t tail,
                                                      int lane, Beyond beyond) {
  const uint32_t WSf = b.fill(b.WS);
  const uint32_t pWS = b.after(WSf), pNL = b.after(b.NL), pW = pWS | pNL;
  uint32_t st = (b.WS & ~pW) | (b.NL & ~pW & ~sym) | (b.WS & pWS & b.before(solid));
  // the first whitespace after a CR/LF run: it starts a piece when the run is a
  // symbol piece's tail or when no CR/LF follows its stretch
  const uint32_t x = b.WS & pNL;
  if (__ballot(x != 0u) != 0ull) {
    const uint32_t ws = WSf & ~b.D;
    const uint32_t sum = bm_add(ws, x);
    const uint32_t end_nl = sum & ~ws & b.NL & ~b.D;              // CR/LF right after such a stretch
    const uint32_t more = ws & ~bm_add_rev(ws, bm_shr1(end_nl));  // the stretches before those
    uint32_t ok = ~more | tail;
    if (bm_test(ws & ~sum, PT_WIN - 1)) {  // a stretch reaches the window's end
      const int q = bm_last(x);
      if (q < PT_HALO + PT_OWN && !bm_test(tail, q) && !beyond()) ok &= ~bm_range(q, q + 1, lane);
    }
    st |= x & ok;
  }
  return st;
}

// cl100k-style piece starts (valid at the tile's own positions).  publish(sum)
// is called with the tile's summary before carry(), which waits for earlier
// tiles; last_ws() is whitespace_starts' beyond().
template <class Pub, class Carry, class LastWs>
__device__ __forceinline__ uint32_t cl100k_starts(const RunBits& b, uint32_t own, const uint8_t* buf,
                                                  const uint8_t* dstart, int lane, bool first_tile, Pub publish,
                                                  Carry carry, LastWs last_ws) {
  const uint32_t pL = b.after(b.fill(b.L)), pO = b.after(b.fill(b.O)), pSP = b.after(b.SP);
  const uint32_t nl_heads = b.NL & ~b.after(b.NL), nl = b.NL & ~b.D;
  uint32_t sym = nl & pO;  // heads of CR/LF runs that a symbol precedes
  const NumberRuns nr = number_runs(b, first_tile, lane);
  publish(number_summary(b, nr, own, lane) | nl_summary(b, own, nl_heads, sym));
  RunCarry in{};
  const uint32_t cut0 = cut_bytes(b, lane);
  const bool nl_in = !first_tile && covers_context(b.NL | cut0);
  if (!first_tile && (nl_in || number_enters(b, nr))) in = carry(nl_in ? SUM_TAIL_ALL : SUM_N_ALL);
  if (nl_in && in.tail && lane == 0) sym |= nl & (cut0 + 1u);
  uint32_t st = whitespace_starts(b, b.L | b.N | b.O, pO, b.after(bm_flood(nl, sym)), lane, last_ws);
  st |= number_part(b, nr, in.n, lane);
  // symbols; letters, which take one preceding whitespace character but CR/LF,
  // or a symbol that neither a symbol nor U+0020 precedes
  const uint32_t z = b.fill(b.O & (pO | pSP));
  st |= (b.O & ~pO & ~pSP) | (b.L & ~pL & ~b.after(b.fill(b.WS)) & (~pO | b.after(z)));
  contractions<TT_PATTERN_CL100K>(b, pO, pSP, buf, dstart, lane, st);
  return st;
}

// ---- o200k-style -------------------------------------------------------------
//   P1  [^\r\n\p{L}\p{N}]? [Lu Lt Lm Lo M]* [Ll Lm Lo M]+ CT?
//   P2  [^\r\n\p{L}\p{N}]? [Lu Lt Lm Lo M]+ [Ll Lm Lo M]* CT?
//   P3  \p{N}{1,3}      P4  U+0020? [^\s\p{L}\p{N}]+ [\r\n/]*
//   P5  \s*[\r\n]+     P6  \s+(?!\S)     P7  \s+
// U: Lu, Lt; Lo: Ll; X: Lm, Lo; M: marks.  The rules, from the alternatives:
//   - A mark is symbol material inside a symbol run that already holds two
//     symbols side by side or begins after U+0020 (a lone symbol before a mark
//     is P1's first character), else a letter that, like X, is in both sets.
//   - Inside a run of letters a piece is [U X]* [Ll X]+: a U starts a piece when
//     a Ll, or X's that follow one, precede it.  A run that ends in U's with no
//     Ll after the piece's start ends the piece after its last X (P1 gives the
//     U's back), so the U's after that X start a piece when what follows them is
//     no letter.
//   - A contraction after a letter belongs to its piece; the next character
//     starts a piece.  In a row of them ('s's's) every second one is a letter
//     behind its own apostrophe.
//   - A symbol piece takes the CR/LF after it and then CR/LF and slashes.
//   - Everything else as in cl100k.
// tests/test_run_rules.py compares the whole set with a matcher that tries the
// alternatives, on all strings of up to four of 15 characters of every class and
// on random longer ones, in tiles of this size and of 32 to 96 bytes.
//
// The context tells the state at the tile's first byte when a character in it
// resets the rules whatever precedes it (`reset` below), or when it is one run
// of X's, which only matters to a U right after them.  Else (a context of
// nothing but marks, slashes, CR/LF or a row of contractions) the state that
// the tile before publishes takes the place of the context: one character of a
// class that stands for it, or a piece start.
struct O2Maps {
  uint32_t U, Lo, X, M, APO, SLASH;
};
// upper_then_letter() tells whether a letter follows the run of U's that reaches
// the window's end.
template <class Pub, class Carry, class LastWs, class Upper>
__device__ __forceinline__ uint32_t o200k_starts(RunBits b, O2Maps m, uint32_t own, const uint8_t* buf,
                                                 const uint8_t* dstart, int lane, bool first_tile, Pub publish,
                                                 Carry carry, LastWs last_ws, Upper upper_then_letter) {
  const NumberRuns nr = number_runs(b, first_tile, lane);
  const uint32_t tile_chars = b.C & own;
  RunCarry in{};
  bool in_tail = false;  // the context is the tail of a symbol piece
  const uint32_t cut0 = cut_bytes(b, lane);
  const bool x_in = !first_tile && covers_context((b.fill(m.X) & ~b.D) | cut0);
  if (!first_tile && !x_in) {
    const uint32_t let = m.U | m.Lo | m.X, apo2 = bm_shl1(bm_shl1(m.APO)), o = b.O & ~m.SLASH;
    const uint32_t reset = b.N | b.WS | b.D | ((m.U | m.Lo) & b.after(b.fill(let)) & ~apo2 & ~bm_shl1(apo2)) |
                           (b.O & ~m.APO & b.after(b.fill(let))) | (o & b.after(b.fill(o)));
    // (the neighbours of the first eight positions may lie outside)
    if ((__ballot((reset & 0xFFFFFF00u) != 0u) & 1ull) == 0ull) {
      in = carry(SUM_STATE_ALL | SUM_N_ALL);
      const bool both = bm_last(b.C & bm_range(0, PT_HALO, lane)) == bm_last((m.X | m.M) & bm_range(0, PT_HALO, lane));
      const uint32_t k = in.state > ST_SUFFIX ? in.state - ST_SUFFIX : 0u;  // bytes of a suffix in this tile
      const uint32_t keep = lane == 0 ? 0u : lane == 1 ? ~((1u << k) - 1u) : ~0u;
      const uint32_t top = lane == 0 ? 0x80000000u : 0u;
      m.U = (m.U & keep) | (in.state == ST_UP && !both ? top : 0u);
      m.Lo = (m.Lo & keep) | (in.state == ST_LOW ? top : 0u);
      m.X = (m.X & keep) | (in.state == ST_UP && both ? top : 0u);
      m.M &= keep;
      m.APO &= keep;
      m.SLASH &= keep;
      b.O = (b.O & keep) | (in.state == ST_LONE ? top : in.state == ST_RUN ? top | (top >> 1) : 0u);
      b.NL = (b.NL & keep) | (in.state == ST_TAIL || in.state == ST_NONE ? top : 0u);
      b.WS &= keep;
      b.SP &= keep;
      b.D = (b.D & (lane == 0 ? 0u : ~0u)) | (in.state >= ST_SUFFIX && lane == 1 ? 1u << k : 0u);
      in_tail = in.state == ST_TAIL;
    }
  }
  const uint32_t pSP = b.after(b.SP);
  const uint32_t ts = (b.NL | m.SLASH) & ~b.D;  // what a symbol piece's tail can hold after its first CR/LF
  const bool marks = __ballot(m.M != 0u) != 0ull;
  // Symbols, without the slashes that a tail takes; each pass settles at least
  // one more slash, and text without a slash in a tail takes one pass.
  uint32_t taken = 0, X = m.X, S = b.O, tail;
  for (;;) {
    const uint32_t o = b.O & ~taken;
    S = o;
    if (marks) {
      const uint32_t om = (b.fill(o) | b.fill(m.M)) & ~b.D;
      const uint32_t in_run = bm_flood(om, o & (b.after(b.fill(o)) | pSP) & om);
      X = m.X | (m.M & ~in_run);
      S |= m.M & in_run;
    }
    uint32_t s = ts & b.NL & b.after(b.fill(S));
    if (in_tail && lane == 0) s |= ts;
    tail = bm_flood(ts, s);
    const uint32_t next = m.SLASH & tail;
    if (__ballot(next != taken) == 0ull) break;
    taken = next;
  }
  // contractions after letters
  const uint32_t letters0 = m.U | m.Lo | X;
  uint32_t v1 = 0, v2 = 0;  // apostrophes of suffixes of one byte, and of two
  {
    uint32_t cand = m.APO & b.after(b.fill(letters0)) & bm_shr1((m.U | m.Lo) & ~b.D);
    while (cand) {
      const int a = __builtin_ctz(cand);
      cand &= cand - 1u;
      const uint32_t len = suffix_bytes<TT_PATTERN_O200K>(buf, dstart, 32 * lane + a);
      if (len == 1u) v1 |= 1u << a;
      if (len == 2u) v2 |= 1u << a;
    }
  }
  uint32_t ct_end = 0, ct = 0;  // first positions after contractions; their bytes
  const uint32_t v = v1 | v2;
  if (__ballot(v != 0u) != 0ull) {
    auto end_of = [&](uint32_t x) -> uint32_t { return bm_shl1(bm_shl1((x & v1) | bm_shl1(x & v2))); };
    // of apostrophes right after another's suffix, every second one
    uint32_t take = v & ~end_of(v), cur = take;
    for (;;) {
      cur = end_of(end_of(cur) & v) & v;
      if (__ballot(cur != 0u) == 0ull) break;
      take |= cur;
    }
    ct_end = end_of(take);
    ct = take | bm_shl1(take | bm_shl1(take & v2));
  }
  const uint32_t U = m.U & ~ct, Lo = m.Lo & ~ct, let = letters0 & ~ct;
  X &= ~ct;
  S &= ~ct;
  // the state of a run of X's: whether a Ll precedes it
  const uint32_t Xf = b.fill(X), Xr = Xf & ~b.D, Lof = b.fill(Lo);
  uint32_t low = bm_flood(Xr, X & b.after(Lof) & Xr);
  const uint32_t run0 = x_in ? bm_flood(Xr, lane == 0 ? Xr & (cut0 + 1u) : 0u) : 0u;  // the run that enters the window
  const uint32_t pO = b.after(b.fill(S));
  const uint32_t z = S & (pO | pSP);  // symbols inside a run
  {
    const int last = bm_last(tile_chars);
    uint32_t state = ST_NONE;
    if (last >= 0) {
      if (bm_test(let, last)) state = bm_test(Lo | low, last) ? ST_LOW : ST_UP;
      if (bm_test(S, last)) state = bm_test(z, last) ? ST_RUN : ST_LONE;
      if (bm_test(tail, last)) state = ST_TAIL;
    }
    for (uint32_t k = 0; k < 3u; ++k)
      if (bm_test(ct_end, PT_HALO + PT_OWN + (int)k)) state = ST_SUFFIX + k;
    const bool all = x_in && __ballot((tile_chars & ~run0) != 0u) == 0ull;
    publish(number_summary(b, nr, own, lane) | (state << SUM_STATE_SHIFT) | (all ? SUM_STATE_ALL : 0u));
  }
  const bool x_asks = x_in && __ballot((U & b.after(run0) & own) != 0u) != 0ull;
  if (!first_tile && (x_asks || number_enters(b, nr))) in = carry((x_asks ? SUM_STATE_ALL : 0u) | SUM_N_ALL);
  if (x_asks && in.state == ST_LOW) low |= run0;

  uint32_t st = U & b.after(Lof | low);
  const uint32_t h2 = U & ~b.after(b.fill(U)) & b.after(Xf & ~low);
  if (__ballot(h2 != 0u) != 0ull) {
    const uint32_t Uf = b.fill(U) & ~b.D;
    const uint32_t sum = bm_add(Uf, h2 & Uf);
    const uint32_t then = sum & ~Uf & let & ~b.D;  // a letter right after such a run
    uint32_t more = Uf & ~bm_add_rev(Uf, bm_shr1(then));
    if (bm_test(Uf & ~sum, PT_WIN - 1)) {
      const int q = bm_last(h2);
      if (q < PT_HALO + PT_OWN && upper_then_letter()) more |= bm_range(q, q + 1, lane);
    }
    st |= h2 & ~more;
  }
  st |= let & ~b.after(b.fill(let)) & ~b.after(b.fill(b.WS)) & (~pO | b.after(b.fill(z)));
  st |= whitespace_starts(b, m.U | m.Lo | m.X | m.M | b.O | b.N, pO, b.after(tail), lane, last_ws);
  st |= number_part(b, nr, in.n, lane);
  st |= S & ~pO & ~pSP;
  return st & ~tail;
}

// ---- DeepSeek-style ------------------------------------------------------------
//   S1  \p{N}{1,3}      S2  runs of U+4E00-9FA5, U+3040-309F, U+30A0-30FF
//   S3  D1 [ASCII punctuation][A-Za-z]+   D2 [^\r\n\p{L}\p{P}\p{S}]?[\p{L}\p{M}]+
//       D3 U+0020? [\p{P}\p{S}]+ [\r\n]*   D4 \s*[\r\n]+   D5 \s+(?!\S)   D6 \s+
// Numbers, the CJK/kana set and the rest are stretches of their own, so the
// rules never look at a class of another stretch (it counts as the end of the
// text).  In the rest (AL: ASCII letters, L: other letters and marks, AP and PS:
// ASCII and other punctuation and symbols, O: none of the classes):
//   - D1 joins ASCII letters to a lone AP (not after a symbol or U+0020); another
//     letter after them starts a piece;
//   - a letter run otherwise takes one whitespace character but CR/LF, or one O,
//     before it; of a run of O's only the last is taken;
//   - symbols as in cl100k, whitespace as in cl100k.
// In the CJK/kana set letters and marks, symbols, and the others form runs, of
// the others again the last joins letters.  Compared in the same way with the
// splitters applied in sequence.
struct DsMaps {
  uint32_t AL, L, AP, PS, O, KL, KP, KO;
};
template <class Pub, class Carry, class LastWs>
__device__ __forceinline__ uint32_t deepseek_starts(const RunBits& b, const DsMaps& m, uint32_t own, int lane,
                                                    bool first_tile, Pub publish, Carry carry, LastWs last_ws) {
  const uint32_t P = m.AP | m.PS, let = m.AL | m.L;
  const uint32_t pSP = b.after(b.SP), pP = b.after(b.fill(P));
  const uint32_t nl_heads = b.NL & ~b.after(b.NL), nl = b.NL & ~b.D;
  uint32_t sym = nl & pP;
  const NumberRuns nr = number_runs(b, first_tile, lane);
  // (whether a symbol that is the window's first character is a lone one is not
  // known: the context of such a symbol and ASCII letters tells no more than one
  // of letters alone)
  const uint32_t first = !first_tile && lane == 0 ? b.C & (0u - b.C) : 0u, edge = m.AP & first & ~b.D;
  const uint32_t join = m.AL & b.after(m.AP & ~pP & ~pSP & ~edge), al = m.AL & ~b.D;
  uint32_t d1 = bm_flood(al, join);  // ASCII letters behind a lone symbol
  const bool al_in = !first_tile && covers_context(al | (edge ? edge | (edge - 1u) : 0u));
  const uint32_t run0 = al_in ? bm_flood(al, lane == 0 ? al & (0u - al) : 0u) : 0u;
  {
    const int last = bm_last(b.C & own);
    uint32_t sum = number_summary(b, nr, own, lane) | nl_summary(b, own, nl_heads, sym);
    if (last >= 0 && bm_test(d1, last)) sum |= ST_LOW << SUM_STATE_SHIFT;
    if (al_in && covers_tile(b, own, al)) sum |= SUM_STATE_ALL;
    publish(sum);
  }
  RunCarry in{};
  const uint32_t cut0 = cut_bytes(b, lane);
  const bool nl_in = !first_tile && covers_context(b.NL | cut0);
  const bool al_asks = al_in && __ballot((m.L & b.after(run0) & own) != 0u) != 0ull;
  if (!first_tile && (nl_in || al_asks || number_enters(b, nr)))
    in = carry((nl_in ? SUM_TAIL_ALL : 0u) | (al_asks ? SUM_STATE_ALL : 0u) | SUM_N_ALL);
  if (nl_in && in.tail && lane == 0) sym |= nl & (cut0 + 1u);
  if (al_asks && in.state == ST_LOW) d1 |= run0;
  const uint32_t pO = b.after(b.fill(m.O)), pWS = b.after(b.fill(b.WS));
  uint32_t st = (let & ~b.after(b.fill(let)) & ~pWS & ~pO & ~join) | (m.L & b.after(d1));
  st |= (m.O & (~pO | b.before(let))) | (P & ~pP & ~pSP);
  const uint32_t pKO = b.after(b.fill(m.KO));
  st |= (m.KL & ~b.after(b.fill(m.KL)) & ~pKO) | (m.KP & ~b.after(b.fill(m.KP))) | (m.KO & (~pKO | b.before(m.KL)));
  st |= whitespace_starts(b, let | P | m.O, pP, b.after(bm_flood(nl, sym)), lane, last_ws);
  return st | number_part(b, nr, in.n, lane);
}

}  // namespace tt
