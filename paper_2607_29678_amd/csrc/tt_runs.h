// Piece starts of the GPT-2- and cl100k-style patterns from bitmaps of the
// window (Sec. 4.1: the run-local rules; Sec. 4.2 lists decode, classify, runs,
// predicate and scans as stages over characters).
//
// The block classifies its window and turns the classes into bitmaps: one bit
// per byte position, one bitmap per class, 64 words of 32 positions.  One wave
// then holds the whole window, a word per lane, and every rule is a few bitwise
// operations for all 2,048 positions at once: the class of the character before
// a position is the class bitmap shifted by one (classes spread over the
// continuation bytes of their characters first, when there are any), and a
// property of a whole run is carried along it by an integer addition over the
// bitmap, 64 lanes wide, with the carries between lanes resolved by one scalar
// addition.  The same wave numbers the units.  Evaluating the rules per
// character in every thread, with a block-wide segmented scan for cl100k, took
// 13.6 us of a tile in multilingual text (scan and carries 6.4, rules 7.2) and
// 5.3 us under GPT-2 (with the wait for the slowest wave), most of it
// instruction issue by eight waves and up to nine block barriers; one wave and
// one barrier take 2.2 and 1.0 us.  Whole device-resident calls: 1M
// multilingual characters 66.1 -> 47.5 us, 100K of code and prose 24.4 -> 18.6,
// a 16M corpus 351 -> 309 us.
#pragma once

#include "tt_bpe.h"
#include "tt_internal.h"

namespace tt {

// Bitmaps of the window; a position's bit k in its classification word is at
// 4 k + (position & 3).
enum { BM_L = 0, BM_N = 1, BM_O = 2, BM_WS = 3, BM_NL = 4, BM_SP = 5, BM_APO = 6, BM_CUT = 7, BM_COUNT = 8 };
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

// Contractions: an apostrophe that no symbol and no U+0020 precedes begins one
// when a suffix letter (or two) follows.  No piece starts at the suffix, and
// one starts after it when the letters go on.  `starts` is edited in place.
// GPT-2: lower-case suffixes; cl100k: folded, and U+017F counts as s.
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
    const uint8_t* p = buf + PT_PAD + 32 * lane + a + 1;  // (staged up to 16 bytes past the window)
    uint32_t c1 = p[0], c2 = p[1];
    uint32_t len = 0;
    const bool split = dstart != nullptr && dstart[PT_PAD + 32 * lane + a + 2] != 0;  // (a document starts at c2)
    if (PAT == TT_PATTERN_CL100K) {
      if (c1 == 0xC5u && c2 == 0xBFu) len = 2;  // U+017F
      c1 |= 0x20u;
      c2 |= 0x20u;
    }
    if (c1 == 's' || c1 == 't' || c1 == 'm' || c1 == 'd') len = 1;
    if (!split && ((c2 == 'e' && (c1 == 'r' || c1 == 'v')) || (c1 == 'l' && c2 == 'l'))) len = 2;
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

// trailing-run summary of a tile (cl100k): bit 0 the run spans the whole tile,
// bits 1..2 the number characters of the run mod 3, bit 3 a symbol precedes it
constexpr uint32_t SUM_RUNALL = 1u;
// What runs that enter the window from before it bring along: the length of a
// number run mod 3 at the tile's first byte, and whether a symbol precedes a
// CR/LF run.
struct RunCarry {
  uint32_t n;
  bool sym;
};

// A tile's summary, from its own positions (`own`): only number and CR/LF runs
// are ever asked for.
__device__ __forceinline__ uint32_t cl100k_summary(const RunBits& b, uint32_t own, uint32_t n_heads,
                                                   uint32_t nl_heads, uint32_t nl_sym) {
  const int last = bm_last(b.C & own);
  if (last < 0) return SUM_RUNALL;
  if (bm_test(b.N, last)) {
    const int h = bm_last(((b.C & ~b.N) | n_heads) & own);
    const int lane = (int)(threadIdx.x & 63u);
    const uint32_t c = (uint32_t)__popc(b.N & own & bm_range(max(h, 0), PT_WIN, lane));
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_sum(c), 63);
    return (h < 0 ? SUM_RUNALL : 0u) | ((total % 3u) << 1);
  }
  if (bm_test(b.NL, last)) {
    const int h = bm_last(nl_heads & own);  // (the last head of a CR/LF run is the trailing run's)
    const int other = bm_last(b.C & ~b.NL & own);
    if (max(h, other) < 0) return SUM_RUNALL;
    return h >= 0 && bm_test(nl_sym, h) ? 8u : 0u;
  }
  return 0u;
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

// cl100k-style piece starts (valid at the tile's own positions).  publish(sum)
// is called with the tile's summary before carry(), which waits for earlier
// tiles and is called only when a number or CR/LF run spans all the context
// before the tile; beyond() tells whether the whitespace stretch that reaches
// the window's end is the last of its whitespace run.
template <class Pub, class Carry, class Beyond>
__device__ __forceinline__ uint32_t cl100k_starts(const RunBits& b, uint32_t own, const uint8_t* buf,
                                                  const uint8_t* dstart, int lane, bool first_tile, Pub publish,
                                                  Carry carry, Beyond beyond) {
  const uint32_t WSf = b.fill(b.WS);
  const uint32_t pWS = b.after(WSf), pNL = b.after(b.NL), pL = b.after(b.fill(b.L)), pN = b.after(b.fill(b.N)),
                 pO = b.after(b.fill(b.O)), pSP = b.after(b.SP);
  const uint32_t pW = pWS | pNL;
  uint32_t n_heads = b.N & ~pN;
  const uint32_t nl_heads = b.NL & ~pNL;
  // (what precedes the window's first character is not known)
  if (!first_tile && lane == 0) n_heads &= ~(b.C & (0u - b.C)) | b.D;
  uint32_t nl_sym = b.NL & pO;  // heads of CR/LF runs that a symbol precedes
  publish(cl100k_summary(b, own, n_heads, nl_heads, nl_sym));
  // a run that covers the 32 bytes before the tile (lane 0's word)
  const uint32_t n_breaks = (b.C & ~b.N) | n_heads;
  static_assert(PT_HALO == 32, "the context before the tile is one bitmap word");
  RunCarry in{0u, false};
  const uint64_t l0_n = __ballot(b.N != 0u && n_breaks == 0u), l0_nl = __ballot(b.NL == 0xFFFFFFFFu);
  if (!first_tile && ((l0_n | l0_nl) & 1ull)) in = carry();
  if (in.sym && (l0_nl & 1ull) && lane == 0) nl_sym |= 1u;

  // whitespace
  const uint32_t solid = b.L | b.N | b.O;
  uint32_t st = (b.WS & ~pW) | (b.NL & ~pW & ~pO) | (b.WS & pWS & b.before(solid));
  // the first whitespace after a CR/LF run: it starts a piece when a symbol
  // precedes the run (whose piece takes the CR/LF) or when no CR/LF follows
  // its stretch
  const uint32_t x = b.WS & pNL;
  if (__ballot(x != 0u) != 0ull) {
    const uint32_t nl = b.NL & ~b.D;
    const uint32_t s = nl_sym & nl;
    const uint32_t sym_run = nl & ~bm_add(nl, s);  // CR/LF runs that a symbol precedes
    const uint32_t ws = WSf & ~b.D;
    const uint32_t sum = bm_add(ws, x);
    const uint32_t end_nl = sum & ~ws & b.NL & ~b.D;          // CR/LF right after such a stretch
    const uint32_t more = ws & ~bm_add_rev(ws, bm_shr1(end_nl));  // the stretches before those
    uint32_t ok = ~more | b.after(sym_run);
    if (bm_test(ws & ~sum, PT_WIN - 1)) {  // a stretch reaches the window's end
      const int q = bm_last(x);
      if (!bm_test(b.after(sym_run), q) && !beyond()) ok &= ~bm_range(q, q + 1, lane);
    }
    st |= x & ok;
  }
  // numbers in threes from the head of their run
  if (__ballot(b.N != 0u) != 0ull) {
    // characters of the trailing number run of every word, summed over words
    // that one run covers (top bit: something else is in the word)
    constexpr uint32_t RESET = 0x80000000u;
    const uint32_t br = n_breaks ? 31u - (uint32_t)__builtin_clz(n_breaks) : 0u;
    uint32_t v = n_breaks ? (RESET | (uint32_t)__popc(b.N >> br)) : (uint32_t)__popc(b.N);
    if (lane == 0 && n_breaks == 0u) v = RESET | in.n;
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
    st |= number_starts(b.N, n_heads, before % 3u);
  }
  // symbols; letters, which take one preceding whitespace character but CR/LF,
  // or a symbol that neither a symbol nor U+0020 precedes
  const uint32_t z = b.fill(b.O & (pO | pSP));
  st |= (b.O & ~pO & ~pSP) | (b.L & ~pL & ~pWS & (~pO | b.after(z)));
  contractions<TT_PATTERN_CL100K>(b, pO, pSP, buf, dstart, lane, st);
  return st;
}

}  // namespace tt
