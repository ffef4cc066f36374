// The tile kernel: one block decides the pieces of 1,984 bytes of the request
// and encodes them, with no host round trip and no kernel boundary between
// pre-tokenization and BPE.
//
// Pre-tokenization.  The paper replaces the sequential leftmost-first regex
// scan by an equivalent per-character predicate: classify every character
// into letter / number / whitespace / other, form maximal same-class runs,
// and decide whether a character starts a piece from its offset in its run,
// at most four characters of lookback and a few per-run aggregates (Sec. 4.1,
// "Removing the sequential regex scan"; Sec. 4.2 lists the stages: decode,
// classify, runs, predicate, scans).  A block stages a 2,048-byte window (32
// bytes of context on each side of the bytes it owns) in LDS, every thread
// decodes and classifies four positions, and one wave evaluates the rules of
// the pattern on bitmaps of the window (tt_runs.h).
// Runs that reach past the window are resolved without a second pass:
//   - backwards from summaries that earlier blocks publish;
//   - forwards by reading the bytes after the window, which only a whitespace
//     stretch or a run of capitals that reaches its end may need.
//
// Units.  For encoding, a piece is also cut at every byte position whose byte
// pair (b[q-1], b[q]) is the junction of no merge: the first merge that joins
// across a position has its left operand ending in b[q-1] and its right one
// starting with b[q], so no merge ever crosses such a position and the two
// sides are independent BPE problems.
//
// BPE (Sec. 4.2, "GPU BPE").  The block encodes every unit that starts in its
// bytes except its last one, whose end lies in a later tile: that unit is the
// "incoming" unit of the next tile that has a unit start, which learns its
// start from the position the earlier tiles publish right after their scan.
// Units go to the smallest execution unit that holds them (part of a wave, a
// wave, or the whole block over rows in LDS or, past the window size, global
// memory), and the tile's tokens go to their place after a look-back over the
// counts of earlier tiles.
//
// Block order is taken from an atomic ticket, so a block only ever waits on
// blocks that started before it.  What a block publishes before it waits on
// anything, later blocks get at once; the rest (counts of all tiles up to this
// one, and o200k-style summaries of tiles whose own context does not tell) only
// ever depends on earlier tiles.
#include "class_table.inc"
#include "class_table_o200k.inc"
#include "class_table_deepseek.inc"
#include "tt_bpe.h"
#include "tt_internal.h"
#include "tt_deepseek.h"
#include "tt_o200k.h"
#include "tt_runs.h"

namespace tt {

namespace {

// Words published for later blocks are self-contained values (the consumer
// reads nothing else the producer wrote), so relaxed device-scope atomics are
// enough: they are coherent across the chip without ordering other accesses.
__device__ __forceinline__ uint64_t ld_word(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_word(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// One lane waits for a word tagged with the call's epoch in its high half,
// sleeping between polls so that the wave does not flood the cache with loads.
__device__ __forceinline__ uint64_t wait_word(const uint64_t* p, uint32_t epoch) {
  uint64_t x = ld_word(p);
  while ((uint32_t)(x >> 32) != epoch) {
    __builtin_amdgcn_s_sleep(1);
    x = ld_word(p);
  }
  return x;
}

constexpr int CLS_L1_BYTES = 4352, CLS_L2_BYTES = TT_CLS_NBLOCKS * 64;

// The probed class table, staged in LDS by every block, and the bitmap bits of
// every ASCII character (built by the block).
struct ClassLds {
  uint8_t l1[CLS_L1_BYTES] __attribute__((aligned(16)));
  uint8_t l2[CLS_L2_BYTES] __attribute__((aligned(16)));
  uint32_t asc[128];
};

// The 4-bit class table of the o200k- and DeepSeek-style patterns (same layout,
// room for the larger), staged in LDS by every block, and the bitmap bits of
// every ASCII character and of every class.
constexpr int O2_NBLOCKS = TT_O2_NBLOCKS > TT_DS_NBLOCKS ? TT_O2_NBLOCKS : TT_DS_NBLOCKS;
struct O2Lds {
  uint8_t l1[4352] __attribute__((aligned(16)));
  uint8_t l2[O2_NBLOCKS * 128] __attribute__((aligned(16)));
  uint2 asc[128];
  uint2 cls[16];
};

// 2-bit class of a non-ASCII code point from the probed table.
__device__ __forceinline__ uint32_t table_class(const ClassLds& ct, uint32_t cp) {
  const uint32_t blk = ct.l1[cp >> 8];
  const uint32_t b = ct.l2[blk * 64u + ((cp & 255u) >> 2)];
  return (b >> ((cp & 3u) * 2u)) & 3u;
}

// Class of an ASCII code point for the o200k-style pattern.
__device__ __forceinline__ uint32_t o2_ascii_class(uint32_t cp) {
  if ((cp - 'A') < 26u) return O2_UP;
  if ((cp - 'a') < 26u) return O2_LO;
  if ((cp - '0') < 10u) return O2_N;
  if (cp == 10u || cp == 13u) return O2_NL;
  if (cp == 32u || (cp - 9u) < 5u) return O2_WS;
  return O2_O;
}
// Bitmap bits (tt_runs.h) of a class of the o200k- and DeepSeek-style patterns,
// and of an ASCII character.
__device__ __forceinline__ uint2 bit_of(int k) {
  return k < 8 ? make_uint2(1u << (4 * k), 0u) : make_uint2(0u, 1u << (4 * (k - 8)));
}
template <int PAT>
__device__ __forceinline__ uint2 o2_class_bits(uint32_t c) {
  if (PAT == TT_PATTERN_O200K) {
    switch (c) {
      case O2_UP: return bit_of(BM2_U);
      case O2_LO: return bit_of(BM2_LO);
      case O2_BO: return bit_of(BM2_X);
      case O2_MK: return bit_of(BM2_M);
      case O2_N: return bit_of(BM_N);
      case O2_WS: return bit_of(BM_WS);
      case O2_NL: return bit_of(BM_NL);
      case O2_O: return bit_of(BM_O);
    }
    return make_uint2(0u, 0u);
  }
  switch (c) {
    case DS_AL: return bit_of(BMD_AL);
    case DS_L:
    case DS_M: return bit_of(BMD_L);
    case DS_N: return bit_of(BM_N);
    case DS_AP: return bit_of(BMD_AP);
    case DS_PS: return bit_of(BMD_PS);
    case DS_SP:
    case DS_WS: return bit_of(BM_WS);
    case DS_NL: return bit_of(BM_NL);
    case DS_KL:
    case DS_KM: return bit_of(BMD_KL);
    case DS_KP: return bit_of(BMD_KP);
    case DS_KO: return bit_of(BMD_KO);
    case DS_O: return bit_of(BMD_O);
  }
  return make_uint2(0u, 0u);
}
template <int PAT>
__device__ __forceinline__ uint2 o2_ascii_bits(uint32_t cp) {
  uint2 e = o2_class_bits<PAT>(PAT == TT_PATTERN_O200K ? o2_ascii_class(cp) : ds_ascii_class(cp));
  if (cp == 32u) e.x |= bit_of(BM_SP).x;
  if (PAT == TT_PATTERN_O200K && cp == 39u) e.y |= bit_of(BM2_APO).y;
  if (PAT == TT_PATTERN_O200K && cp == 47u) e.y |= bit_of(BM2_SLASH).y;
  return e;
}

// Bitmap bits (tt_runs.h) of an ASCII character, and of a character of a class
// of the probed table.
__device__ __forceinline__ uint32_t ascii_bits(uint32_t cp) {
  if (((cp | 32u) - 'a') < 26u) return 1u << (4 * BM_L);
  if ((cp - '0') < 10u) return 1u << (4 * BM_N);
  if (cp == 10u || cp == 13u) return 1u << (4 * BM_NL);
  if (cp == 32u) return (1u << (4 * BM_WS)) | (1u << (4 * BM_SP));
  if ((cp - 9u) < 5u) return 1u << (4 * BM_WS);
  if (cp == 39u) return (1u << (4 * BM_O)) | (1u << (4 * BM_APO));
  return 1u << (4 * BM_O);
}
__device__ __forceinline__ uint32_t class_bits(uint32_t cls2) {  // 0 other, 1 letter, 2 number, 3 whitespace
  constexpr uint32_t AT = (4u * BM_O) | (4u * BM_L) << 8 | (4u * BM_N) << 16 | (4u * BM_WS) << 24;
  return 1u << ((AT >> (8u * cls2)) & 31u);
}

template <typename F>
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v, int lane, F comb) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    uint32_t o = __shfl_up(v, d, 64);
    if (lane >= d) v = comb(o, v);
  }
  return v;
}


// The NW little-endian words of the L bytes at window index a (bytes past L
// read as zero), from aligned LDS words: NW + 1 word loads and one byte
// alignment per word.  Reads window bytes [a & ~3, a + 4 NW + 4).
template <int NW>
__device__ __forceinline__ void unit_words(const uint8_t* buf, uint32_t a, uint32_t L, uint32_t (&w)[NW]) {
  const uint32_t p = PT_PAD + a;
  const uint32_t* d = reinterpret_cast<const uint32_t*>(buf + (p & ~3u));
  const uint32_t sh = p & 3u;
  uint32_t x[NW + 1];
#pragma unroll
  for (int i = 0; i <= NW; ++i) x[i] = d[i];
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const uint32_t v = __builtin_amdgcn_alignbyte(x[i + 1], x[i], sh);
    const int rem = (int)L - 4 * i;  // bytes of word i inside the unit
    w[i] = rem >= 4 ? v : rem <= 0 ? 0u : (v & ((1u << (8 * rem)) - 1u));
  }
}

// ignore_merges: the internal ID of the vocabulary string equal to the L
// bytes byte(0 .. L) (2 <= L), or DICT_NONE.  Strings of up to DICT2_MAX bytes
// are probed with their bytes as the key (from the window when aw >= 0, i.e.
// the bytes start at window index aw); longer ones by two hashes of their
// bytes, confirmed by comparing the bytes with the stored string.
template <class ByteF>
__device__ uint32_t piece_find(const DevTables& tb, const uint8_t* buf, int64_t aw, uint32_t L, ByteF byte) {
  if (L <= (uint32_t)DICT2_MAX) {
    uint32_t kw[6] = {0u, 0u, 0u, 0u, 0u, 0u};
    if (aw >= 0 && aw + DICT2_MAX + 4 <= PT_WIN + 16) {
      unit_words(buf, (uint32_t)aw, L, kw);
    } else {
      for (uint32_t j = 0; j < L; ++j) kw[j >> 2] |= byte(j) << (8 * (j & 3));
    }
    if (L <= (uint32_t)DICT_MAX) return dict_find(tb.vdict, tb.vdnb, kw[0], kw[1], kw[2], L);
    return dict2_find(tb.vdict2, tb.vdnb2, kw, L);
  }
  uint32_t h1 = LONG_SEED1, h2 = LONG_SEED2;
  for (uint32_t j = 0; j < L; ++j) {
    const uint32_t b = byte(j);
    h1 = long_hash_step(h1, b);
    h2 = long_hash_step(h2, b);
  }
  h1 = long_hash_final(h1, L);
  h2 = long_hash_final(h2, L);
  const uint32_t b1 = 2u * bucket_of(h1, tb.vlnb), b2 = 2u * bucket_of(h2, tb.vlnb);
  const u32x4 e[4] = {tb.vlong[b1], tb.vlong[b1 + 1], tb.vlong[b2], tb.vlong[b2 + 1]};
  for (int i = 0; i < 4; ++i) {
    if (e[i].x != h1 || e[i].y != L) continue;
    bool same = true;
    for (uint32_t j = 0; j < L && same; ++j) same = tb.vblob[e[i].w + j] == byte(j);
    if (same) return e[i].z;
  }
  return DICT_NONE;
}

constexpr int SMALL_CAP = PT_OWN / 3 + 2;              // units of 3..SMALL_MAX bytes in a tile (the incoming one too)
constexpr int MED_CAP = PT_WIN / (SMALL_MAX + 1) + 2;  // units of 17..WAVE_MAX bytes in a tile
// wave units are taken longest first, in classes of 8 bytes
constexpr int MED_CLASSES = (WAVE_MAX - SMALL_MAX + 7) / 8;
static_assert(SMALL_MAX < 64 && MED_CLASSES <= 64, "the start of each length (class) is one wave scan");
__device__ __forceinline__ uint32_t med_class(uint32_t L) { return (uint32_t)(WAVE_MAX - L) >> 3; }
constexpr int BIG_CAP = PT_WIN / (WAVE_MAX + 1) + 2;   // longer units in a tile
constexpr uint16_t U_INCOMING = 0xFFFFu;               // list entry for the incoming unit

// LDS of the classification phase and of the BPE phase share one region:
// nothing of the first is read after the unit scan, nothing of the second is
// written before it.
template <bool WIDE>
struct RulesMem;
template <>
struct RulesMem<false> {    // GPT-2, cl100k
  ClassLds cls;             // character classes
  uint32_t join[2048];      // junction byte pairs of the merges
  uint32_t bm[8 * BM_STRIDE];   // bitmaps of the window
  uint32_t bm_doc[BM_WORDS];    // batch: document starts
  uint32_t nocut[PT_WIN / 32];  // ignore_merges: window positions no junction cut may split
};
template <>
struct RulesMem<true> {     // o200k, DeepSeek
  O2Lds cls;
  uint32_t join[2048];
  uint32_t bm[16 * BM_STRIDE];
  uint32_t bm_doc[BM_WORDS];
  uint32_t nocut[PT_WIN / 32];
};
template <bool WIDE>
union PhaseMem {
  RulesMem<WIDE> a;
  struct {
    uint32_t tok[PT_WIN];     // tokens of unit k at tok[ustart[k] ..]
    uint16_t uoff[PT_WIN];    // first output of each unit within the tile
    uint16_t small[SMALL_CAP];  // units of 3..16 bytes, sorted by length
    union {
      uint32_t wscr[PT_THREADS / 64][256];  // wave engine for 65..128 bytes: one area per wave
      struct {                              // block engine for 129..ROWS_LDS bytes
        uint64_t tok[2 * ROWS_LDS];
        uint64_t sel[ROWS_LDS / 64 + 2];
      } rows;
    } x;
  } b;
  struct {                    // the tile's own outputs, in order
    uint32_t id[PT_WIN];      // (over tok[]: written after it is read)
    uint32_t span[PT_WIN];    // span export: byte start in the window | byte length << 16
  } c;
};

template <bool WIDE>
struct PtShared {
  uint8_t buf[PT_PAD + PT_WIN + 16] __attribute__((aligned(16)));     // window bytes
  uint8_t dstart[PT_PAD + PT_WIN + 16] __attribute__((aligned(16)));  // 1 where a document starts
  PhaseMem<WIDE> ph;
  uint16_t ustart[PT_OWN + 2];  // window index of every unit start in the owned bytes
  uint16_t ucnt[PT_OWN + 2];    // tokens of each unit
  RowsShared<PT_THREADS / 64> rows;
  uint16_t med[MED_CAP];
  uint16_t big[BIG_CAP];
  uint32_t hist[SMALL_MAX + 1];  // small units per length, then where each length starts
  uint32_t hmed[MED_CLASSES];    // wave units per length class, then where each class starts
  uint32_t n_small, n_med, n_big;
  uint32_t pass_next;            // next pass of the wave engines to take (in steps of 64)
  uint32_t wave_tot[PT_THREADS / 64];
  uint32_t tile;
  uint32_t s_prev;            // start of the incoming unit
  uint32_t prefix;            // outputs of all earlier tiles
  uint32_t err;               // invalid input in this tile or an earlier one
  uint32_t inc_cnt;           // its tokens
  uint32_t uw[BM_WORDS], upre[BM_WORDS];  // unit starts, and those before each word
  uint32_t m;                 // their number
  uint32_t cwave[PT_THREADS / 64];  // span export: per-wave sums
  uint32_t whole[PT_WIN / 32];  // ignore_merges: starts of pieces that are vocabulary entries
  uint32_t ncw[BM_WORDS], ncpre[BM_WORDS];  // span export: non-continuation bytes, and those before each word
  uint32_t cbase;             // span export: non-continuation bytes before the tile
  uint32_t ctile;             // span export: non-continuation bytes the tile owns
};

}  // namespace

// A token's span as one store (the caller's array is aligned to its int32
// elements only).
typedef int Span __attribute__((ext_vector_type(4), aligned(4)));

// Word a tile publishes for the placement of its outputs:
//   bits 0..30 a count, bit 31 set when the count is inclusive (all outputs of
//   the tiles up to this one) rather than this tile's own, bit 32 set when
//   invalid input was seen (inclusive: in any tile up to this one), bits 33..63
//   the epoch of the call.
constexpr uint64_t PL_INC = 1ull << 31, PL_ERR = 1ull << 32;
constexpr int PL_EPOCH_SHIFT = 33;

// Decoupled look-back (one wave): the sum of the counts of the tiles before tile t,
// newest first, until one whose published count is already inclusive.  A window of 64
// earlier tiles is read at once and read again until every tile the sum needs has
// published (earlier tiles publish their own count before they look back, so
// the walk never waits on a tile that is itself waiting).
__device__ __forceinline__ uint32_t lookback_counts(uint64_t* words, uint32_t t, uint64_t ep, uint32_t epoch,
                                                    int lane) {
  uint32_t prefix = 0;
  int64_t base = (int64_t)t - 1;
  for (;;) {
    const int64_t j = base - lane;
    uint64_t x = ep | PL_INC;  // before the first tile: an inclusive zero
    if (j >= 0) x = ld_word(&words[j]);
    const bool ready = (x >> PL_EPOCH_SHIFT) == (uint64_t)epoch;
    const uint64_t m_inc = __ballot(ready && (x & PL_INC));
    const uint64_t m_rdy = __ballot(ready);
    const int first = m_inc ? __ffsll((unsigned long long)m_inc) - 1 : 63;
    const uint64_t need = first >= 63 ? ~0ull : ((2ull << first) - 1ull);
    if ((m_rdy & need) != need) {
      __builtin_amdgcn_s_sleep(1);
      continue;
    }
    const uint32_t c = lane <= first ? (uint32_t)(x & 0x7FFFFFFFull) : 0u;
    prefix += (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_sum(c), 63);
    if (m_inc) break;
    base -= 64;
  }
  return prefix;
}

// The tile's own count, published as soon as it is known (one thread).
__device__ __forceinline__ void publish_count(const Work& w, uint32_t t, uint32_t count, bool bad) {
  const uint64_t ep = (uint64_t)w.epoch << PL_EPOCH_SHIFT;
  st_word(&w.tile_agg[t], ep | (t == 0 ? PL_INC : 0ull) | (bad ? PL_ERR : 0ull) | count);
}

// The place of the tile's outputs (wave 0; the tile's own count is published before):
// the number of outputs before this tile, in every thread.  The last tile also writes
// the output length, or the error.  (The look-back is lookback_counts' with the error
// flags; as one function for both, a 16M-character corpus took 0.4% longer.)
//
// With span export (cagg != nullptr), wave 1 runs the same look-back over the
// tiles' non-continuation byte counts at the same time; each tile published
// its own count early, so this walk rarely waits.  The sum before the tile
// ends in sh.cbase.
template <class Sh>
__device__ uint32_t place_tile(const Work& w, Sh& sh, uint32_t t, uint32_t count, bool bad, int tid, int lane,
                               int wave, uint64_t* cagg = nullptr, uint32_t c_tile = 0) {
  const uint64_t ep = (uint64_t)w.epoch << PL_EPOCH_SHIFT;
  if (cagg != nullptr) {
    if (t == 0) {
      if (tid == 0) {
        st_word(&cagg[0], ep | PL_INC | c_tile);
        sh.cbase = 0;
      }
    } else if (wave == 1) {
      const uint32_t cpre = lookback_counts(cagg, t, ep, w.epoch, lane);
      if (lane == 0) {
        st_word(&cagg[t], ep | PL_INC | (cpre + c_tile));
        sh.cbase = cpre;
      }
    }
  }
  uint64_t* pl = w.tile_agg;
  if (t == 0) {
    if (tid == 0) {
      sh.prefix = 0;
      sh.err = bad ? 1u : 0u;
    }
  } else if (wave == 0) {
    uint32_t prefix = 0;
    bool err = bad;
    int64_t base = (int64_t)t - 1;
    for (;;) {
      const int64_t j = base - lane;
      uint64_t x = ep | PL_INC;  // before the first tile: an inclusive zero
      if (j >= 0) x = ld_word(&pl[j]);
      const bool ready = (x >> PL_EPOCH_SHIFT) == (uint64_t)w.epoch;
      const uint64_t m_inc = __ballot(ready && (x & PL_INC));
      const uint64_t m_rdy = __ballot(ready);
      const int first = m_inc ? __ffsll((unsigned long long)m_inc) - 1 : 63;
      const uint64_t need = first >= 63 ? ~0ull : ((2ull << first) - 1ull);
      if ((m_rdy & need) != need) {
        __builtin_amdgcn_s_sleep(1);
        continue;
      }
      const bool use = lane <= first;
      const uint32_t c = use ? (uint32_t)(x & 0x7FFFFFFFull) : 0u;
      prefix += (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_sum(c), 63);
      err = err || __ballot(use && (x & PL_ERR)) != 0ull;
      if (m_inc) break;
      base -= 64;
    }
    if (lane == 0) {
      st_word(&pl[t], ep | PL_INC | (err ? PL_ERR : 0ull) | (prefix + count));
      sh.prefix = prefix;
      sh.err = err ? 1u : 0u;
    }
  }
  __syncthreads();
  if (tid == 0) {
    if (t == w.n_tiles - 1) *w.out_len = sh.err ? (int64_t)TT_ERR_INVALID_UTF8 : (int64_t)(sh.prefix + count);
  }
  return sh.prefix;
}

// Phase stamps (a diagnostic build of the library, compiled with
// TT_PHASE_STAMPS; the product build has none of this): thread 0 of every tile
// writes the 100 MHz wall clock at each phase boundary into tt_phase_buf, slot
// k of the tile's TT_PHASE_SLOTS, and tt_phase_stamps copies them to the host.
// Slots: 0 entry, 1 ticket and tables, 2 window staged, 3 classified, 4 (span
// export) character counts published, 5 piece and unit starts known, 6 dispatch
// done, 7 wave engines done, 8 block engine done, 9 placement look-back done, 10
// tokens written; inside the dispatch 11 units numbered, 12 unit starts listed,
// 13 incoming unit found and dictionaries probed, 14 length lists built; 20 the
// incoming unit's start known (by the thread that dispatches it); inside the
// starts 21 the rules done, 22 the vocabulary probes of ignore_merges done; 23
// the block index; 24 + w: wave w done with the starts (the same point as 5, per
// wave); 15 where the block runs (XCD in the high word, the hardware ID register
// in the low word).
#ifdef TT_PHASE_STAMPS
constexpr int TT_PHASE_SLOTS = 32, TT_PHASE_TILES = 8192;
__device__ unsigned long long tt_phase_buf[TT_PHASE_TILES * TT_PHASE_SLOTS];
#define TT_PHASE_BY(k, who)                                                                    \
  do {                                                                                         \
    if ((who) && t < (uint32_t)TT_PHASE_TILES) tt_phase_buf[(size_t)t * TT_PHASE_SLOTS + (k)] = wall_clock64(); \
  } while (0)
#else
#define TT_PHASE_BY(k, who) \
  do {                      \
  } while (0)
#endif
#define TT_PHASE(k) TT_PHASE_BY(k, tid == 0)

// The kernel's one argument; tile_args() reads it again from where the launch put
// it, for a rare phase: it then adds nothing to what the phases around it hold in
// scalar registers.
struct TileArgs {
  Work w;
  DevTables tb;
};
__device__ __forceinline__ const TileArgs& tile_args() {
  auto p = (const __attribute__((address_space(4))) TileArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  asm("" : "+s"(p));  // (not merged with earlier reads)
  return *(const TileArgs*)p;
}

// MODE 0: split-level export; the outputs are the byte offsets of the pieces.
// MODE 1: encoding; the outputs are the (internal) IDs of the units' tokens.
// MODE 2: encoding with span export: also the byte and character span of every
//         token (Appendix, Route C; the records of Definition d:records).
// WAVES:  wavefronts per SIMD the registers are allotted for: 6 (three blocks on
//         a compute unit) or 8 (four; launch_pat says when).
template <int PAT, bool BATCH, int MODE, bool IGN, int WAVES>
__global__ __launch_bounds__(PT_THREADS) __attribute__((amdgpu_waves_per_eu(WAVES))) void tile_kernel(TileArgs args) {
  const Work& w = args.w;
  const DevTables& tb = args.tb;
  constexpr bool SEG = MODE >= 1;
  constexpr bool SPANS = MODE == 2;
  constexpr bool DS = PAT == TT_PATTERN_DEEPSEEK;
  constexpr bool WIDE = PAT == TT_PATTERN_O200K || DS;  // 4-bit classes, up to 16 bitmaps
  __shared__ PtShared<WIDE> sh;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int64_t n = w.n;
#ifdef TT_PHASE_STAMPS
  const unsigned long long phase_s0 = wall_clock64();
#endif

  if (tid <= SMALL_MAX) sh.hist[tid] = 0;
  if (tid >= 64 && tid < 64 + MED_CLASSES) sh.hmed[tid - 64] = 0;
  if (IGN && tid < PT_WIN / 32) {
    sh.ph.a.nocut[tid] = 0;
    sh.whole[tid] = 0;
  }
  // the ticket's round trip (tickets are handed out one at a time) overlaps
  // the staging of the tables, which do not depend on the tile
  uint32_t ticket = 0;
  if (tid == 0) ticket = atomicAdd(&w.ctrl->tile_ticket, 1u);
  {
    // the class table (12.9 KB) is read once per block
    static_assert(CLS_L1_BYTES % 16 == 0 && CLS_L2_BYTES % 16 == 0, "class table staging uses 16-byte words");
    if constexpr (WIDE) {
      constexpr int N1 = 4352 / 16, N2 = (DS ? TT_DS_NBLOCKS : TT_O2_NBLOCKS) * 128 / 16;
      const uint4* s1 = reinterpret_cast<const uint4*>(DS ? TT_DS_L1 : TT_O2_L1);
      const uint4* s2 = reinterpret_cast<const uint4*>(DS ? TT_DS_L2 : TT_O2_L2);
      uint4* d1 = reinterpret_cast<uint4*>(sh.ph.a.cls.l1);
      uint4* d2 = reinterpret_cast<uint4*>(sh.ph.a.cls.l2);
      for (int i = tid; i < N1 + N2; i += PT_THREADS) {
        if (i < N1) d1[i] = s1[i];
        else d2[i - N1] = s2[i - N1];
      }
      if (tid < 128) sh.ph.a.cls.asc[tid] = o2_ascii_bits<PAT>((uint32_t)tid);
      if (tid >= 128 && tid < 144) sh.ph.a.cls.cls[tid - 128] = o2_class_bits<PAT>((uint32_t)(tid - 128));
    } else {
      constexpr int N1 = CLS_L1_BYTES / 16, N2 = CLS_L2_BYTES / 16;
      const uint4* s1 = reinterpret_cast<const uint4*>(TT_CLS_L1);
      const uint4* s2 = reinterpret_cast<const uint4*>(TT_CLS_L2);
      uint4* d1 = reinterpret_cast<uint4*>(sh.ph.a.cls.l1);
      uint4* d2 = reinterpret_cast<uint4*>(sh.ph.a.cls.l2);
      for (int i = tid; i < N1 + N2; i += PT_THREADS) {
        if (i < N1) d1[i] = s1[i];
        else d2[i - N1] = s2[i - N1];
      }
      if (tid < 128) sh.ph.a.cls.asc[tid] = ascii_bits((uint32_t)tid);
    }
  }
  if (SEG) {
    // the junction bitmap (8 KB) is read once per block
    const uint4* src = reinterpret_cast<const uint4*>(tb.join);
    uint4* dst = reinterpret_cast<uint4*>(sh.ph.a.join);
    for (int i = tid; i < 512; i += PT_THREADS) dst[i] = src[i];
  }
  if (tid == 0) {
    sh.tile = ticket - w.ticket_base;
    sh.n_med = 0;
    sh.pass_next = 0;
    sh.n_big = 0;
    sh.inc_cnt = 0;
  }
  __syncthreads();
  const uint32_t t = wave_uniform(sh.tile);
  const uint32_t n_tiles = w.n_tiles;
  if (t >= n_tiles) return;
#ifdef TT_PHASE_STAMPS
  if (tid == 0 && t < (uint32_t)TT_PHASE_TILES) {
    tt_phase_buf[(size_t)t * TT_PHASE_SLOTS] = phase_s0;
    tt_phase_buf[(size_t)t * TT_PHASE_SLOTS + 20] = 0;  // (written later only by a tile with an incoming unit)
    tt_phase_buf[(size_t)t * TT_PHASE_SLOTS + 23] = blockIdx.x;
    // where the block runs: the XCD (XCC_ID register) and the hardware ID
    // register (compute unit, shader array and engine in bits 8-15)
    const uint32_t xcc = (uint32_t)__builtin_amdgcn_s_getreg((3 << 11) | 20) & 15u;
    const uint32_t hw = (uint32_t)__builtin_amdgcn_s_getreg((31 << 11) | 4);
    tt_phase_buf[(size_t)t * TT_PHASE_SLOTS + 15] = ((unsigned long long)xcc << 32) | hw;
  }
#endif
  TT_PHASE(1);
  const int64_t t0 = (int64_t)t * PT_OWN;
  const int64_t w0 = t0 - PT_HALO;

  auto inside = [&](int q) -> bool {
    int64_t p = w0 + q;
    return p >= 0 && p < n;
  };

  // ---- stage the window: 8 bytes per thread, one 64-bit load when possible --
  // LDS index of window position q is q + PT_PAD, for q in [-PT_PAD, PT_WIN + 16)
  auto stage_chunk = [&](int c) {  // window bytes [8c, 8c + 8)
    const int q0 = 8 * c;
    const int64_t p0 = w0 + q0;
    uint2 v = make_uint2(0u, 0u);
    if (p0 >= 0 && p0 + 8 <= n && ((reinterpret_cast<uintptr_t>(w.text + p0) & 7u) == 0)) {
      v = *reinterpret_cast<const uint2*>(w.text + p0);
    } else {
      uint32_t lo = 0, hi = 0;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        int64_t p = p0 + k;
        uint32_t b = (p >= 0 && p < n) ? w.text[p] : 0u;
        if (k < 4) lo |= b << (8 * k);
        else hi |= b << (8 * (k - 4));
      }
      v = make_uint2(lo, hi);
    }
    *reinterpret_cast<uint2*>(&sh.buf[PT_PAD + q0]) = v;
    if (!BATCH) return;  // (the text start is the only document start)
    uint2 d = make_uint2(0u, 0u);
    if (p0 <= 0 && p0 + 8 > 0) d.x = (p0 == 0) ? 1u : 0u;  // the text start is a document start
    if (p0 < 0 && p0 + 8 > 0) {
      int k = (int)(-p0);
      if (k < 4) d.x = 1u << (8 * k);
      else d.y = 1u << (8 * (k - 4));
    }
    *reinterpret_cast<uint2*>(&sh.dstart[PT_PAD + q0]) = d;
  };
  {
    constexpr int NCH = PT_WIN / 8;  // chunks of the window proper
    if (tid < NCH) stage_chunk(tid);
    else if (tid < NCH + 3) stage_chunk(tid == NCH ? -1 : tid - 1);  // [-8, 0) and [PT_WIN, PT_WIN + 16)
  }
  uint2 docs = make_uint2(0u, 0u);  // batch: the first documents at or after the window's start and end
  if (BATCH) {
    docs = w.tile_docs[t];
  }
  __syncthreads();
  if (BATCH) {
    for (int64_t j = (int64_t)docs.x + tid; j < w.n_docs; j += PT_THREADS) {
      int64_t d = w.doc_off[j];
      if (d >= w0 + PT_WIN + 16) break;
      if (d >= n) continue;
      sh.dstart[PT_PAD + (d - w0)] = 1;
    }
    __syncthreads();
  }

  TT_PHASE(2);
  // ---- decode, validate, classify ------------------------------------------
  // A thread's four positions are one aligned word of the window.  It reads
  // its word and the words on either side (bytes and document-start flags) and
  // decides everything from registers: a sequence starts at most three bytes
  // before a position it covers and ends at most three bytes after.  Four
  // ASCII bytes inside the text take their codes from the ASCII table.
  // The codes are bits of the window's bitmaps, only
  // the lead bytes of longer sequences are decoded, one after the other (a
  // word of valid text holds two at most), and continuation bytes are checked
  // as byte masks of the whole word: 2.0 us of a tile in multilingual text, 4.1
  // at most (decoding at all four positions took 4.2, 10.4 at most).
  static_assert(PT_BPT == 4 && PT_PAD % 4 == 0, "classification works on aligned 4-byte words");
  bool bad = false;
  if (SPANS) {
    // the bitmap of non-continuation bytes (bytes that begin a character)
    const int q0 = tid * PT_BPT;
    const int64_t p0 = w0 + q0;
    const uint32_t x = *reinterpret_cast<const uint32_t*>(&sh.buf[PT_PAD + q0]);
    uint32_t nib = __builtin_amdgcn_udot4((~(x & ~(x << 1)) >> 7) & 0x01010101u, 0x08040201u, 0u, false);
    if (p0 < 0 || p0 + PT_BPT > n)
      for (int j = 0; j < PT_BPT; ++j)
        if (p0 + j < 0 || p0 + j >= n) nib &= ~(1u << j);
    store_nibbles(sh.ncw, q0, lane, nib);
  }
  {
    const int q0 = tid * PT_BPT;
    const int64_t p0 = w0 + q0;  // text position of the first of the four
    const uint32_t* bw = reinterpret_cast<const uint32_t*>(&sh.buf[PT_PAD + q0 - 4]);
    const uint32_t x0 = bw[0], x1 = bw[1], x2 = bw[2];
    // the low bits of four bytes as a nibble
    auto nibble = [](uint32_t x) -> uint32_t { return __builtin_amdgcn_udot4(x & 0x01010101u, 0x08040201u, 0u, false); };
    uint32_t dw1 = 0;
    if (BATCH) dw1 = *reinterpret_cast<const uint32_t*>(&sh.dstart[PT_PAD + q0]);
    // junction cuts: the byte pairs that no merge joins
    uint32_t cuts = 0;
    if (SEG && !IGN) {
      const uint64_t bb = x0 | ((uint64_t)x1 << 32);
#pragma unroll
      for (int j = 0; j < PT_BPT; ++j) {
        const uint32_t key = (uint32_t)(bb >> (8 * (j + 3)));  // b[q-1] | b[q] << 8
        const uint32_t k2 = ((key & 255u) << 8) | ((key >> 8) & 255u);
        cuts |= ((~sh.ph.a.join[k2 >> 5] >> (k2 & 31u)) & 1u) << j;
      }
    }
    const auto* asc = sh.ph.a.cls.asc;
    const auto a0 = asc[x1 & 127u], a1 = asc[(x1 >> 8) & 127u], a2 = asc[(x1 >> 16) & 127u], a3 = asc[(x1 >> 24) & 127u];
    uint32_t e, e2 = 0;  // bitmaps 0..7, and 8..15
    if constexpr (WIDE) {
      e = a0.x | (a1.x << 1) | (a2.x << 2) | (a3.x << 3);
      e2 = a0.y | (a1.y << 1) | (a2.y << 2) | (a3.y << 3);
    } else {
      e = a0 | (a1 << 1) | (a2 << 2) | (a3 << 3);
    }
    if (((x0 | x1) & 0x80808080u) != 0u) {
      const uint32_t ascii = nibble(~x1 >> 7) * 0x11111111u;  // (not the bytes above 127)
      e &= ascii;
      e2 &= ascii;
      const bool own = q0 >= PT_HALO && q0 < PT_HALO + PT_OWN;
      static_assert(PT_HALO % PT_BPT == 0 && PT_OWN % PT_BPT == 0, "a word is the tile's own or not");
      // bit 7 of every byte: leads of at least two, three and four bytes, in
      // this word and the one before, and the continuation bytes they call for
      const uint32_t l2 = x1 & (x1 << 1) & 0x80808080u, m2 = x0 & (x0 << 1) & 0x80808080u;
      const uint32_t l3 = l2 & (x1 << 2), m3 = m2 & (x0 << 2), l4 = l3 & (x1 << 3), m4 = m3 & (x0 << 3);
      const uint32_t want = __builtin_amdgcn_alignbyte(l2, m2, 3) | __builtin_amdgcn_alignbyte(l3, m3, 2) |
                            __builtin_amdgcn_alignbyte(l4, m4, 1);
      const uint32_t cont = x1 & ~(x1 << 1) & 0x80808080u;
      // (a document starts with a character; past the end of the text, where
      // the window is zero, a sequence that the end cuts shows up)
      bad = ((want ^ cont) | (cont & (dw1 << 7))) != 0u && (own || p0 + PT_BPT > n);
      uint32_t leads = l2;
      while (leads) {
        const uint32_t j = (uint32_t)__builtin_ctz(leads) >> 3;
        leads &= leads - 1u;
        const uint32_t v = __builtin_amdgcn_alignbyte(x2, x1, j);
        uint32_t cp;
        const uint32_t b0 = v & 255u;
        // (its continuation bytes are checked above: here, that the lead is
        // one and the ranges of the second byte)
        const uint32_t len = decode_sel(b0, (v >> 8) & 255u, (v >> 16) & 255u, v >> 24, 4u, cp);
        bad = bad || (own && len == 0u);
        cp = len ? cp : 0xFFFDu;
        if constexpr (WIDE) {
          const auto& ct = sh.ph.a.cls;
          const uint2 c = ct.cls[DS ? ds_table_class(ct.l1, ct.l2, cp) : o2_table_class(ct.l1, ct.l2, cp)];
          e |= c.x << j;
          e2 |= c.y << j;
        } else {
          e |= class_bits(table_class(sh.ph.a.cls, cp)) << j;
        }
      }
    }
    if (p0 < 0 || p0 + PT_BPT > n) {  // nothing is set outside the text
      uint32_t in = 0;
      for (int j = 0; j < PT_BPT; ++j) in |= (p0 + j >= 0 && p0 + j < n ? 1u : 0u) << j;
      e &= in * 0x11111111u;
      e2 &= in * 0x11111111u;
    }
    e |= cuts << (4 * BM_CUT);
    sh.ph.a.bm[(lane & 7) * BM_STRIDE + (tid >> 3)] = to_bitmaps(e, lane);
    if constexpr (WIDE) sh.ph.a.bm[(8 + (lane & 7)) * BM_STRIDE + (tid >> 3)] = to_bitmaps(e2, lane);
    if (BATCH) store_nibbles(sh.ph.a.bm_doc, q0, lane, nibble(dw1));
  }
  const bool tile_bad = __syncthreads_or(bad) != 0;
  // span export: the characters that begin before each word of the window, and
  // the tile's own, published before this block waits on anything (the
  // look-back that sums them runs at the end)
  if (SPANS && wave == 1) {
    const uint32_t x = sh.ncw[lane];
    const uint32_t c = (uint32_t)__popc(x), incl = wave_incl_sum(c);
    sh.ncpre[lane] = incl - c;
    const uint32_t own = (uint32_t)__popc(x & bm_range(PT_HALO, PT_HALO + PT_OWN, lane));
    const uint32_t c_tile = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_sum(own), 63);
    if (lane == 0) {
      sh.ctile = c_tile;
      st_word(&w.tile_cagg[t], ((uint64_t)w.epoch << PL_EPOCH_SHIFT) | c_tile);
    }
  }

  TT_PHASE(3);
  const int qb = tid * PT_BPT;  // the thread's first position
  uint32_t flags = 0;           // bit j: a piece (then: a unit) starts at qb + j
  TT_PHASE(4);
  // ---- piece starts ---------------------------------------------------------
  {
    // one wave evaluates the rules on the bitmaps and, where no vocabulary
    // probe comes between, cuts the pieces into units and numbers them
    if (wave == 0) {
      const uint32_t* bm = &sh.ph.a.bm[lane];
      auto map = [&](int k) -> uint32_t { return bm[k * BM_STRIDE]; };
      RunBits b{};
      b.N = map(BM_N);
      b.WS = map(BM_WS);
      b.NL = map(BM_NL);
      b.SP = map(BM_SP);
      b.D = BATCH ? sh.ph.a.bm_doc[lane] : (t == 0 && lane == PT_HALO / 32 ? 1u : 0u);
      b.C = b.N | b.WS | b.NL;
      O2Maps m2{};
      DsMaps md{};
      if constexpr (PAT == TT_PATTERN_O200K) {
        m2 = O2Maps{map(BM2_U), map(BM2_LO), map(BM2_X), map(BM2_M), map(BM2_APO), map(BM2_SLASH)};
        b.O = map(BM_O);
        b.C |= b.O | m2.U | m2.Lo | m2.X | m2.M;
      } else if constexpr (DS) {
        md = DsMaps{map(BMD_AL), map(BMD_L), map(BMD_AP), map(BMD_PS), map(BMD_O), map(BMD_KL), map(BMD_KP), map(BMD_KO)};
        b.C |= md.AL | md.L | md.AP | md.PS | md.O | md.KL | md.KP | md.KO;
      } else {
        b.L = map(BM_L);
        b.O = map(BM_O);
        b.APO = map(BM_APO);
        b.C |= b.L | b.O;
      }
      const int in_end = n - w0 < PT_WIN ? (int)(n - w0) : PT_WIN;
      b.K = bm_range(t == 0 ? PT_HALO : 0, in_end, lane) & ~b.C;
      b.multi = __ballot(b.K != 0u) != 0ull;
      const uint32_t own = bm_range(PT_HALO, min(in_end, PT_HALO + PT_OWN), lane);
      const uint8_t* ds = BATCH ? sh.dstart : nullptr;
      auto publish = [&](uint32_t sum) {
        if (lane == 0) st_word(&w.tile_sum[t], ((uint64_t)w.epoch << 32) | sum);
      };
      // back tile by tile (usually one step) until what is asked for (the
      // SUM_*_ALL bits) is known
      auto carry = [&](uint32_t ask) -> RunCarry {
        uint32_t acc = 0, val = 0;
        if (lane == 0) {
          uint32_t open = ask;
          for (int64_t j = (int64_t)t - 1; j >= 0 && open != 0u; --j) {
            const uint32_t v = (uint32_t)wait_word(&w.tile_sum[j], w.epoch);
            if (open & SUM_N_ALL) acc += (v >> 1) & 3u;
            const uint32_t now = open & ~v;  // told by this tile
            if (now & SUM_TAIL_ALL) val |= v & SUM_TAIL;
            if (now & SUM_STATE_ALL) val |= v & (15u << SUM_STATE_SHIFT);
            open &= ~now;
          }
        }
        acc = wave_uniform(acc);
        val = wave_uniform(val);
        return RunCarry{acc % 3u, (val & SUM_TAIL) != 0u, (val >> SUM_STATE_SHIFT) & 15u};
      };
      auto class_of = [&](uint32_t cp) -> uint32_t {
        const auto& ct = sh.ph.a.cls;
        if constexpr (DS) return cp < 128u ? ds_ascii_class(cp) : ds_table_class(ct.l1, ct.l2, cp);
        else if constexpr (WIDE) return cp < 128u ? o2_ascii_class(cp) : o2_table_class(ct.l1, ct.l2, cp);
        else return cp == 10u || cp == 13u ? 4u : cp < 128u ? (cp == 32u || (cp - 9u) < 5u ? 3u : 0u) : table_class(ct, cp);
      };
      // The first class after the window that `in` does not hold (ASCII bytes by
      // `plain`, which holds part of `in`), within the document.
      auto beyond = [&](auto plain, auto in) -> uint32_t {
        if (w0 + PT_WIN >= n) return ~0u;
        int64_t lim = n;
        if (BATCH && docs.y < (uint32_t)w.n_docs) lim = w.doc_off[docs.y];
        return first_outside(w.text + (w0 + PT_WIN), (uint32_t)(lim - (w0 + PT_WIN)), lane, plain, in, class_of);
      };
      constexpr uint32_t C_WS = DS ? (uint32_t)DS_WS : WIDE ? (uint32_t)O2_WS : 3u;
      constexpr uint32_t C_NL = DS ? (uint32_t)DS_NL : WIDE ? (uint32_t)O2_NL : 4u;
      // whether no CR/LF follows the whitespace stretch that reaches the window's end
      auto last_ws = [&]() -> bool {
        return beyond([](uint32_t c) { return c == 0x20u || c == 0x09u || c == 0x0Bu || c == 0x0Cu; },
                      [](uint32_t c) { return c == C_WS || (DS && c == (uint32_t)DS_SP); }) != C_NL;
      };
      uint32_t st;
      if constexpr (PAT == TT_PATTERN_GPT2) {
        st = gpt2_starts(b, sh.buf, ds, lane);
      } else if constexpr (PAT == TT_PATTERN_CL100K) {
        st = cl100k_starts(b, own, sh.buf, ds, lane, t == 0, publish, carry, last_ws);
      } else if constexpr (DS) {
        st = deepseek_starts(b, md, own, lane, t == 0, publish, carry, last_ws);
      } else {
        st = o200k_starts(b, m2, own, sh.buf, ds, lane, t == 0, publish, carry, last_ws, [&]() -> bool {
          const uint32_t c = beyond([](uint32_t x) { return x - 'A' < 26u; }, [](uint32_t x) { return x == O2_UP; });
          return c == O2_LO || c == O2_BO || c == O2_MK;
        });
      }
      uint32_t u = st & own;
      if (SEG && !IGN) u |= map(BM_CUT) & own & ~b.D;
      const uint32_t c = (uint32_t)__popc(u);
      const uint32_t incl = wave_incl_sum(c);
      sh.uw[lane] = u;
      sh.upre[lane] = incl - c;
      if (lane == 63) sh.m = incl;
      if (SEG && !IGN) {
        // the tile's last unit start, published before this block waits on
        // anything (a carry only waits for words published before any wait)
        const int l = bm_last(u);
        if (lane == 0) st_word(&w.tile_last[t], ((uint64_t)w.epoch << 32) | (l < 0 ? NO_START : (uint32_t)(w0 + l)));
      }
    }
    __syncthreads();
    flags = (sh.uw[tid >> 3] >> (qb & 31)) & 15u;
  }
  TT_PHASE(21);
  const bool last = t == n_tiles - 1;
  if (IGN) {
    // ignore_merges: a piece that is a vocabulary entry is that entry's ID
    // (Sec. 4.2: the vocabulary is probed first and the merge loop skipped).
    // Pieces are numbered by a block scan (their starts go to sh.ustart until
    // the unit scan), every piece that ends inside the tile is probed, and no
    // junction cut may split a piece found in the vocabulary.  The pieces that
    // cross the tile's edges are not cut at all: the next tile encodes the
    // last one whole, as its incoming unit, and probes it there.
    const uint32_t pc = __popc(flags);
    const uint32_t pinc = wave_incl_sum(pc);
    __syncthreads();
    if (lane == 63) sh.wave_tot[wave] = pinc;
    __syncthreads();
    uint32_t pw = 0, pm = 0;
    for (int v = 0; v < PT_THREADS / 64; ++v) {
      if (v < wave) pw += sh.wave_tot[v];
      pm += sh.wave_tot[v];
    }
    {
      uint32_t k = pw + pinc - pc;
#pragma unroll 1
      for (int j = 0; j < PT_BPT; ++j)
        if ((flags >> j) & 1u) sh.ustart[k++] = (uint16_t)(qb + j);
    }
    if (tid == 0) sh.ustart[pm] = (uint16_t)(last ? n - w0 : 0xFFFFu);  // end of the last piece, if known
    __syncthreads();
#pragma unroll 1
    for (uint32_t k = (uint32_t)tid; k < pm; k += PT_THREADS) {
      const uint32_t a = sh.ustart[k], e = sh.ustart[k + 1];
      if (e == 0xFFFFu) continue;
      const uint32_t L = e - a;
      if (L < 2u || L > tb.vmax) continue;
      const uint32_t id = piece_find(tb, sh.buf, (int64_t)a, L, [&](uint32_t j) -> uint32_t { return sh.buf[PT_PAD + a + j]; });
      if (id == DICT_NONE) continue;
      w.stage[w0 + a] = id;
      atomicOr(&sh.whole[a >> 5], 1u << (a & 31u));
      for (uint32_t q = a + 1; q < e; ++q) atomicOr(&sh.ph.a.nocut[q >> 5], 1u << (q & 31u));
    }
    // the incoming piece's tail and the tile's last piece
    const uint32_t first = pm > 0 ? sh.ustart[0] : (uint32_t)(PT_HALO + PT_OWN);
    const uint32_t lastp = pm > 0 ? sh.ustart[pm - 1] : (uint32_t)PT_HALO;
    uint32_t mask = 0;
#pragma unroll
    for (int j = 0; j < PT_BPT; ++j) {
      const uint32_t q = (uint32_t)(qb + j);
      const bool own = q >= (uint32_t)PT_HALO && q < (uint32_t)(PT_HALO + PT_OWN);
      if (own && ((t > 0 && q < first) || (!last && q > lastp))) mask |= 1u << j;
    }
    if (mask) atomicOr(&sh.ph.a.nocut[qb >> 5], mask << (qb & 31));
    __syncthreads();
  }
  TT_PHASE(22);
  if (SEG && IGN) {
    // BPE segments: add the byte positions inside pieces that no merge spans
    // (q is not a piece start, so q - 1 lies in the same piece)
    const uint32_t* bwp = reinterpret_cast<const uint32_t*>(&sh.buf[PT_PAD + qb - 4]);
    const uint64_t bb = bwp[0] | ((uint64_t)bwp[1] << 32);  // bytes of positions qb - 4 .. qb + 3
#pragma unroll
    for (int j = 0; j < PT_BPT; ++j) {
      const int q = qb + j;
      const uint32_t key = (uint32_t)((bb >> (8 * (j + 3))) & 0xFFFFull);  // (b[q-1], b[q]) as b[q-1] | b[q] << 8
      const uint32_t k2 = ((key & 255u) << 8) | (key >> 8);
      const bool joined = (sh.ph.a.join[k2 >> 5] >> (k2 & 31u)) & 1u;
      const bool eligible = q >= PT_HALO && q < PT_HALO + PT_OWN && inside(q) && inside(q - 1) &&
                            !(flags & (1u << j)) && !(BATCH && sh.dstart[PT_PAD + q]) &&
                            !((sh.ph.a.nocut[q >> 5] >> (q & 31)) & 1u);
      if (eligible && !joined) flags |= 1u << j;
    }
  }

  TT_PHASE(5);
  TT_PHASE_BY(24 + wave, lane == 0);
  // ---- units: numbered by the wave that found them, or by a block scan of the
  // start flags
  const uint32_t cnt = __popc(flags);
  uint32_t m, texcl;  // unit starts of the tile, and those before this thread's positions
  if constexpr (IGN) {
    const uint32_t inc = wave_incl_sum(cnt);
    __syncthreads();
    if (lane == 63) sh.wave_tot[wave] = inc;
    __syncthreads();
    uint32_t wpre = 0;
    m = 0;
    for (int v = 0; v < PT_THREADS / 64; ++v) {
      if (v < wave) wpre += sh.wave_tot[v];
      m += sh.wave_tot[v];
    }
    m = wave_uniform(m);
    texcl = wave_uniform(wpre) + inc - cnt;
  } else {
    m = wave_uniform(sh.m);
    texcl = sh.upre[tid >> 3] + (uint32_t)__popc(sh.uw[tid >> 3] & ((1u << (qb & 31)) - 1u));
  }

  if (MODE == 0) {
    // split export: the tile's piece offsets go straight to their place
    if (tid == 0) publish_count(w, t, m, tile_bad);
    const uint32_t prefix = place_tile(w, sh, t, m, tile_bad, tid, lane, wave);
    uint32_t k = prefix + texcl;
#pragma unroll 1
    for (int j = 0; j < PT_BPT; ++j)
      if (((flags >> j) & 1u) && k < (uint32_t)n) w.out_ids[k++] = (int32_t)(w0 + qb + j);
    return;
  }

  TT_PHASE(11);
  // the tile's last unit start, published before this block waits on anything
  if constexpr (!IGN) {
    // (published with the starts)
  } else if (m == 0) {
    if (tid == 0) st_word(&w.tile_last[t], ((uint64_t)w.epoch << 32) | NO_START);
  } else if (cnt != 0u && texcl + cnt == m) {
    st_word(&w.tile_last[t], ((uint64_t)w.epoch << 32) | (uint32_t)(w0 + qb + 31 - __builtin_clz(flags)));
  }
  {
    uint32_t k = texcl;
#pragma unroll 1
    for (int j = 0; j < PT_BPT; ++j)
      if ((flags >> j) & 1u) sh.ustart[k++] = (uint16_t)(qb + j);
  }
  if (tid == 0) sh.ustart[m] = (uint16_t)(last ? n - w0 : 0);

  // The units this tile encodes: its own units but the last (whose end lies
  // in a later tile), all of them in the last tile, and the incoming unit
  // that ends at its first unit start.
  const bool has_inc = t > 0 && (m > 0 || last);
  const uint32_t m_proc = last ? m : (m > 0 ? m - 1 : 0);
  __syncthreads();
  const uint32_t e_inc = wave_uniform(m > 0 ? (uint32_t)(w0 + sh.ustart[0]) : (uint32_t)n);
  auto byte_abs = [&](uint32_t p) -> uint32_t {
    const int64_t q = (int64_t)p - w0;
    return (q >= -PT_PAD && q < PT_WIN + 16) ? (uint32_t)sh.buf[PT_PAD + q] : (uint32_t)w.text[p];
  };
  // The incoming unit starts at the last unit start of the nearest earlier
  // tile that has one (usually the previous tile).  Only the thread that
  // dispatches it waits for that word; the others dispatch their own units
  // meanwhile.  (Only invalid input, whose text starts with a continuation
  // byte, leaves no unit start before the tile; its output is discarded.)
  TT_PHASE(12);
  uint32_t sp_own = 0;
  if (has_inc && (uint32_t)tid == m_proc % (uint32_t)PT_THREADS) {
    uint32_t found = NO_START;
    for (int64_t j = (int64_t)t - 1; j >= 0; --j) {
      const uint64_t x = wait_word(&w.tile_last[j], w.epoch);
      if ((uint32_t)x != NO_START) {
        found = (uint32_t)x;
        break;
      }
    }
    sh.s_prev = found;
    sp_own = found != NO_START ? found : 0u;
    TT_PHASE_BY(20, true);
  }
  auto inc_byte_own = [&](uint32_t j) -> uint32_t { return byte_abs(sp_own + j); };
  auto inc_out_own = [&](uint32_t j, uint32_t id) { w.stage[sp_own + j] = id; };

  // ---- BPE dispatch ---------------------------------------------------------
  // Units of one or two bytes are finished here, and so are units of up to 24
  // bytes found in the whole-unit dictionaries.  Other units of up to WAVE_MAX
  // bytes go to the wave engines: those of 3..16 bytes counting-sorted by
  // length (units that share a wave should take about as many rounds), longer
  // ones in 8-byte classes.  Longer units go to the whole block.
  constexpr int UPT = (PT_OWN + 1 + PT_THREADS - 1) / PT_THREADS;  // units per thread
  const uint32_t U = m_proc + (has_inc ? 1u : 0u);
  uint32_t mine[UPT];  // units of the wave engines: (length << 16) | position within its length class
#pragma unroll
  for (int r = 0; r < UPT; ++r) {
    mine[r] = 0;
    const uint32_t u = (uint32_t)(tid + r * PT_THREADS);
    if (u >= U) continue;
    const bool inc_u = u == m_proc;
    const uint32_t a = inc_u ? 0u : sh.ustart[u];
    const uint32_t L = inc_u ? e_inc - sp_own : sh.ustart[u + 1] - a;
    if (IGN) {
      // a piece found in the vocabulary (its ID was staged at its first byte);
      // the incoming unit is a whole piece and is probed here
      uint32_t id = DICT_NONE;
      if (!inc_u && ((sh.whole[a >> 5] >> (a & 31u)) & 1u)) {
        id = w.stage[w0 + a];
      } else if (inc_u && L >= 2u && L <= tb.vmax) {
        id = piece_find(tb, sh.buf, (int64_t)sp_own - w0, L, [&](uint32_t j) -> uint32_t { return inc_byte_own(j); });
      }
      if (id != DICT_NONE) {
        if (inc_u) {
          inc_out_own(0, id);
          sh.inc_cnt = 1;
        } else {
          sh.ph.b.tok[a] = id;
          sh.ucnt[u] = 1;
        }
        continue;
      }
    }
    if (L <= 2u) {
      const uint32_t b0 = inc_u ? inc_byte_own(0) : sh.buf[PT_PAD + a];
      uint32_t c = 1, t0 = b0, t1 = 0;
      if (L == 2u) {
        const uint32_t b1 = inc_u ? inc_byte_own(1) : sh.buf[PT_PAD + a + 1];
        const uint32_t r2 = tb.pairj[(b0 << 8) | b1].rank;
        if (r2 != RANK_INF) {
          t0 = 256u + r2;
        } else {
          c = 2;
          t1 = b1;
        }
      }
      if (inc_u) {
        inc_out_own(0, t0);
        if (c == 2) inc_out_own(1, t1);
        sh.inc_cnt = c;
      } else {
        sh.ph.b.tok[a] = t0;
        if (c == 2) sh.ph.b.tok[a + 1] = t1;
        sh.ucnt[u] = (uint16_t)c;
      }
    } else {
      // units of 3..24 bytes: the whole-unit dictionaries first.  Their bytes
      // are in the window (an incoming unit this short ends at the tile's
      // first unit start, so it starts at least PT_HALO - 24 bytes into it).
      uint32_t found = DICT_NONE;
      const int64_t aw = inc_u ? (int64_t)sp_own - w0 : (int64_t)a;
      if (L <= (uint32_t)DICT2_MAX && aw >= 0 && aw + DICT2_MAX + 4 <= PT_WIN + 16) {
        if (L <= (uint32_t)DICT_MAX) {
          uint32_t kw[3];
          unit_words(sh.buf, (uint32_t)aw, L, kw);
          found = dict_find(tb.dict, tb.dnb, kw[0], kw[1], kw[2], L);
        } else {
          uint32_t kw[6];
          unit_words(sh.buf, (uint32_t)aw, L, kw);
          found = dict2_find(tb.dict2, tb.dnb2, kw, L);
        }
      }
      if (found != DICT_NONE) {
        if (inc_u) {
          inc_out_own(0, found);
          sh.inc_cnt = 1;
        } else {
          sh.ph.b.tok[a] = found;
          sh.ucnt[u] = 1;
        }
      } else if (L <= (uint32_t)SMALL_MAX) {
        mine[r] = (L << 16) | atomicAdd(&sh.hist[L], 1u);
      } else if (L <= (uint32_t)WAVE_MAX) {
        mine[r] = (L << 16) | atomicAdd(&sh.hmed[med_class(L)], 1u);
      } else {
        sh.big[atomicAdd(&sh.n_big, 1u)] = inc_u ? U_INCOMING : (uint16_t)u;
      }
    }
  }
  __syncthreads();
  const uint32_t s_prev = wave_uniform(has_inc && sh.s_prev != NO_START ? sh.s_prev : 0u);
  const uint32_t L_inc = has_inc ? e_inc - s_prev : 0u;
  auto inc_byte = [&](uint32_t j) -> uint32_t { return byte_abs(s_prev + j); };
  auto inc_out = [&](uint32_t j, uint32_t id) { w.stage[s_prev + j] = id; };
  TT_PHASE(13);
  // where each length (class) starts: a wave scan over the counts (wave 0 for
  // units of up to 16 bytes, wave 1 for the longer ones)
  if (wave == 0) {
    const bool in = lane >= 3 && lane <= SMALL_MAX;
    const uint32_t c = in ? sh.hist[lane] : 0u;
    const uint32_t incl = wave_incl_sum(c);
    if (in) sh.hist[lane] = incl - c;
    if (lane == SMALL_MAX) sh.n_small = incl;
  } else if (wave == 1) {
    const bool in = lane < MED_CLASSES;
    const uint32_t c = in ? sh.hmed[lane] : 0u;
    const uint32_t incl = wave_incl_sum(c);
    if (in) sh.hmed[lane] = incl - c;
    if (lane == MED_CLASSES - 1) sh.n_med = incl;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < UPT; ++r) {
    if (mine[r] == 0) continue;
    const uint32_t u = (uint32_t)(tid + r * PT_THREADS);
    const uint16_t e = u == m_proc ? U_INCOMING : (uint16_t)u;
    const uint32_t L = mine[r] >> 16, pos = mine[r] & 0xFFFFu;
    if (L <= (uint32_t)SMALL_MAX) sh.ph.b.small[sh.hist[L] + pos] = e;
    else sh.med[sh.hmed[med_class(L)] + pos] = e;
  }
  __syncthreads();
  TT_PHASE(14);
  const uint32_t n_small = wave_uniform(sh.n_small), n_med = wave_uniform(sh.n_med);

  TT_PHASE(6);
  // The wave engines.  A pass is what a wave encodes at once: one unit of
  // 65..128 bytes, one of 33..64, two of 17..32, four of 9..16 or eight of
  // 3..8.  Passes are ordered by the units' length, longest first (they take
  // the most rounds); a wave's first pass is the one of its own number, and
  // the waves take the others from a shared counter as they become free.
  {
    const uint32_t n2 = wave_uniform(sh.hmed[med_class(64)]);        // units of 65..128 bytes
    const uint32_t b32 = wave_uniform(sh.hmed[med_class(32)]);       // first unit of 17..32 bytes
    const uint32_t n8 = wave_uniform(sh.hist[9]);                    // units of 3..8 bytes
    const uint32_t p64 = b32, p32 = p64 + (n_med - b32 + 1u) / 2u;   // passes up to each width
    const uint32_t p16 = p32 + (n_small - n8 + 3u) / 4u, p8 = p16 + (n8 + 7u) / 8u;
    uint32_t i = wave_uniform((uint32_t)wave);
#pragma unroll 1
    while (i < p8) {
      if (i < n2) {
        const uint32_t u = wave_uniform(sh.med[i]);
        const bool inc_u = u == U_INCOMING;
        const uint32_t a = inc_u ? 0u : sh.ustart[u];
        const uint32_t L = inc_u ? L_inc : sh.ustart[u + 1] - a;
        const uint32_t c = bpe_wave2(
            L,
            [&](int j) -> uint32_t {
              return inc_u ? inc_byte((uint32_t)j) : (uint32_t)sh.buf[PT_PAD + a + (uint32_t)j];
            },
            tb, sh.ph.b.x.wscr[wave],
            [&](int j, uint32_t id) {
              if (inc_u) inc_out((uint32_t)j, id);
              else sh.ph.b.tok[a + (uint32_t)j] = id;
            });
        if (lane == 0) {
          if (inc_u) sh.inc_cnt = c;
          else sh.ucnt[u] = (uint16_t)c;
        }
      } else {
        // the lane's unit: entry k of its list, counted so that the longest
        // come first (the short units' list is in ascending order)
        const uint32_t W = i < p64 ? 64u : i < p32 ? 32u : i < p16 ? 16u : 8u;
        const uint32_t g = (uint32_t)lane / W;
        uint32_t k, e;
        if (W >= 32u) {
          k = W == 64u ? i : b32 + 2u * (i - p64) + g;
          e = n_med;
        } else {
          k = W == 16u ? 4u * (i - p32) + g : n_small - n8 + 8u * (i - p16) + g;
          e = W == 16u ? n_small - n8 : n_small;
        }
        const uint16_t* list = W >= 32u ? sh.med : sh.ph.b.small;
        const bool has = k < e;
        const uint32_t u = has ? list[W >= 32u ? k : n_small - 1u - k] : 0u;
        const bool inc_u = has && u == U_INCOMING;
        const uint32_t a = !has || inc_u ? 0u : sh.ustart[u];
        const uint32_t L = !has ? 0u : inc_u ? L_inc : sh.ustart[u + 1] - a;
        const uint32_t j = (uint32_t)lane & (W - 1u);
        uint32_t id = 0u;
        if (j < L) id = inc_u ? inc_byte(j) : (uint32_t)sh.buf[PT_PAD + a + j];
        const uint64_t alive = W == 64u ? bpe_lanes<true>(64u, L, id, tb, id) : bpe_lanes<false>(W, L, id, tb, id);
        const uint64_t own = alive & (W == 64u ? ~0ull : (((1ull << W) - 1ull) << ((uint32_t)lane - j)));
        if ((alive >> lane) & 1ull) {
          const uint32_t o = bits_below(own);
          if (inc_u) inc_out(o, id);
          else sh.ph.b.tok[a + o] = id;
        }
        if (has && j == 0u) {
          const uint32_t c = (uint32_t)__popcll(own);
          if (inc_u) sh.inc_cnt = c;
          else sh.ucnt[u] = (uint16_t)c;
        }
      }
      // all 64 lanes add one (no branch on the lane before the broadcast,
      // which would make the loop exit divergent), so a wave's grab moves the
      // counter by 64 and lane 0 reads a multiple of 64
      i = (uint32_t)(PT_THREADS / 64) + wave_uniform(atomicAdd(&sh.pass_next, 1u)) / 64u;
    }
  }
  __syncthreads();

  TT_PHASE(7);
  // ---- BPE, whole block per longer unit ------------------------------------
  // (units of more than WAVE_MAX bytes, rare in text: rows in LDS up to ROWS_LDS
  // bytes, else in global scratch at the unit's byte offset; there the selection
  // masks of a unit of L > ROWS_LDS bytes at byte s take words
  // [s/16, s/16 + L/64 + 2), which never reach the next unit's)
  const uint32_t n_big = sh.n_big;
  // With six waves per SIMD (requests that do not fill the chip) the engine's code
  // is placed behind the kernel's and reads its arguments again: 100K of prose and
  // code 17.65 -> 17.05 us; with eight it stays in line (8M characters 133 us, 135 the
  // other way).
  if (__builtin_expect(n_big != 0u, WAVES == 8))
#pragma unroll 1
  for (uint32_t i = 0; i < n_big; ++i) {
    const uint32_t u = sh.big[i];
    const bool inc_u = u == U_INCOMING;
    const uint32_t a = inc_u ? 0u : sh.ustart[u];
    const uint32_t L = inc_u ? L_inc : sh.ustart[u + 1] - a;
    const uint64_t s0 = inc_u ? (uint64_t)s_prev : (uint64_t)(w0 + a);
    const Work& rw = WAVES == 8 ? w : tile_args().w;
    const DevTables& rt = WAVES == 8 ? tb : tile_args().tb;
    const uint8_t* __restrict__ src = rw.text + s0;
    uint32_t* stage = rw.stage + s0;
    auto out = [&](uint32_t j, uint32_t id) {
      if (inc_u) stage[j] = id;
      else sh.ph.b.tok[a + j] = id;
    };
    uint32_t c;
    if (L <= (uint32_t)ROWS_LDS) {
      auto& rows = sh.ph.b.x.rows;
      c = bpe_rows<PT_THREADS / 64>(L, src, rt, rows.tok, ROWS_LDS, rows.sel, sh.rows, out);
    } else {
      const uint64_t nn = (uint64_t)n;
      uint64_t* sc = reinterpret_cast<uint64_t*>(rw.scratch);
      c = bpe_rows<PT_THREADS / 64>(L, src, rt, sc + s0, nn, sc + 2 * nn + s0 / 16, sh.rows, out);
    }
    if (tid == 0) {
      if (inc_u) sh.inc_cnt = c;
      else sh.ucnt[u] = (uint16_t)c;
    }
    __syncthreads();
  }

  TT_PHASE(8);
  // ---- output: the tile's tokens, in order, at their place --------------------
  uint32_t csum = 0;
#pragma unroll 1
  for (int j = 0; j < PT_BPT; ++j) {
    const uint32_t k = (uint32_t)(tid * PT_BPT + j);
    csum += k < m_proc ? sh.ucnt[k] : 0u;
  }
  const uint32_t cinc = wave_incl_sum(csum);
  if (lane == 63) sh.wave_tot[wave] = cinc;
  __syncthreads();
  uint32_t cpre = 0, ctot = 0;
  for (int v = 0; v < PT_THREADS / 64; ++v) {
    if (v < wave) cpre += sh.wave_tot[v];
    ctot += sh.wave_tot[v];
  }
  // The count is published before the tokens are put in order, so that later
  // tiles wait for neither that nor this tile's own look-back.
  const uint32_t inc_cnt = has_inc ? sh.inc_cnt : 0u;
  if (tid == 0) publish_count(w, t, inc_cnt + ctot, tile_bad);
  {
    uint32_t o = cpre + cinc - csum;
#pragma unroll 1
    for (int j = 0; j < PT_BPT; ++j) {
      const uint32_t k = (uint32_t)(tid * PT_BPT + j);
      if (k < m_proc) {
        sh.ph.b.uoff[k] = (uint16_t)o;
        o += sh.ucnt[k];
      }
    }
  }
  __syncthreads();
  // Token o of unit k sits at position ustart[k] + o.  The tokens become the
  // caller's IDs and are packed in order while the look-back's words arrive, so
  // that after it every store is a full line of consecutive outputs (which
  // matters most when the output is pinned host memory).
  // Packing per wave after the look-back, with the count published only there,
  // took 267 us for a 16M corpus (now 246), 47.6 us for 1M multilingual
  // characters (45.2) and 18.7 us for 100K (17.5).
  const int32_t* __restrict__ ext = tb.ext_id;
  auto ext_of = [&](uint32_t v) -> int32_t { return v < tb.n_ids ? ext[v] : -1; };
  auto len_of = [&](uint32_t v) -> uint32_t { return v < tb.n_ids ? tb.tok_len[v] : 0u; };
  {
    uint32_t before = texcl;  // unit starts at or before position q
    uint32_t val[PT_BPT], at_of[PT_BPT], span[PT_BPT];
    uint32_t has = 0;
#pragma unroll
    for (int j = 0; j < PT_BPT; ++j) {
      const int q = qb + j;
      const bool st = (flags >> j) & 1u;
      before += st ? 1u : 0u;
      val[j] = 0;
      at_of[j] = 0;
      span[j] = 0;
      if (before == 0u || before - 1u >= m_proc) continue;
      const uint32_t k = before - 1u;
      const uint32_t o = (uint32_t)q - sh.ustart[k];
      if (o < sh.ucnt[k]) {
        const uint32_t tok = sh.ph.b.tok[q];
        val[j] = (uint32_t)ext_of(tok);
        at_of[j] = sh.ph.b.uoff[k] + o;
        has |= 1u << j;
        if (SPANS) span[j] = len_of(tok);
      }
    }
    if (SPANS) {
      // byte start of every token: its unit's start plus the byte lengths of
      // the unit's earlier tokens (byte-level BPE fixes every token's length):
      // a scan over the positions, restarted at every unit start
      constexpr uint32_t HEAD = 0x80000000u;
      auto seg_add = [](uint32_t a, uint32_t b) -> uint32_t {
        return (b & HEAD) ? b : ((a & HEAD) | ((a + b) & ~HEAD));
      };
      uint32_t agg = 0;
#pragma unroll
      for (int j = 0; j < PT_BPT; ++j) agg = seg_add(agg, (((flags >> j) & 1u) ? HEAD : 0u) | span[j]);
      const uint32_t winc = wave_incl_scan(agg, lane, seg_add);
      if (lane == 63) sh.cwave[wave] = winc;
      uint32_t st = (uint32_t)__shfl_up((int)winc, 1, 64);
      if (lane == 0) st = 0;
      __syncthreads();
      uint32_t wpre = 0;
      for (int v = 0; v < wave; ++v) wpre = seg_add(wpre, sh.cwave[v]);
      st = seg_add(wpre, st);
      uint32_t bf = texcl;
#pragma unroll
      for (int j = 0; j < PT_BPT; ++j) {
        const uint32_t hd = (flags >> j) & 1u, len = span[j];
        bf += hd;
        if ((has >> j) & 1u) span[j] = (sh.ustart[bf - 1u] + (hd ? 0u : (st & ~HEAD))) | (len << 16);
        st = seg_add(st, (hd ? HEAD : 0u) | len);
      }
    }
    __syncthreads();  // every read of tok[] and uoff[] is done
#pragma unroll
    for (int j = 0; j < PT_BPT; ++j)
      if ((has >> j) & 1u) {
        sh.ph.c.id[at_of[j]] = val[j];
        if (SPANS) sh.ph.c.span[at_of[j]] = span[j];
      }
  }
  uint32_t inc_val = 0;
  if ((uint32_t)tid < inc_cnt) inc_val = (uint32_t)ext_of(w.stage[s_prev + (uint32_t)tid]);
  // (place_tile ends with a barrier, which also publishes the packed outputs)
  const uint32_t prefix = place_tile(w, sh, t, inc_cnt + ctot, tile_bad, tid, lane, wave,
                                     SPANS ? w.tile_cagg : nullptr, SPANS ? sh.ctile : 0u);
  TT_PHASE(9);
  // Valid input gives every tile a disjoint byte range and at most one output
  // per byte, so every output index is below n.  Invalid input (whose output
  // is discarded) can break that; the bound keeps it inside the buffer.
  const uint32_t lim = (uint32_t)n;
  int32_t* __restrict__ out = w.out_ids;
  uint16_t* __restrict__ out16 = SPANS ? nullptr : w.out16;
  uint8_t* __restrict__ out_hi = SPANS ? nullptr : w.out_hi;
  auto put = [&](uint32_t at, uint32_t v) {
    if (at >= lim) return;
    if (out16) {
      out16[at] = (uint16_t)v;
      if (out_hi) out_hi[at] = (uint8_t)(v >> 16);
    } else {
      out[at] = (int32_t)v;
    }
  };
  if ((uint32_t)tid < inc_cnt) put(prefix + (uint32_t)tid, inc_val);
  for (uint32_t i = (uint32_t)tid + PT_THREADS; i < inc_cnt; i += 4u * PT_THREADS) {  // (a long incoming unit)
    uint32_t v[4];
#pragma unroll
    for (uint32_t k = 0; k < 4u; ++k) v[k] = w.stage[s_prev + min(i + k * PT_THREADS, inc_cnt - 1u)];
#pragma unroll
    for (uint32_t k = 0; k < 4u; ++k) {
      const int32_t e = ext[min(v[k], tb.n_ids - 1u)];
      v[k] = v[k] < tb.n_ids ? (uint32_t)e : 0xFFFFFFFFu;
    }
#pragma unroll
    for (uint32_t k = 0; k < 4u; ++k)
      if (i + k * PT_THREADS < inc_cnt) put(prefix + i + k * PT_THREADS, v[k]);
  }
  const uint32_t obase = prefix + inc_cnt;
  for (uint32_t i = (uint32_t)tid; i < ctot; i += PT_THREADS) put(obase + i, sh.ph.c.id[i]);
  if (BATCH) {
    // The output offset of every document whose first unit this tile encodes
    // (a document starts a unit), and in the last tile the total, or the error.
    if constexpr (IGN) {  // (else the unit starts are still there)
      store_nibbles(sh.uw, qb, lane, flags);
      if ((tid & 7) == 0) sh.upre[tid >> 3] = texcl;
      __syncthreads();
    }
    for (int64_t j = (int64_t)docs.x + tid; j <= w.n_docs; j += PT_THREADS) {
      const int64_t d = w.doc_off[j];
      if (d >= n) {
        if (!last) break;
        w.out_doc_off[j] = sh.err ? (int64_t)TT_ERR_INVALID_UTF8 : (int64_t)(obase + ctot);
        continue;
      }
      if (d >= t0 + PT_OWN) break;
      if (has_inc && d == (int64_t)s_prev) {
        w.out_doc_off[j] = prefix;
      } else if (d >= t0) {
        const uint32_t q = (uint32_t)(d - w0);
        const uint32_t k = sh.upre[q >> 5] + (uint32_t)__popc(sh.uw[q >> 5] & ((1u << (q & 31u)) - 1u));
        if (k < m_proc) w.out_doc_off[j] = obase + sh.ph.b.uoff[k];
      }
    }
    // an incoming unit that starts before the listed documents
    if (has_inc && (int64_t)s_prev < w0 - PT_PAD && tid == 0) {
      int64_t lo = 0, hi = docs.x;
      while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (w.doc_off[mid] < (int64_t)s_prev) lo = mid + 1;
        else hi = mid;
      }
      if (lo < (int64_t)docs.x && w.doc_off[lo] == (int64_t)s_prev) w.out_doc_off[lo] = prefix;
    }
  }
  if (SPANS) {
    // Character spans from the count of non-continuation bytes before a byte:
    // begin is the character that holds the token's first byte, end one past
    // the character that holds its last.
    Span* __restrict__ spans = reinterpret_cast<Span*>(w.out_spans);
    const uint32_t c0 = sh.cbase - sh.ncpre[PT_HALO / 32];  // characters that begin before the window
    auto chars_before = [&](uint32_t q) -> uint32_t {       // window position, below PT_WIN
      return c0 + sh.ncpre[q >> 5] + (uint32_t)__popc(sh.ncw[q >> 5] & ((1u << (q & 31u)) - 1u));
    };
    auto put_span = [&](uint32_t at, uint32_t b, uint32_t len) {  // b: byte start in the window
      const uint32_t e = min(b + len, (uint32_t)PT_WIN - 1u);     // (a unit of the tile ends inside the window)
      if (at < lim)
        spans[at] = Span{(int)(w0 + b), (int)(w0 + e), (int)(chars_before(b + 1u) - 1u), (int)chars_before(e)};
    };
    for (uint32_t i = (uint32_t)tid; i < ctot; i += PT_THREADS) {
      const uint32_t v = sh.ph.c.span[i];
      put_span(obase + i, v & 0xFFFFu, v >> 16);
    }
    if (inc_cnt == 0u) {
      // (no incoming unit)
    } else if ((int64_t)s_prev >= w0) {
      // the incoming unit lies in the window: one wave, 64 tokens at a time
      if (wave == PT_THREADS / 64 - 1) {
        uint32_t b = (uint32_t)((int64_t)s_prev - w0);
#pragma unroll 1
        for (uint32_t base = 0; base < inc_cnt; base += 64) {
          const uint32_t i = base + (uint32_t)lane;
          const uint32_t len = i < inc_cnt ? len_of(w.stage[s_prev + i]) : 0u;
          const uint32_t incl = wave_incl_sum(len);
          if (i < inc_cnt) put_span(prefix + i, b + incl - len, len);
          b += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        }
      }
    } else {
      // a unit that starts before the window: the characters that begin between
      // its start and the window, then a scan over its tokens, PT_THREADS at a
      // time, of their lengths and of the characters that begin in them
      // characters that begin in the 16 bytes from p on, or in those before e: four
      // loads in flight (the request may lie across the bus; a byte a load took
      // 3.15 ms for 400,000 letters of one unit, now 2.24)
      auto begins = [&](uint32_t p, uint32_t e) -> uint32_t {
        uint32_t x[4], c = 0;
#pragma unroll
        for (uint32_t i = 0; i < 4u; ++i) {
          const uint32_t q = p + 4u * i;
          x[i] = 0;
          if (q >= e) continue;
          if (q + 4u <= (uint32_t)n) __builtin_memcpy(&x[i], w.text + q, 4);
          else for (uint32_t k = 0; q + k < e; ++k) x[i] |= (uint32_t)w.text[q + k] << (8u * k);
        }
#pragma unroll
        for (uint32_t i = 0; i < 4u; ++i) {
          const uint32_t q = p + 4u * i, left = e > q ? e - q : 0u;
          const uint32_t in = left >= 4u ? 0x80808080u : 0x80808080u & ((1u << (8u * left)) - 1u);
          c += (uint32_t)__popc(~(x[i] & ~(x[i] << 1)) & in);
        }
        return c;
      };
      auto block_scan = [&](uint32_t v, uint32_t& total) -> uint32_t {  // exclusive
        const uint32_t incl = wave_incl_sum(v);
        __syncthreads();
        if (lane == 63) sh.cwave[wave] = incl;
        __syncthreads();
        uint32_t pre = 0;
        total = 0;
        for (int k = 0; k < PT_THREADS / 64; ++k) {
          if (k < wave) pre += sh.cwave[k];
          total += sh.cwave[k];
        }
        return pre + incl - v;
      };
      uint32_t c = 0, total;
      for (uint32_t p = s_prev + 16u * (uint32_t)tid; (int64_t)p < w0; p += 16u * PT_THREADS) c += begins(p, (uint32_t)w0);
      block_scan(c, total);
      uint32_t chars = c0 - total, byte = s_prev;  // before the unit's next tokens
#pragma unroll 1
      for (uint32_t base = 0; base < inc_cnt; base += PT_THREADS) {
        const uint32_t i = base + (uint32_t)tid;
        const uint32_t len = i < inc_cnt ? len_of(w.stage[s_prev + i]) : 0u;
        uint32_t tb_all, tc_all;
        const uint32_t b = byte + block_scan(len, tb_all);
        const uint32_t e = (uint32_t)min((uint64_t)b + len, (uint64_t)n);  // (past the end: invalid input)
        uint32_t own = 0;
        for (uint32_t p = b; p < e; p += 16u) own += begins(p, e);
        const uint32_t cb = chars + block_scan(own, tc_all);
        if (i < inc_cnt && prefix + i < lim)
          spans[prefix + i] = Span{(int)b, (int)(b + len), (int)(cb - (b < e && begins(b, b + 1u) == 0u ? 1u : 0u)), (int)(cb + own)};
        byte += tb_all;
        chars += tc_all;
      }
    }
  }
#ifdef TT_PHASE_STAMPS
  __syncthreads();
  TT_PHASE(10);
#endif
}

namespace {
template <int PAT>
hipError_t launch_pat(const Work& w, const DevTables& tb, int mode, bool batch, bool ignore, hipStream_t s) {
  dim3 grid(w.n_tiles), block(PT_THREADS);
#define TT_TILE_W(B, M, I, V) return launch(tile_kernel<PAT, B, M, I, V>, grid, block, s, TileArgs{w, tb})
#define TT_TILE(B, M, I) TT_TILE_W(B, M, I, 6)
  // GPT-2- and cl100k-style encoding of one request fits 64 registers and 40 KB of
  // LDS, so a fourth block fits on a compute unit: a 16M-character corpus takes 249 us
  // instead of 305.  Where three blocks per unit already hold every tile the
  // tighter registers only cost (1M multilingual characters 44.8 -> 46.6 us, 100K
  // of prose and code 17.0 -> 18.1), so the line is at the tiles that three blocks on each of the chip's
  // 256 units hold.  A batch does not fit (registers spill to scratch memory) and
  // stays with three: 1.7M characters in 64 documents take 182 us, 199 with four
  // blocks; 16M in 512 829 and 852 (GPT-2), 1,441 and 1,426 (cl100k, whose runs
  // differ by 2 %); host to host.
  constexpr uint32_t RESIDENT_TILES = 3 * 256;
  if constexpr (PAT == TT_PATTERN_GPT2 || PAT == TT_PATTERN_CL100K) {
    if (mode == 1 && !ignore && !batch && w.n_tiles > RESIDENT_TILES) TT_TILE_W(false, 1, false, 8);
  }
  if (mode == 0) {
    if (ignore) return hipErrorInvalidValue;  // the split export has no model stage
    if (batch) TT_TILE(true, 0, false);
    else TT_TILE(false, 0, false);
  } else if (mode == 1) {
    if (batch && ignore) TT_TILE(true, 1, true);
    else if (batch) TT_TILE(true, 1, false);
    else if (ignore) TT_TILE(false, 1, true);
    else TT_TILE(false, 1, false);
  } else {
    if (batch) return hipErrorInvalidValue;  // span export is for single requests
    if (ignore) TT_TILE(false, 2, true);
    else TT_TILE(false, 2, false);
  }
#undef TT_TILE
#undef TT_TILE_W
}
}  // namespace

hipError_t launch_tile(const Work& w, const DevTables& tb, int pattern, int mode, bool ignore, hipStream_t s) {
  const bool batch = w.doc_off != nullptr;
  switch (pattern) {
    case TT_PATTERN_GPT2: return launch_pat<TT_PATTERN_GPT2>(w, tb, mode, batch, ignore, s);
    case TT_PATTERN_CL100K: return launch_pat<TT_PATTERN_CL100K>(w, tb, mode, batch, ignore, s);
    case TT_PATTERN_O200K: return launch_pat<TT_PATTERN_O200K>(w, tb, mode, batch, ignore, s);
    case TT_PATTERN_DEEPSEEK: return launch_pat<TT_PATTERN_DEEPSEEK>(w, tb, mode, batch, ignore, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace tt

#ifdef TT_PHASE_STAMPS
// The phase stamps of the first n_tiles tiles of the last call (n_tiles *
// TT_PHASE_SLOTS words, tile-major) into out (host memory).  Diagnostic build
// only; returns TT_OK, TT_ERR_BAD_ARG or TT_ERR_HIP.
extern "C" int tt_phase_stamps(unsigned long long* out, int n_tiles) {
  if (!out || n_tiles < 0 || n_tiles > tt::TT_PHASE_TILES) return TT_ERR_BAD_ARG;
  const hipError_t e = hipMemcpyFromSymbol(out, HIP_SYMBOL(tt::tt_phase_buf),
                                           (size_t)n_tiles * tt::TT_PHASE_SLOTS * sizeof(unsigned long long), 0,
                                           hipMemcpyDeviceToHost);
  return e == hipSuccess ? TT_OK : TT_ERR_HIP;
}
#endif
