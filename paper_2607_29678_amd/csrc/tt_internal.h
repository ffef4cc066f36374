// Internal definitions of the MI355X tokenizer library (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/toktier.h"
#include "tt_copy.h"

namespace tt {

// ---------------------------------------------------------------------------
// Token IDs inside the library.  Byte b is ID b and the result of the merge
// of rank r is ID 256 + r; the output stage maps them to the caller's IDs.
// A proper merge list makes this a bijection onto the IDs BPE can produce
// (every operand is a byte or an earlier result, and results are unique), and
// it lets a merge table slot hold the key and the rank in 64 bits: the result
// of a merge is implied by its rank.
// ---------------------------------------------------------------------------
constexpr uint32_t ID_BITS = 21;
constexpr uint32_t ID_LIMIT = (1u << ID_BITS) - 1u;       // internal IDs are < ID_LIMIT
constexpr uint32_t MAX_MERGES = ID_LIMIT - 256u;          // 2,096,895
constexpr uint64_t KEY_MASK = (1ull << (2 * ID_BITS)) - 1ull;
constexpr uint64_t SLOT_EMPTY = ~0ull;                    // its key is (ID_LIMIT, ID_LIMIT)
constexpr uint32_t RANK_INF = 0xFFFFFFFFu;

__host__ __device__ inline uint64_t slot_key(uint32_t a, uint32_t b) {
  return (uint64_t)a | ((uint64_t)b << ID_BITS);
}

// A value that is the same in every lane of the wave, moved to a scalar
// register (values read from LDS otherwise occupy a vector register per lane).
__device__ __forceinline__ uint32_t wave_uniform(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

// Bucket of a 32-bit hash among nb buckets: the high word of hash * nb (any
// bucket count; the high bits of a multiplicative hash are the good ones).
__host__ __device__ inline uint32_t bucket_of(uint32_t h, uint32_t nb) { return (uint32_t)(((uint64_t)h * nb) >> 32); }

// The merge table is a two-choice cuckoo table of 16-byte buckets holding
// two slots each: a pair lives in one of the two buckets its hashes name, so
// every lookup is exactly two independent 16-byte loads (one memory round
// trip, no probe chain).  Pairs of two bytes, the only pairs before any
// merge, also have a direct 64 K-entry table (PairJ).
//
// The two hashes of a pair are sums of 24-bit products (internal IDs have 21
// bits, so they cost two full-rate instructions each; a 32-bit product takes
// four times as long) and the bucket is their top bits: the bucket count is
// 2^(32 - shift), at a load of at most 0.8 (half of that where the next power of two
// is just reached, and less where a small table's pairs crowd a few buckets).
constexpr uint32_t PAIR_K[4] = {0x9E3779u, 0xC2B2AFu, 0x85EBCBu, 0xD6E8FDu};
__host__ __device__ inline uint32_t mul24(uint32_t a, uint32_t k) {
#ifdef __HIP_DEVICE_COMPILE__
  return (uint32_t)__umul24(a, k);
#else
  return a * k;  // (both below 2^24: the low 32 bits of the product)
#endif
}
__host__ __device__ inline uint32_t pair_bucket(uint32_t a, uint32_t b, uint32_t shift) {
  return (mul24(a, PAIR_K[0]) + mul24(b, PAIR_K[1])) >> shift;
}
__host__ __device__ inline uint32_t pair_bucket2(uint32_t a, uint32_t b, uint32_t shift) {
  return (mul24(a, PAIR_K[2]) + mul24(b, PAIR_K[3])) >> shift;
}

typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));

// What a byte pair (x, y) says before any merge: the rank of merging the two
// bytes, and the lowest rank among all merges across a boundary between a
// token that ends in x and one that starts with y (RANK_INF: none).
struct PairJ {
  uint32_t rank, low;
};

// Whole-unit dictionary: a unit of 3..DICT_MAX bytes whose BPE is a single
// token is found with one lookup.  An entry holds the unit's bytes (zero
// padded, little-endian words), and its length and token: (id << 4) | length.
// Two-choice cuckoo table of two entries per bucket; a unit lives in one of
// the two buckets its hashes name (four 16-byte loads, one round trip).
constexpr int DICT_MAX = 12;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__host__ __device__ inline uint32_t unit_hash(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t len) {
  uint32_t x = w0 * 0x9E3779B1u + w1 * 0x85EBCA77u + w2 * 0xC2B2AE3Du + len;
  x ^= x >> 15;
  return x * 0x2C1B3C6Du;
}
__host__ __device__ inline uint32_t unit_hash2(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t len) {
  uint32_t x = (w0 * 0x27D4EB2Fu) ^ (w1 * 0x165667B1u) ^ (w2 * 0xD3A2646Cu) ^ (len * 0xFD7046C5u);
  x ^= x >> 13;
  return x * 0x297A2D39u;
}
constexpr uint32_t DICT_NONE = 0xFFFFFFFFu;
__device__ __forceinline__ bool dict_match(const u32x4& e, uint32_t w0, uint32_t w1, uint32_t w2, uint32_t len) {
  return e.x == w0 && e.y == w1 && e.z == w2 && (e.w & 15u) == len;
}
__device__ __forceinline__ uint32_t dict_find(const u32x4* __restrict__ dict, uint32_t nb, uint32_t w0, uint32_t w1,
                                              uint32_t w2, uint32_t len) {
  const uint32_t b1 = 2u * bucket_of(unit_hash(w0, w1, w2, len), nb);
  const uint32_t b2 = 2u * bucket_of(unit_hash2(w0, w1, w2, len), nb);
  const u32x4 e0 = dict[b1], e1 = dict[b1 + 1], e2 = dict[b2], e3 = dict[b2 + 1];
  uint32_t r = DICT_NONE;
  r = dict_match(e0, w0, w1, w2, len) ? e0.w >> 4 : r;
  r = dict_match(e1, w0, w1, w2, len) ? e1.w >> 4 : r;
  r = dict_match(e2, w0, w1, w2, len) ? e2.w >> 4 : r;
  r = dict_match(e3, w0, w1, w2, len) ? e3.w >> 4 : r;
  return r;
}

// Long-unit dictionary: the same for units of DICT_MAX+1..DICT2_MAX bytes.
// An entry is two 16-byte words, {bytes 0..15} and {bytes 16..23, (id << 5) |
// length, 0}; one entry per bucket, two choices (four 16-byte loads).
constexpr int DICT2_MAX = 24;

__host__ __device__ inline uint32_t unit_hash6(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, uint32_t w4,
                                               uint32_t w5, uint32_t len) {
  uint32_t x = w0 * 0x9E3779B1u + w1 * 0x85EBCA77u + w2 * 0xC2B2AE3Du + w3 * 0x27D4EB2Fu + w4 * 0x165667B1u +
               w5 * 0xD3A2646Cu + len;
  x ^= x >> 15;
  return x * 0x2C1B3C6Du;
}
__host__ __device__ inline uint32_t unit_hash6b(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, uint32_t w4,
                                                uint32_t w5, uint32_t len) {
  uint32_t x = (w0 * 0x27D4EB2Fu) ^ (w1 * 0x165667B1u) ^ (w2 * 0xD3A2646Cu) ^ (w3 * 0xFD7046C5u) ^
               (w4 * 0xB55A4F09u) ^ (w5 * 0x9E3779B1u) ^ (len * 0x85EBCA77u);
  x ^= x >> 13;
  return x * 0x297A2D39u;
}
__device__ __forceinline__ uint32_t dict2_find(const u32x4* __restrict__ dict, uint32_t nb, const uint32_t (&w)[6],
                                               uint32_t len) {
  const uint32_t b1 = 2u * bucket_of(unit_hash6(w[0], w[1], w[2], w[3], w[4], w[5], len), nb);
  const uint32_t b2 = 2u * bucket_of(unit_hash6b(w[0], w[1], w[2], w[3], w[4], w[5], len), nb);
  const u32x4 a0 = dict[b1], a1 = dict[b1 + 1], c0 = dict[b2], c1 = dict[b2 + 1];
  uint32_t r = DICT_NONE;
  if (a0.x == w[0] && a0.y == w[1] && a0.z == w[2] && a0.w == w[3] && a1.x == w[4] && a1.y == w[5] &&
      (a1.z & 31u) == len)
    r = a1.z >> 5;
  if (c0.x == w[0] && c0.y == w[1] && c0.z == w[2] && c0.w == w[3] && c1.x == w[4] && c1.y == w[5] &&
      (c1.z & 31u) == len)
    r = c1.z >> 5;
  return r;
}

// Vocabulary strings longer than DICT2_MAX (piece probes under
// ignore_merges): one 16-byte entry {hash, length, ID, offset of the bytes in
// a blob} per bucket slot, two slots per bucket, two choices from two hashes
// of the bytes; a hit on (hash, length) is confirmed by comparing the bytes.
__host__ __device__ inline uint32_t long_hash_step(uint32_t h, uint32_t b) { return (h ^ b) * 0x01000193u; }
constexpr uint32_t LONG_SEED1 = 0x811C9DC5u, LONG_SEED2 = 0x9747B28Cu;
__host__ __device__ inline uint32_t long_hash_final(uint32_t h, uint32_t len) {
  h ^= len * 0x9E3779B1u;
  h ^= h >> 16;
  h *= 0x85EBCA6Bu;
  h ^= h >> 13;
  return h;
}

// Everything a kernel needs to know about a tokenizer handle.
struct DevTables {
  const u64x2* slots;       // cuckoo buckets of two slots: key (left | right << 21), rank in bits 42..63
  uint32_t shift;           // 32 - log2(bucket count)
  const PairJ* pairj;       // [65536] of the byte pair (x << 8 | y)
  const uint32_t* join;     // [2048] bit (x << 8 | y): some merge joins a token ending
                            // in byte x to a token starting with byte y
  const int32_t* ext_id;    // [n_ids] caller's ID of every internal ID
  uint32_t n_ids;           // 256 + M
  const u32x4* dict;        // whole-unit dictionary (two entries per bucket)
  uint32_t dnb;             // dictionary bucket count
  const u32x4* dict2;       // long-unit dictionary (one two-word entry per bucket)
  uint32_t dnb2;            // its bucket count
  const uint32_t* tok_len;  // [n_ids] byte length of every internal ID (span export)
  // ignore_merges: whole-piece probes of every vocabulary string (lowest ID)
  uint32_t vmax;            // longest vocabulary string in bytes (0: no probes)
  const u32x4* vdict;       // strings of 2..DICT_MAX bytes, whole-unit dictionary layout
  uint32_t vdnb;
  const u32x4* vdict2;      // strings of DICT_MAX+1..DICT2_MAX bytes, long-unit dictionary layout
  uint32_t vdnb2;
  const u32x4* vlong;       // longer strings: {hash, length, ID, blob offset}, two per bucket
  uint32_t vlnb;
  const uint8_t* vblob;     // bytes of the longer strings
};

// Rank of the pair (a, b), or RANK_INF if no merge joins it.  Only the high
// word of the matching slot is kept (key bits 32..41 below the rank): no empty
// slot matches, because no internal ID has all 21 bits set.  Ranks have 21
// bits, so the shift that takes the key bits off can be an arithmetic one,
// which leaves all ones (no match) as they are.
static_assert(MAX_MERGES < (1u << 21), "the sign bit of a slot's high word is free");
__device__ __forceinline__ uint32_t probe_rank(const DevTables& tb, uint32_t a, uint32_t b) {
  const u64x2* __restrict__ tab = tb.slots;
  const u64x2 x = tab[pair_bucket(a, b, tb.shift)], y = tab[pair_bucket2(a, b, tb.shift)];
  const uint32_t klo = a | (b << ID_BITS), khi = b >> (32 - ID_BITS);
  constexpr uint32_t HI_KEY = (1u << (2 * ID_BITS - 32)) - 1u;
  uint32_t hi = 0xFFFFFFFFu;
  auto check = [&](uint64_t v) {
    const uint32_t vh = (uint32_t)(v >> 32);
    hi = ((uint32_t)v == klo && (vh & HI_KEY) == khi) ? vh : hi;
  };
  check(x.x);
  check(x.y);
  check(y.x);
  check(y.y);
  return (uint32_t)((int32_t)hi >> (2 * ID_BITS - 32));
}

// ---------------------------------------------------------------------------
// Control words of a workspace.  Nothing is cleared between calls: every call
// has an epoch (1, 2, ...), words that later blocks wait on carry the epoch of
// the call that wrote them, and the tile ticket only ever grows (a call's
// tiles are tickets [ticket_base, ticket_base + n_tiles)).
// ---------------------------------------------------------------------------
struct Ctrl {
  uint32_t tile_ticket;
  uint32_t pad;
};
constexpr uint32_t EPOCH_LIMIT = 0x7FFFFFFFu;  // epochs are 1 .. EPOCH_LIMIT - 1 (31 bits)

constexpr uint32_t NO_START = 0xFFFFFFFFu;  // tile_last: no unit starts in the tile

// Buffers and parameters of one call (all device memory).
struct Work {
  const uint8_t* text;      // request bytes (caller's or staged)
  uint32_t n;               // bytes
  const int64_t* doc_off;   // batch: n_docs+1 byte offsets (no document is empty), else nullptr
  int32_t n_docs;
  const uint2* tile_docs;   // batch: [tiles] the first document at or after the first byte of the
                            // tile's padded window, and at or after the window's end
  Ctrl* ctrl;
  uint32_t epoch;           // this call's epoch
  uint32_t ticket_base;     // first tile ticket of this call
  uint32_t n_tiles;
  uint64_t* tile_sum;       // [tiles] (epoch << 32) | what the tile's last run brings into the next one
  uint64_t* tile_last;      // [tiles] (epoch << 32) | last unit start in the tile, or NO_START
  uint64_t* tile_agg;       // [tiles] output counts for the placement look-back (epoch-tagged)
  uint64_t* tile_cagg;      // [tiles] span export: non-continuation byte counts, same protocol
  uint32_t* stage;          // [n] tokens of incoming units, at the unit's first byte
  uint32_t* scratch;        // rows of units longer than ROWS_LDS bytes: 4 * n words, then n / 16 + 8 masks
  int32_t* out_spans;       // span export: [T][4] byte begin, byte end, char begin, char end
  int32_t* out_ids;         // output (caller IDs, or piece offsets for the split export)
  uint16_t* out16;          // encode without span export: when set, the IDs go here as 16-bit
                            // values instead (their low 16 bits when out_hi is set too)
  uint8_t* out_hi;          // with out16: bits 16..23 of every ID (every caller ID is below 2^24)
  int64_t* out_len;         // output length, or -error
  int64_t* out_doc_off;     // batch: n_docs+1 output offsets, the last one the total or -error
};

// Tiles and geometry --------------------------------------------------------
constexpr int PT_THREADS = 512;                   // tile block
constexpr int PT_BPT = 4;                          // bytes per thread
constexpr int PT_WIN = PT_THREADS * PT_BPT;        // window bytes in LDS
constexpr int PT_HALO = 32;                        // context bytes each side
constexpr int PT_OWN = PT_WIN - 2 * PT_HALO;       // bytes a tile decides
constexpr int PT_PAD = 8;  // LDS arrays also hold window positions [-8, 0) and [PT_WIN, PT_WIN + 16)

constexpr int SMALL_MAX = 16;                      // units listed by exact length (bytes)
constexpr int WAVE_MAX = 128;                      // longest unit that one wave encodes (bytes)
constexpr int ROWS_LDS = 480;                      // longer units: rows in LDS up to this length

inline uint32_t n_tiles_for(uint32_t n) { return (n + PT_OWN - 1) / PT_OWN; }

// Launchers (defined in the .hip files) -------------------------------------
// A launch's own status.  (The runtime's last error may be an older one that
// nobody has read: taken for the launch's, it would leave the ticket base behind
// the tickets that the tiles took, and the next call's tiles waiting for ever.)
template <class... P, class... A>
inline hipError_t launch(void (*kernel)(P...), dim3 grid, dim3 block, hipStream_t st, A... a) {
  return [&](P... p) -> hipError_t {
    void* args[] = {&p...};
    return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, args, 0, st);
  }(a...);
}
// mode 0: split export (outputs are piece byte offsets); mode 1: encode;
// mode 2: encode with span export (single requests)
// ignore: probe whole pieces in the vocabulary first (modes 1 and 2)
hipError_t launch_tile(const Work& w, const DevTables& t, int pattern, int mode, bool ignore, hipStream_t s);

// Facts of a handle for the host-side session code and the entry points
// outside tt_api.hip.
int handle_pattern(const tt_tokenizer* h);
int handle_device(const tt_tokenizer* h);
bool handle_ignore(const tt_tokenizer* h);  // ignore_merges
DevTables handle_tables(const tt_tokenizer* h);
bool handle_has_added(const tt_tokenizer* h);  // added-token literals (sessions do not take them)
uint32_t handle_max_token_bytes(const tt_tokenizer* h);  // longest token, in bytes
// Span export of a host request through the stream's pinned staging, with one
// synchronisation: on success *ids and *spans point at the T records there,
// valid (and writable) until the next call on the stream.  len <= SPANS_PINNED_MAX.
// TT_ERR_OOM when there is no pinned memory for them (tt_encode_spans then copies).
constexpr int64_t SPANS_PINNED_MAX = 1 << 22;
int encode_spans_staged(tt_tokenizer* h, const uint8_t* utf8, int64_t len, int32_t** ids, int32_t** spans, int64_t* T,
                        void* stream);

}  // namespace tt
