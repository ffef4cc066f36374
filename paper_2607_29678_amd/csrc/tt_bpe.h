// Exact byte-level BPE of one unit (a piece, or a segment of a piece that no
// merge can cross), on the GPU.
//
// A unit starts as the IDs of its bytes; the adjacent pair with the lowest
// merge rank is merged, leftmost first, until no pair has a rank (the model
// stage of the front-end/model factorisation, Appendix, Definition
// d:frontend and Lemma l:homo).  Two facts license the parallel schedules
// below (Sec. 4.2, "GPU BPE"): with a proper merge list, merging all leftmost
// non-overlapping occurrences of the round's lowest-ranked pair at once equals
// merging them one by one, and after a merge only the pairs that touch the new
// token need a new rank lookup.  The unit length picks the execution unit
// (Sec. 4.2 dispatches by piece length):
//   bpe_lanes   <= 64 bytes:  one wave64 holds 8 units of <= 8 bytes, 4 of <= 16,
//                             2 of <= 32 or one of <= 64, one byte per lane;
//   bpe_wave2   <= 128 bytes: one wave64, two tokens per lane;
//   bpe_rows    longer:       NW waves over rows of 64 tokens in LDS or global
//                             memory.
// IDs are internal: byte b is b, the result of merge r is 256 + r.
#pragma once

#include "tt_internal.h"

namespace tt {

constexpr uint32_t RANK_DIRTY = 0xFFFFFFFEu;  // pair changed; its rank must be looked up again

// Leftmost non-overlapping choice among the set bits of m, where bit j stands
// for the pair (token j, token j+1).  Two chosen pairs may not share a token,
// so within every run of consecutive set bits the left-to-right greedy choice
// takes the run's first bit and every second bit after it.  Runs that start on
// an even bit are isolated with one carry propagation: adding their start bits
// clears exactly those runs.
__device__ __forceinline__ uint64_t leftmost_nonoverlapping(uint64_t m) {
  const uint64_t EVEN = 0x5555555555555555ull;
  const uint64_t starts = m & ~(m << 1);
  const uint64_t even_runs = ((m + (starts & EVEN)) ^ m) & m;
  return (even_runs & EVEN) | (m & ~even_runs & ~EVEN);
}

// Number of set bits of m below the calling lane.
__device__ __forceinline__ uint32_t bits_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Minimum over the 64 lanes of a wave, in every lane (DPP row steps, then
// the row broadcasts; the full result ends in lane 63).
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
  int x = (int)v;
  x = (int)min((uint32_t)x, (uint32_t)__builtin_amdgcn_update_dpp(x, x, 0xB1, 0xF, 0xF, false));   // quad_perm 1,0,3,2
  x = (int)min((uint32_t)x, (uint32_t)__builtin_amdgcn_update_dpp(x, x, 0x4E, 0xF, 0xF, false));   // quad_perm 2,3,0,1
  x = (int)min((uint32_t)x, (uint32_t)__builtin_amdgcn_update_dpp(x, x, 0x141, 0xF, 0xF, false));  // row_half_mirror
  x = (int)min((uint32_t)x, (uint32_t)__builtin_amdgcn_update_dpp(x, x, 0x140, 0xF, 0xF, false));  // row_mirror
  x = (int)min((uint32_t)x, (uint32_t)__builtin_amdgcn_update_dpp(x, x, 0x142, 0xA, 0xF, false));  // row_bcast15
  x = (int)min((uint32_t)x, (uint32_t)__builtin_amdgcn_update_dpp(x, x, 0x143, 0xC, 0xF, false));  // row_bcast31
  return (uint32_t)__builtin_amdgcn_readlane(x, 63);
}

// Inclusive sum over the lanes of a wave (DPP: shifts within rows of 16
// lanes, then the row broadcasts carry row totals forward).
__device__ __forceinline__ uint32_t wave_incl_sum(uint32_t v) {
  int x = (int)v;
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false); // row_bcast:15 into rows 1, 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false); // row_bcast:31 into rows 2, 3
  return (uint32_t)x;
}

// ---------------------------------------------------------------------------
// Units of at most 64 bytes: 64 / W units on one wave64, W lanes per unit (W is
// 8, 16, 32 or 64, the same for the whole wave), one byte position per lane.
//
// A token stays at the lane of its first byte and the lanes of its other bytes
// are dead, so a round moves no token: a merge changes the left token's ID and
// clears the right token's bit in the wave's alive mask (a scalar), and every
// lane finds the tokens after it from that mask.  Lane i holds the rank of the
// pair (token i, next token).
//
// Which pairs a round merges.  Merging only the lowest rank of the unit makes
// the number of rounds the number of different ranks (14 on average for units
// of 17..32 bytes of multilingual text).  But no merge ever crosses the byte
// boundary (x, y) with a rank below J(x, y), the lowest rank among the merges
// whose left operand ends in x and whose right operand starts with y
// (DevTables::pairj).  So when a pair's rank r is below J at the boundary before
// its left token and below J at the boundary after its right one, its two
// tokens are cut off from the rest of the unit until rank r is reached: they
// merge with each other then, whatever happens elsewhere before, and merging
// them now gives the same result.  A round merges all such pairs and the
// occurrences of the unit's lowest rank (leftmost first, without overlap).
// Two pairs taken in one round never share a token unless they are occurrences
// of the lowest rank: J at the boundary inside a pair is at most its rank.
// Rounds per unit, multilingual text: 13.7 -> 6.1 (17..32 bytes), 9.9 -> 5.0
// (13..16), 6.8 -> 4.1 (9..12); agent transcript: 17.0 -> 9.4, 11.8 -> 6.5,
// 7.7 -> 4.4.  A round is bound by instruction issue when every wave of
// a compute unit is in this loop (five waves per SIMD at four cycles an
// instruction), else by latency: one L2 round trip for the rank lookups.
// Engine phase of a tile, mean / slowest, against one thread per unit of 3..16
// bytes and one or two units per wave merging lowest ranks only: 1M-character
// agent transcript 8.4 / 19.5 -> 4.4 / 10.8 us, multilingual 14.7 / 29.6 ->
// 9.9 / 20.7 us; a 16M-character corpus 414 -> 351 us (whole calls).
//
// L is the length of the calling lane's unit (0: none), byte the byte at the
// lane's position in it.  On return id is the token at the calling lane's
// position if the lane is set in the returned mask.  Every lane of the wave
// calls it.
// ---------------------------------------------------------------------------

// Minimum over the W lanes of the calling lane's group, in every lane of it.
__device__ __forceinline__ uint32_t group_min_u32(uint32_t v, uint32_t W) {
  // (an old value of all ones is the identity of the minimum, which lets the
  // lane move fuse with it)
#define TT_MIN_DPP(ctrl) v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, ctrl, 0xF, 0xF, false))
  TT_MIN_DPP(0xB1);   // quad_perm 1,0,3,2
  TT_MIN_DPP(0x4E);   // quad_perm 2,3,0,1
  TT_MIN_DPP(0x141);  // row_half_mirror
  if (W > 8u) TT_MIN_DPP(0x140);  // row_mirror
#undef TT_MIN_DPP
  if (W > 16u) {  // rows 0 and 1, rows 2 and 3
    const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = min((uint32_t)p[0], (uint32_t)p[1]);
  }
  if (W > 32u) {  // the two halves
    const auto p = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    v = min((uint32_t)p[0], (uint32_t)p[1]);
  }
  return v;
}

// Trailing zeros, all ones for zero (one instruction).
__device__ __forceinline__ uint32_t ffbl(uint32_t x) { return (uint32_t)__builtin_ffs((int)x) - 1u; }

// WIDE: W is 64 (a unit spans both halves of the wave); else a unit lies in
// one half, and the masks a lane looks at are one word.
template <bool WIDE>
__device__ __forceinline__ uint64_t bpe_lanes(uint32_t W, uint32_t L, uint32_t byte, const DevTables& tb,
                                              uint32_t& id) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t j = lane & (W - 1u);  // byte position in the unit
  const uint32_t half = lane & 32u;
  // the unit's lanes after this one, as a mask of the wave (WIDE) or of the half
  const uint64_t above64 = ~((2ull << lane) - 1ull);
  const uint32_t h = lane & 31u;
  const uint32_t above = (W >= 32u ? ~0u : (((1u << W) - 1u) << (h - j))) & ~((2u << h) - 1u);
  id = byte;
  uint32_t rk = RANK_INF, jr = RANK_INF;  // J at the boundary after this byte
  {
    const uint32_t idn = (uint32_t)__builtin_amdgcn_ds_bpermute((int)((lane + 1u) << 2), (int)id);
    if (j + 1u < L) {
      const PairJ e = tb.pairj[(id << 8) | idn];
      rk = e.rank;
      jr = e.low;
    }
  }
  const uint32_t jl = (uint32_t)__builtin_amdgcn_ds_bpermute((int)((lane + 63u) << 2), (int)jr);
  const uint32_t bl = j == 0u ? RANK_INF : jl;  // J at the boundary before this byte
  // the lower of the two bounds of the pair that starts here
  uint32_t bd = bl;
  {
    const uint32_t b2 = (uint32_t)__builtin_amdgcn_ds_bpermute((int)((lane + 2u) << 2), (int)bl);
    if (j + 2u < L) bd = min(bd, b2);
  }
  uint64_t alive = __ballot(j < L);
  for (;;) {
    const uint32_t m = group_min_u32(rk, W);
    if (__ballot(m != RANK_INF) == 0ull) break;
    uint64_t sel = __ballot(rk < bd) | (__ballot(rk == m) & __ballot(rk != RANK_INF));
    // the token after each chosen one: adding at the position above it carries
    // through the dead lanes up to the next live one
    uint64_t nx = ((sel << 1) + ~alive) & alive;
    if (nx & sel) {
      // overlapping occurrences (a run of one token): every second one from
      // the start of the run; the tokens of a run are equally long
      const uint64_t upto = sel & ~nx & ((2ull << lane) - 1ull);
      const uint32_t s = upto ? 63u - (uint32_t)__builtin_clzll(upto) : lane;
      const uint64_t x = alive & above64;
      const uint32_t span = x ? (uint32_t)__builtin_ctzll(x) - lane : 1u;
      const bool odd = (((lane - s) / span) & 1u) != 0u;
      sel &= ~(nx & __ballot(odd));
      nx = ((sel << 1) + ~alive) & alive;
    }
    alive &= ~nx;
    const bool me_sel = __builtin_amdgcn_inverse_ballot_w64(sel);
    id = me_sel ? 256u + rk : id;
    // the next two live tokens of the unit, and whether the next one merged
    uint32_t n1, n2;
    bool has1, has2, nsel;
    if (WIDE) {
      const uint64_t x1 = alive & above64, x2 = x1 & (x1 - 1ull);
      has1 = x1 != 0ull;
      has2 = x2 != 0ull;
      n1 = has1 ? (uint32_t)__builtin_ctzll(x1) : lane;
      n2 = has2 ? (uint32_t)__builtin_ctzll(x2) : lane;
      nsel = (sel >> n1) & 1ull;
    } else {
      const uint32_t ah = half ? (uint32_t)(alive >> 32) : (uint32_t)alive;
      const uint32_t sh = half ? (uint32_t)(sel >> 32) : (uint32_t)sel;
      const uint32_t x1 = ah & above, x2 = x1 & (x1 - 1u);
      has1 = x1 != 0u;
      has2 = x2 != 0u;
      n1 = ffbl(x1);  // (all ones for none: the permutes and the shift take it modulo 32)
      n2 = ffbl(x2);
      nsel = (sh >> (n1 & 31u)) & 1u;
      n1 = (n1 & 31u) | half;
      n2 = (n2 & 31u) | half;
    }
    const uint32_t idn = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(n1 << 2), (int)id);
    const uint32_t b2 = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(n2 << 2), (int)bl);
    bd = has2 ? min(bl, b2) : bl;
    const bool pair = __builtin_amdgcn_inverse_ballot_w64(alive) && has1;
    rk = pair ? rk : RANK_INF;
    if (pair && (me_sel || nsel)) rk = probe_rank(tb, id, idn);
  }
  return alive;
}

// ---------------------------------------------------------------------------
// One wave64, at most 128 bytes: lane i holds tokens i and 64 + i and the
// ranks of the pairs starting there.  A round merges the lowest rank over
// a 128-bit occurrence mask (the choice in the second row continues the
// alternation of a run that crosses from the first, through the carry of the
// first row's last bit); the survivors are compacted through the wave's own
// 256 words of LDS `scr` (token IDs, then ranks), written and read back by the
// same wave.  Every lane of the wave calls it with the same arguments.
// ---------------------------------------------------------------------------
template <class ByteF, class OutF>
__device__ __forceinline__ uint32_t bpe_wave2(uint32_t L, ByteF byte, const DevTables& tb, uint32_t* scr, OutF out) {
  const int lane = (int)(threadIdx.x & 63u);
  const uint32_t l0 = (uint32_t)lane, l1 = 64u + (uint32_t)lane;
  uint32_t n = L;  // <= 128
  uint32_t id0 = l0 < n ? byte(lane) : 0u;
  uint32_t id1 = l1 < n ? byte(64 + lane) : 0u;
  auto next0 = [&]() -> uint32_t {  // token after position lane (row 0)
    const uint32_t nx = (uint32_t)__shfl_down((int)id0, 1, 64);
    const uint32_t head1 = (uint32_t)__builtin_amdgcn_readlane((int)id1, 0);
    return lane == 63 ? head1 : nx;
  };
  uint32_t nx0 = next0(), nx1 = (uint32_t)__shfl_down((int)id1, 1, 64);
  uint32_t rk0 = l0 + 1u < n ? tb.pairj[(id0 << 8) | nx0].rank : RANK_INF;
  uint32_t rk1 = l1 + 1u < n ? tb.pairj[(id1 << 8) | nx1].rank : RANK_INF;
  for (;;) {
    const uint32_t m = wave_min_u32(min(rk0, rk1));
    if (m == RANK_INF) break;
    const uint64_t s0 = leftmost_nonoverlapping(__ballot(rk0 == m));
    const uint64_t c = s0 >> 63;  // the pair (63, 64) is chosen: token 64 is taken
    const uint64_t s1 = leftmost_nonoverlapping(__ballot(rk1 == m) & ~c);
    const uint64_t v0 = n >= 64u ? ~0ull : ((1ull << n) - 1ull);
    const uint64_t v1 = n >= 128u ? ~0ull : (n > 64u ? ((1ull << (n - 64u)) - 1ull) : 0ull);
    const uint64_t k0 = v0 & ~(s0 << 1), k1 = v1 & ~((s1 << 1) | c);
    const bool me0 = (s0 >> lane) & 1ull, me1 = (s1 >> lane) & 1ull;
    const bool nxs0 = lane < 63 ? ((s0 >> (lane + 1)) & 1ull) != 0ull : (s1 & 1ull) != 0ull;
    const bool nxs1 = lane < 63 && ((s1 >> (lane + 1)) & 1ull) != 0ull;
    const uint32_t c0 = (uint32_t)__popcll(k0);
    if ((k0 >> lane) & 1ull) {
      const uint32_t p = bits_below(k0);
      scr[p] = me0 ? 256u + m : id0;
      scr[128 + p] = (me0 || nxs0) ? RANK_DIRTY : rk0;
    }
    if ((k1 >> lane) & 1ull) {
      const uint32_t p = c0 + bits_below(k1);
      scr[p] = me1 ? 256u + m : id1;
      scr[128 + p] = (me1 || nxs1) ? RANK_DIRTY : rk1;
    }
    n = c0 + (uint32_t)__popcll(k1);
    // (one wave writes and reads its own words: LDS operations of a wave are
    // performed in order)
    id0 = l0 < n ? scr[l0] : 0u;
    const uint32_t r0 = l0 < n ? scr[128 + l0] : RANK_INF;
    id1 = l1 < n ? scr[l1] : 0u;
    const uint32_t r1 = l1 < n ? scr[128 + l1] : RANK_INF;
    nx0 = next0();
    nx1 = (uint32_t)__shfl_down((int)id1, 1, 64);
    rk0 = r0;
    if (r0 == RANK_DIRTY) rk0 = l0 + 1u < n ? probe_rank(tb, id0, nx0) : RANK_INF;
    rk1 = r1;
    if (r1 == RANK_DIRTY) rk1 = l1 + 1u < n ? probe_rank(tb, id1, nx1) : RANK_INF;
  }
  if (l0 < n) out(lane, id0);
  if (l1 < n) out(64 + lane, id1);
  return n;
}

// ---------------------------------------------------------------------------
// Longer units: NW waves over rows of 64 tokens.  T holds two buffers of
// `stride` >= L tokens and `sel` one selection mask per row; they may live in LDS
// or in global memory (visible to the whole block).  Every thread of the block
// calls it with the same arguments.
//
// A token is one word: ID, rank of the pair it starts and J at the byte
// boundary before it (21 bits each, see bpe_lanes for J and for the pairs a
// round merges).  Each wave owns a range of rows and a round reads them twice:
// first the choice among the pairs and the number of tokens left, then, with the
// counts of the waves before it known, the merged tokens with the ranks of their
// new pairs and the next round's lowest rank.  How the choice in a wave's rows
// depends on the wave before (an occurrence at its end) only matters to the run
// of occurrences the rows begin with: its choice shifts by one.
// One block works while later tiles wait for its count, so a round is bound by
// the latency of a row's loads and by the instructions of eight waves: rows are
// taken a few at a time with their loads and rank lookups in flight together
// (two where the ranks are looked up: more would spill registers in the kernel of
// four blocks per compute unit), and rows with no merge are only moved.
// Merging lowest ranks only, with IDs and ranks apart and one load in flight,
// 25,013 bytes of one repeated letter took 12 rounds and 576 us among the tiles of
// a 3.8 MB request (kernel 662 us; another such request 292); now 8 rounds and 168
// us (265; 200).
// ---------------------------------------------------------------------------
template <int NW>
struct RowsShared {
  uint32_t wmin[NW];
  // per wave: tokens its rows keep, and whether their last pair is chosen, if the
  // last pair before them is not chosen (k0) or is (k1); occurrences they begin with
  uint32_t k0[NW], k1[NW], pre[NW];
};

constexpr uint32_t ROW_INF = (1u << ID_BITS) - 1u;  // no rank, in a row token
static_assert(MAX_MERGES <= ROW_INF, "ranks of row tokens are below ROW_INF");

struct RowTok {
  uint64_t v;
  __device__ __forceinline__ static RowTok make(uint32_t id, uint32_t rk, uint32_t bl) {
    return {(uint64_t)(id | (rk << ID_BITS)) | (uint64_t)((rk >> (32 - ID_BITS)) | (bl << (2 * ID_BITS - 32))) << 32};
  }
  __device__ __forceinline__ uint32_t id() const { return (uint32_t)v & ROW_INF; }
  __device__ __forceinline__ uint32_t rk() const { return (uint32_t)(v >> ID_BITS) & ROW_INF; }
  __device__ __forceinline__ uint32_t bl() const { return (uint32_t)(v >> 32) >> (2 * ID_BITS - 32); }
};

template <int NW, class OutF>
__device__ __forceinline__ uint32_t bpe_rows(uint32_t L, const uint8_t* src, const DevTables& tb, uint64_t* T,
                                             uint64_t stride, uint64_t* sel, RowsShared<NW>& sm, OutF out) {
  const uint32_t tid = threadIdx.x;
  const uint32_t lane = tid & 63u;
  const uint32_t wave = wave_uniform(tid >> 6);
  constexpr uint32_t NT = NW * 64, B = 2, C = 4;  // rows in flight with rank lookups, and without
  const uint32_t cap = ROW_INF;
  uint32_t n = L;
  uint32_t cur = 0;

  uint32_t m = ROW_INF;
  for (uint32_t i0 = tid; i0 < n; i0 += NT * C) {
    uint32_t b[C], bp[C], bn[C];
#pragma unroll
    for (uint32_t k = 0; k < C; ++k) {
      const uint32_t i = min(i0 + k * NT, n - 1u);
      b[k] = src[i];
      bp[k] = src[i ? i - 1u : 0u];
      bn[k] = src[min(i + 1u, n - 1u)];
    }
    uint32_t rk[C], bl[C];
#pragma unroll
    for (uint32_t k = 0; k < C; ++k) {
      rk[k] = tb.pairj[(b[k] << 8) | bn[k]].rank;
      bl[k] = tb.pairj[(bp[k] << 8) | b[k]].low;
    }
#pragma unroll
    for (uint32_t k = 0; k < C; ++k) {
      const uint32_t i = i0 + k * NT;
      const uint32_t r = i + 1u < n ? min(rk[k], cap) : cap;
      if (i < n) T[i] = RowTok::make(b[k], r, i ? min(bl[k], cap) : cap).v;
      m = min(m, r);
    }
  }

  for (;;) {
    m = wave_min_u32(m);
    if (lane == 0) sm.wmin[wave] = m;
    __syncthreads();  // (and the tokens are written)
    for (int v = 0; v < NW; ++v) m = min(m, sm.wmin[v]);
    m = wave_uniform(m);
    if (m == cap) break;
    const uint64_t* A = T + (cur ? stride : 0u);
    uint64_t* A2 = T + (cur ? 0u : stride);

    // 1. the choice, as if the last pair before the wave's rows were not chosen
    const uint32_t rows = (n + 63u) / 64u;
    const uint32_t rpw = (rows + NW - 1u) / NW;
    const uint32_t r_lo = min(rows, wave * rpw), r_hi = min(rows, r_lo + rpw);
    const uint32_t toks = min(n, r_hi * 64u) - min(n, r_lo * 64u);
    uint32_t carry = 0, chosen = 0, pre = 0;
    bool in_pre = true;
    for (uint32_t r0 = r_lo; r0 < r_hi; r0 += C) {
      RowTok t[C], t2[C];
#pragma unroll
      for (uint32_t k = 0; k < C; ++k) {
        const uint32_t i = (r0 + k) * 64u + lane;
        t[k].v = A[min(i, n - 1u)];
        t2[k].v = A[min(i + 2u, n - 1u)];
      }
#pragma unroll
      for (uint32_t k = 0; k < C; ++k) {
        if (r0 + k < r_hi) {
          const uint32_t i = (r0 + k) * 64u + lane;
          const uint32_t rk = i + 1u < n ? t[k].rk() : cap;
          const uint32_t bd = i + 2u < n ? min(t[k].bl(), t2[k].bl()) : t[k].bl();
          const uint64_t occ = __ballot(rk == m);
          const uint64_t s = leftmost_nonoverlapping(occ & ~(uint64_t)carry) | (__ballot(rk < bd) & ~occ);
          if (lane == 0) sel[r0 + k] = s;
          chosen += (uint32_t)__popcll(s);
          carry = (uint32_t)(s >> 63);
          if (in_pre) {
            pre += ~occ ? (uint32_t)__builtin_ctzll(~occ) : 64u;
            in_pre = ~occ == 0ull;
          }
        }
      }
    }
    if (lane == 0) {
      // a run that fills the rows carries the shift to their last pair
      const uint32_t chosen1 = chosen - (pre & 1u), carry1 = in_pre ? carry ^ 1u : carry;
      sm.k0[wave] = ((toks - (chosen - carry)) << 1) | carry;
      sm.k1[wave] = ((toks - 1u - (chosen1 - carry1)) << 1) | carry1;
      sm.pre[wave] = pre;
    }
    __syncthreads();
    uint32_t base = 0, n2 = 0, c_in = 0, c_next = 0, pre_next = 0;
    {
      uint32_t c = 0;
      for (uint32_t v = 0; v < NW; ++v) {
        if (v == wave) {
          c_in = c;
          base = n2;
        }
        if (v == wave + 1u) {
          c_next = c;
          pre_next = sm.pre[v];
        }
        if (v * rpw >= rows) continue;  // no rows
        const uint32_t x = c ? sm.k1[v] : sm.k0[v];
        n2 += x >> 1;
        c = x & 1u;
      }
    }
    c_in = wave_uniform(c_in);
    c_next = wave_uniform(c_next);
    base = wave_uniform(base);
    pre_next = wave_uniform(pre_next);
    pre = c_in ? pre : 0u;
    pre_next = c_next ? pre_next : 0u;

    // 2. the tokens after the round
    m = cap;
    carry = c_in;
    for (uint32_t r0 = r_lo; r0 < r_hi; r0 += B) {
      // the masks of the rows and of the one after them, with the shift of the
      // run the wave's rows (or the next wave's) begin with
      uint64_t ms = 0;
      if (lane <= B && r0 + lane < rows) {
        const uint32_t r = r0 + lane;
        ms = sel[r];
        const uint32_t off = r < r_hi ? (r - r_lo) * 64u : 0u, p = r < r_hi ? pre : pre_next;
        const uint32_t k = p > off ? p - off : 0u;
        ms ^= k >= 64u ? ~0ull : ((1ull << k) - 1ull);
      }
      uint64_t s[B + 1];
#pragma unroll
      for (uint32_t k = 0; k <= B; ++k)
        s[k] = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)ms, (int)k) |
               (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(ms >> 32), (int)k) << 32;
      if ((s[0] | s[1] | (s[2] & 3ull) | (uint64_t)carry) == 0ull && (r0 + 2u) * 64u < n && r0 + 1u < r_hi) {
        // nothing merges in or next to two full rows: they move as they are
        RowTok x[2];
#pragma unroll
        for (uint32_t k = 0; k < 2u; ++k) x[k].v = A[(r0 + k) * 64u + lane];
#pragma unroll
        for (uint32_t k = 0; k < 2u; ++k) {
          A2[base + k * 64u + lane] = x[k].v;
          m = min(m, x[k].rk());
        }
        base += 128u;
        continue;
      }
      RowTok t[B], t1[B];
#pragma unroll
      for (uint32_t k = 0; k < B; ++k) {
        const uint32_t i = (r0 + k) * 64u + lane;
        t[k].v = A[min(i, n - 1u)];
        t1[k].v = A[min(i + 1u + (uint32_t)((s[k] >> lane) & 1u), n - 1u)];
      }
      uint32_t id[B], rk[B];
      bool kept[B], dirty[B];
      bool any = false;
#pragma unroll
      for (uint32_t k = 0; k < B; ++k) {
        const uint32_t i = (r0 + k) * 64u + lane;
        const bool in = r0 + k < r_hi && i < n;
        const bool me = (s[k] >> lane) & 1ull;
        const uint64_t keep = ~((s[k] << 1) | (uint64_t)carry);
        if (r0 + k < r_hi) carry = (uint32_t)(s[k] >> 63);
        kept[k] = in && ((keep >> lane) & 1ull);
        // the next token after the round starts at i1; is it a merged one too?
        const uint32_t i1 = i + 1u + (me ? 1u : 0u);
        const uint32_t d = lane + 1u + (me ? 1u : 0u);
        const bool nx = d < 64u ? (s[k] >> d) & 1ull : (s[k + 1] >> (d - 64u)) & 1ull;
        const bool pair = i1 < n;
        id[k] = me ? 256u + t[k].rk() : t[k].id();
        dirty[k] = kept[k] && pair && (me || nx);
        rk[k] = pair ? t[k].rk() : cap;
        any = any || dirty[k];
        t1[k].v = nx ? 256u + t1[k].rk() : t1[k].id();
      }
      if (__ballot(any)) {
        uint32_t q[B];
#pragma unroll
        for (uint32_t k = 0; k < B; ++k) q[k] = probe_rank(tb, dirty[k] ? id[k] : 0u, dirty[k] ? (uint32_t)t1[k].v : 0u);
#pragma unroll
        for (uint32_t k = 0; k < B; ++k) rk[k] = dirty[k] ? min(q[k], cap) : rk[k];
      }
#pragma unroll
      for (uint32_t k = 0; k < B; ++k) {
        const uint64_t kp = __ballot(kept[k]);
        if (kept[k]) {
          A2[base + bits_below(kp)] = RowTok::make(id[k], rk[k], t[k].bl()).v;
          m = min(m, rk[k]);
        }
        base += (uint32_t)__popcll(kp);
      }
    }
    n = wave_uniform(n2);
    cur ^= 1u;
  }
  const uint64_t* A = T + (cur ? stride : 0u);
  for (uint32_t i0 = tid; i0 < n; i0 += NT * C) {
    uint32_t id[C];
#pragma unroll
    for (uint32_t k = 0; k < C; ++k) id[k] = RowTok{A[min(i0 + k * NT, n - 1u)]}.id();
#pragma unroll
    for (uint32_t k = 0; k < C; ++k)
      if (i0 + k * NT < n) out(i0 + k * NT, id[k]);
  }
  return n;
}

}  // namespace tt
