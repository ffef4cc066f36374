// Piece starts by the library's own rules (tt_runs.h), tile by tile, on the CPU.
//
// The rules run as they are, on a wave of 64 fibers (wave.h); what the tile
// kernel does around them (the window's bitmaps, the words tiles publish, the
// look past the window) is done here one tile after the other.  A character's
// class comes as a letter at its first byte ('.' at continuation bytes):
//   all          N number, W whitespace, S U+0020, R CR/LF
//   GPT-2, cl100k L letter, A apostrophe, O other
//   o200k        U Lu and Lt, l Ll, X Lm and Lo, M mark, A, / slash, O
//   DeepSeek     a ASCII letter, L other letter or mark, p ASCII punctuation or
//                symbol, P other ones, K k o letters, symbols and others of the
//                CJK/kana set, O other
#include "wave.h"

#include <string.h>

#include <unordered_map>

#include "tt_runs.h"

using namespace tt;

namespace {

struct Tiles {
  int pattern, n;
  const uint8_t* text;
  const char* cls;
  const uint8_t* docs;  // 1 where a document starts, or null: one text
  std::vector<uint32_t> sums;
  std::unordered_map<uint32_t, char> of;  // the class of every code point of the text
  uint64_t ops;                           // cross-lane operations of the tile that takes the most
};

void one_tile(Tiles& T, int t, uint8_t* out) {
  const int w0 = t * PT_OWN - PT_HALO, n = T.n;
  std::vector<uint8_t> buf(PT_PAD + PT_WIN + 16, 0), dst(PT_PAD + PT_WIN + 16, 0);
  for (int q = -PT_PAD; q < PT_WIN + 16; ++q)
    if (w0 + q >= 0 && w0 + q < n) {
      buf[(size_t)(PT_PAD + q)] = T.text[w0 + q];
      if (T.docs) dst[(size_t)(PT_PAD + q)] = T.docs[w0 + q];
    }
  const uint8_t* ds = T.docs ? dst.data() : nullptr;
  uint32_t starts[wave::LANES];
  T.sums.push_back(0);
  wave::run([&](int lane) {
    auto map = [&](const char* set) -> uint32_t {
      uint32_t m = 0;
      for (int k = 0; k < 32 && lane < BM_WORDS; ++k) {
        const int p = w0 + 32 * lane + k;
        if (p >= 0 && p < n && T.cls[p] != '.' && strchr(set, T.cls[p])) m |= 1u << k;
      }
      return m;
    };
    const bool first = t == 0;
    RunBits b{};
    b.N = map("N");
    b.WS = map("WS");
    b.NL = map("R");
    b.SP = map("S");
    b.D = 0;
    if (T.docs) {
      for (int k = 0; k < 32 && lane < BM_WORDS; ++k) {
        const int p = w0 + 32 * lane + k;
        if (p >= 0 && p < n && T.docs[p]) b.D |= 1u << k;
      }
    } else if (first && lane == PT_HALO / 32) {
      b.D = 1u;
    }
    b.C = b.N | b.WS | b.NL;
    O2Maps m2{};
    DsMaps md{};
    if (T.pattern == TT_PATTERN_O200K) {
      m2 = O2Maps{map("U"), map("l"), map("X"), map("M"), map("A"), map("/")};
      b.O = map("OA/");
      b.C |= b.O | m2.U | m2.Lo | m2.X | m2.M;
    } else if (T.pattern == TT_PATTERN_DEEPSEEK) {
      md = DsMaps{map("a"), map("L"), map("p"), map("P"), map("O"), map("K"), map("k"), map("o")};
      b.C |= md.AL | md.L | md.AP | md.PS | md.O | md.KL | md.KP | md.KO;
    } else {
      b.L = map("L");
      b.O = map("OA");
      b.APO = map("A");
      b.C |= b.L | b.O;
    }
    const int in_end = std::min(n - w0, PT_WIN);
    b.K = bm_range(first ? PT_HALO : 0, in_end, lane) & ~b.C;
    b.multi = __ballot(b.K != 0u) != 0ull;
    const uint32_t own = bm_range(PT_HALO, std::min(in_end, PT_HALO + PT_OWN), lane);
    auto publish = [&](uint32_t sum) { T.sums[(size_t)t] = sum; };
    auto carry = [&](uint32_t ask) -> RunCarry {  // (as the tile kernel's)
      uint32_t acc = 0, val = 0, open = ask;
      for (int j = t - 1; j >= 0 && open != 0u; --j) {
        const uint32_t v = T.sums[(size_t)j];
        if (open & SUM_N_ALL) acc += (v >> 1) & 3u;
        const uint32_t now = open & ~v;
        if (now & SUM_TAIL_ALL) val |= v & SUM_TAIL;
        if (now & SUM_STATE_ALL) val |= v & (15u << SUM_STATE_SHIFT);
        open &= ~now;
      }
      return RunCarry{acc % 3u, (val & SUM_TAIL) != 0u, (val >> SUM_STATE_SHIFT) & 15u};
    };
    auto beyond = [&](auto plain, const char* set) -> uint32_t {
      const int at = w0 + PT_WIN;
      if (at >= n) return ~0u;
      int end = n;
      for (int p = at; T.docs && p < end; ++p)
        if (T.docs[p]) end = p;
      return first_outside(T.text + at, (uint32_t)(end - at), lane, plain,
                           [&](uint32_t c) { return strchr(set, (int)c) != nullptr; },
                           [&](uint32_t cp) { return (uint32_t)T.of.at(cp); });
    };
    auto last_ws = [&]() -> bool {
      return beyond([](uint32_t c) { return c == 0x20u || c == 0x09u || c == 0x0Bu || c == 0x0Cu; }, "WS") != 'R';
    };
    auto upper = [&]() -> bool {
      const uint32_t c = beyond([](uint32_t x) { return x - 'A' < 26u; }, "U");
      return c == 'l' || c == 'X' || c == 'M';
    };
    uint32_t st = 0;
    switch (T.pattern) {
      case TT_PATTERN_GPT2: st = gpt2_starts(b, buf.data(), ds, lane); break;
      case TT_PATTERN_CL100K: st = cl100k_starts(b, own, buf.data(), ds, lane, first, publish, carry, last_ws); break;
      case TT_PATTERN_O200K:
        st = o200k_starts(b, m2, own, buf.data(), ds, lane, first, publish, carry, last_ws, upper);
        break;
      default: st = deepseek_starts(b, md, own, lane, first, publish, carry, last_ws);
    }
    starts[lane] = st & own;
  });
  T.ops = std::max(T.ops, wave::count[0]);
  for (int q = PT_HALO; q < PT_HALO + PT_OWN && w0 + q < n; ++q)
    out[w0 + q] = (starts[q >> 5] >> (q & 31)) & 1u;
}

}  // namespace

// The bytes a tile owns.
extern "C" int run_rules_own() { return PT_OWN; }

// out[p] = 1 where a piece starts; returns the cross-lane operations of the tile
// that takes the most.
extern "C" uint64_t run_rules(int pattern, const uint8_t* text, const char* cls, int n, const uint8_t* docs, uint8_t* out) {
  Tiles T{pattern, n, text, cls, docs, {}, {}, 0};
  for (int p = 0; p < n; ++p)
    if (cls[p] != '.') {
      auto at = [&](int k) -> uint32_t { return p + k < n ? text[p + k] : 0u; };
      uint32_t cp;
      decode_sel(at(0), at(1), at(2), at(3), 4u, cp);
      T.of[cp] = cls[p];
    }
  for (int t = 0; t * PT_OWN < n; ++t) one_tile(T, t, out);
  return T.ops;
}
