// The o200k-style pattern (Sec. 4.1: the o200k lineage adds a case-boundary
// rule and treats Unicode marks specially).  Its alternatives, in order:
//   P1  [^\r\n\p{L}\p{N}]? [Lu Lt Lm Lo M]* [Ll Lm Lo M]+ CT?
//   P2  [^\r\n\p{L}\p{N}]? [Lu Lt Lm Lo M]+ [Ll Lm Lo M]* CT?
//   P3  \p{N}{1,3}
//   P4  U+0020? [^\s\p{L}\p{N}]+ [\r\n/]*
//   P5  \s*[\r\n]+      P6  \s+(?!\S)      P7  \s+
// where CT is the case-insensitive contraction 's 't 're 've 'm 'll 'd.
//
// Here are its classes and the positions where it resets for every left
// context (the synchronizing transitions, which certify splices in incremental
// repair); the tile kernel's rules are in tt_runs.h.
#pragma once

#include "tt_internal.h"

namespace tt {

// Classes of the o200k-style pattern (4 bits of a window code).
enum : uint32_t {
  O2_O = 0,    // other
  O2_UP = 1,   // Lu, Lt: only in the upper-case letter set
  O2_LO = 2,   // Ll: only in the lower-case letter set
  O2_BO = 3,   // Lm, Lo: in both letter sets
  O2_MK = 4,   // M: in both letter sets and in the "not letter, not number" sets
  O2_N = 5,    // \p{N}
  O2_WS = 6,   // \s except CR and LF
  O2_NL = 7,   // CR, LF
  O2_NONE = 15 // continuation byte, or outside the text
};

__host__ __device__ constexpr bool o2_letter(uint32_t c) { return c == O2_UP || c == O2_LO || c == O2_BO; }

// Class of a code point from the probed 4-bit table (levels l1, l2; host
// arrays, or the copy a block keeps in LDS).
template <class P>
__host__ __device__ inline uint32_t o2_table_class(P l1, P l2, uint32_t cp) {
  if (cp == 10u || cp == 13u) return O2_NL;
  const uint32_t blk = l1[cp >> 8];
  const uint32_t v = (l2[blk * 128u + ((cp & 255u) >> 1)] >> ((cp & 1u) * 4u)) & 15u;
  // table values: 0 other, 1 Lu|Lt, 2 Ll, 3 Lm|Lo, 4 M, 5 N, 6 \s
  return v;
}

// Whether a position whose left character has class x (code point cx) and
// whose right character has class y (code point cy) is a synchronizing
// boundary of the o200k-style pattern: every text with these two characters
// there has a piece boundary between them, the pieces to the right depend on
// the left only through x, and the pieces to the left depend on the right
// only through y.  From the alternatives:
//   - a number run head always starts a piece (no set before it takes digits);
//   - a letter is safe after a number or CR/LF (neither can be a prefix), and
//     an upper-case letter after a lower-case one (a lower-case character is
//     only ever matched by the lower-case part of a piece, which ends at the
//     next upper-case letter);
//   - whitespace other than CR/LF is safe after letters, marks, numbers and
//     symbols (no set before it takes it, and it only begins pieces);
//   - CR/LF is safe after letters and numbers (after a symbol or a mark it
//     can be absorbed by a symbol piece);
//   - a symbol is safe after a letter unless it is an apostrophe (a
//     contraction suffix), after a number, after CR/LF unless it is "/" (a
//     symbol piece absorbs CR/LF and "/" after it), and after whitespace other
//     than U+0020 (which would join it);
//   - marks are never safe: they can extend a letter run and a symbol run.
__host__ __device__ constexpr bool o2_sync(uint32_t x, uint32_t y, uint32_t cx, uint32_t cy) {
  switch (y) {
    case O2_N: return x != O2_N && x != O2_NONE;
    case O2_UP: return x == O2_N || x == O2_NL || x == O2_LO;
    case O2_LO:
    case O2_BO: return x == O2_N || x == O2_NL;
    case O2_WS: return o2_letter(x) || x == O2_MK || x == O2_N || x == O2_O;
    case O2_NL: return o2_letter(x) || x == O2_N;
    case O2_O:
      return (o2_letter(x) && cy != 0x27u) || x == O2_N || (x == O2_NL && cy != 0x2Fu) ||
             (x == O2_WS && cx != 0x20u);
    default: return false;
  }
}

}  // namespace tt
