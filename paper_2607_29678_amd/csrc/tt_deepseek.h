// The DeepSeek-style pattern (Sec. 4.1: DeepSeek-family tokenizers apply three
// splitters in sequence; their composition folds into one per-character
// predicate when each splitter re-splits every piece of the stage before and
// unmatched stretches survive as pieces).  The splitters, in order:
//   S1  \p{N}{1,3}
//   S2  runs of CJK ideographs U+4E00-9FA5, hiragana U+3040-309F, katakana U+30A0-30FF
//   S3  D1 [ASCII punctuation or symbol][A-Za-z]+
//       D2 [^\r\n\p{L}\p{P}\p{S}]?[\p{L}\p{M}]+
//       D3 U+0020? [\p{P}\p{S}]+ [\r\n]*
//       D4 \s*[\r\n]+    D5 \s+(?!\S)    D6 \s+
//
// A stretch of numbers, a stretch of the CJK/kana set and a stretch of
// everything else ("groups") are pieces of the first two stages, so every
// group change is a piece boundary that no context moves, and the third
// splitter runs inside one group stretch at a time, which it sees as the
// whole text.  Here are the classes and the synchronizing transitions; the tile
// kernel's rules are in tt_runs.h.
#pragma once

#include "tt_internal.h"
#include "tt_o200k.h"

namespace tt {

// Classes of the DeepSeek-style pattern (4 bits of a window code), as in the
// generated table.
enum : uint32_t {
  DS_O = 0,    // none of the others (controls, format characters, unassigned)
  DS_AL = 1,   // ASCII letter
  DS_L = 2,    // other letter
  DS_M = 3,    // mark
  DS_N = 4,    // \p{N}
  DS_AP = 5,   // ASCII punctuation or symbol
  DS_PS = 6,   // other punctuation or symbol
  DS_SP = 7,   // U+0020
  DS_WS = 8,   // other \s but CR and LF
  DS_NL = 9,   // CR, LF
  DS_KL = 10,  // in the CJK/kana ranges: letter
  DS_KM = 11,  //   mark
  DS_KP = 12,  //   punctuation or symbol
  DS_KO = 13,  //   other
  DS_NONE = 15
};

// Group of a class: 0 the rest, 1 numbers, 2 the CJK/kana set, 3 none.
__host__ __device__ constexpr uint32_t ds_group(uint32_t c) {
  return c == DS_N ? 1u : (c >= DS_KL && c <= DS_KO) ? 2u : c == DS_NONE ? 3u : 0u;
}

// Class of an ASCII code point (equal to the table's; computed, so that it
// does not depend on the table being staged yet).
__host__ __device__ inline uint32_t ds_ascii_class(uint32_t cp) {
  if (((cp | 32u) - 'a') < 26u) return DS_AL;
  if ((cp - '0') < 10u) return DS_N;
  if (cp == 10u || cp == 13u) return DS_NL;
  if (cp == 32u) return DS_SP;
  if (cp == 9u || cp == 11u || cp == 12u) return DS_WS;
  if ((cp - 33u) < 94u) return DS_AP;  // the printable characters left are punctuation and symbols
  return DS_O;
}

template <class P>
__host__ __device__ inline uint32_t ds_table_class(P l1, P l2, uint32_t cp) {
  const uint32_t blk = l1[cp >> 8];
  return (l2[blk * 128u + ((cp & 255u) >> 1)] >> ((cp & 1u) * 4u)) & 15u;
}

// Whether a position whose left character has class x and whose right
// character has class y is a synchronizing boundary of the DeepSeek-style
// pattern: every text with these two characters there has a piece boundary
// between them, the pieces to the right depend on the left only through x,
// and the pieces to the left depend on the right only through y.  A group
// change always is one.  Inside the rest, from the third splitter:
//   - before a letter or mark: after CR/LF, a number or a non-ASCII
//     punctuation mark or symbol (which can neither be D2's first character
//     nor take letters in D1); a non-ASCII letter or a mark also after ASCII
//     punctuation (D1 takes ASCII letters only);
//   - before punctuation or a symbol: after a letter, a mark, CR/LF, other
//     whitespace than U+0020 or a character of none of the classes;
//   - before whitespace: after a letter, a mark, punctuation, a symbol or a
//     character of none of the classes; before CR/LF not after punctuation or
//     a symbol (D3 takes CR/LF after them) nor after whitespace;
//   - before a character of none of the classes: after anything but another
//     such character (which may be D2's first character before letters).
// Inside the CJK/kana set: before a letter or mark, after punctuation or a
// symbol; before punctuation or a symbol, after anything else of the set
// (D3 does not take letters, marks or unassigned code points); before an
// unassigned code point, after anything but another one (which may be D2's
// first character before letters).
__host__ __device__ constexpr bool ds_sync(uint32_t x, uint32_t y) {
  if (x == DS_NONE || y == DS_NONE) return false;
  if (ds_group(x) != ds_group(y)) return true;
  const uint32_t bx = 1u << x;
  switch (y) {
    case DS_AL: return (bx & ((1u << DS_NL) | (1u << DS_PS))) != 0u;
    case DS_L:
    case DS_M: return (bx & ((1u << DS_NL) | (1u << DS_PS) | (1u << DS_AP))) != 0u;
    case DS_AP:
    case DS_PS:
      return (bx & ((1u << DS_AL) | (1u << DS_L) | (1u << DS_M) | (1u << DS_NL) | (1u << DS_O) | (1u << DS_WS))) != 0u;
    case DS_SP:
    case DS_WS: return (bx & ((1u << DS_AL) | (1u << DS_L) | (1u << DS_M) | (1u << DS_AP) | (1u << DS_PS) | (1u << DS_O))) != 0u;
    case DS_NL: return (bx & ((1u << DS_AL) | (1u << DS_L) | (1u << DS_M) | (1u << DS_O))) != 0u;
    case DS_O: return x != DS_O;
    case DS_KL:
    case DS_KM: return x == DS_KP;
    case DS_KP: return x != DS_KP;
    case DS_KO: return x != DS_KO;
    default: return false;
  }
}

}  // namespace tt
