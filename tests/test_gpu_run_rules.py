"""Piece starts from window bitmaps (``tt_runs.h``), at the places where a run
or a character meets the edge of a bitmap word (32 bytes), of the window or of a
tile (1,984 bytes, with 32 bytes of context): split level against the oracle."""

import random

import numpy as np
import pytest

from oracle.pretok import piece_byte_starts

pytestmark = pytest.mark.gpu

OWN = 1984
# pieces of text whose rules look along a run or at neighbouring characters;
# numbers, whitespace and symbols of one to four bytes among them
PARTS = ["x's", "x'S", "x're y", "x'LL", "'ſt", "a'ſb", ".'s", " 's", "'", "''ll", "don't", "x'véa", "1", "12", "1234567",
         "١٢٣٤٥", "１２３", "1²3", " ", "  ", "\t", " ", "　　", "\n", "\r\n", "\n\n \n", "\n  ", "!\n", "!\n\n  x", "?\r\n \t",
         "a\n 　\n", "é", "中文", "Ж", "😀", "…", ".", "...", " .", "_x", "-é", "…a", " …a", "​",
         # case changes, two-case letters, marks, rows of contractions, symbol tails with slashes, controls, kana
         "aB", "ABc", "AB", "中AB", "a中AB", "AB中", "AB中Cd", "ǅa", "ʰB", "e\u0301", "\u0301", "!\u0301", "!!\u0301x",
         " !\u0301a", "A\u0301B", "中\u0301B", "'s's's", "a's's", "É'LL", "!\n/", "!\n//x", "/\n/.\u0301\n/", "//", "a/b",
         "\x01", "\x01\x01a", "!a", "!aé", "!é", "…A", "かな", "・", "か・\u3097", "\u3097か", "\u3099", "〇1"]
PATTERNS = ["gpt2", "cl100k", "o200k", "deepseek"]


def _tok(pattern, table=1):
    from paper_2607_29678_amd import Tokenizer
    from workloads.tables import load_table

    return Tokenizer(*load_table(table), pattern)


def _same(tok, text, pattern):
    assert tok.pretokenize(text.encode()).tolist() == piece_byte_starts(text, pattern), repr(text[:80])


@pytest.mark.parametrize("pattern", PATTERNS)
def test_parts_at_word_and_tile_edges(gpu, pattern):
    rng = random.Random(5)
    with _tok(pattern) as tok:
        for edge in (32, OWN - 32, OWN, OWN + 32, 2 * OWN):
            for _ in range(25):
                before = "".join(rng.choice(PARTS) for _ in range(12))
                after = "".join(rng.choice(PARTS) for _ in range(12))
                pad = edge - rng.randint(0, 24) - len(before.encode())
                fill = "ab " * (max(pad, 0) // 3 + 1)
                _same(tok, fill[:max(pad, 0)] + before + after + " tail" * rng.randint(0, 20), pattern)


@pytest.mark.parametrize("pattern", PATTERNS)
@pytest.mark.parametrize("run", ["7", "٣", "９", "\n", "\r\n", " ", "　", "\n ", "é", "?", "A", "中", "\u0301", "中\u0301",
                                 "!\u0301", "/", "\n/", "'s", "'ll", "か", "a"])
@pytest.mark.parametrize("n", [9, 33, 700, 4100])
def test_runs_across_tiles(gpu, pattern, run, n):
    """Runs longer than the context before a tile, and longer than whole tiles,
    after each kind of character, and before one that what precedes the run
    decides on."""
    with _tok(pattern) as tok:
        for lead in ("", "a", "A", "!", "!!", " !", "1a\n", "!\n", "中"):
            for off in (OWN - 41, OWN - 2, OWN + 31):
                for end in ("", "x", "X", "Xy", "é", "'s", "!", ".a", "\n x", "\u0301A"):
                    if n > 700 and (off == OWN - 2 or end in ("", "x", "!", "X")):
                        continue
                    _same(tok, ("w " * OWN)[:off - len(lead)] + lead + run * n + end, pattern)


@pytest.mark.parametrize("pattern", PATTERNS)
@pytest.mark.parametrize("lead", ["!!", " !", "…!", "a!", "中'", "…", "!…", "😀", "é", "\u0301", "・", "x'", "1", "A", "　"])
def test_leads_at_the_window_edge(gpu, pattern, lead):
    """A character on, or cut by, the window's first byte (32 bytes before the tile), then a run up to the tile and a
    character that what precedes the run decides on."""
    with _tok(pattern) as tok:
        for end in range(OWN - 36, OWN - 27):
            before = ("w " * OWN)[:end - len(lead.encode())] + lead
            for run, tail in (("a", "é tail"), ("a", "中"), ("\n", "  \nx"), ("\n", "\t\r"), ("A", "b"), ("中", "A"),
                              ("\u0301", "A"), ("7", "7"), ("/", "\n x"), ("!", "a")):
                for n in (27, 30, 31, 32, 40):
                    _same(tok, before + run * (n // len(run.encode())) + tail, pattern)


@pytest.mark.parametrize("pattern", PATTERNS)
def test_documents_cut_every_rule(gpu, pattern):
    """Short documents side by side: no rule looks across a document's start."""
    from oracle.bpe import bpe
    from oracle.pretok import pretokenize
    from tests.conftest import oracle_table

    rng = random.Random(9)
    docs = ["".join(rng.choice(PARTS) for _ in range(rng.randint(0, 6))) for _ in range(1500)]
    table = oracle_table(1)
    with _tok(pattern) as tok:
        for d, g in zip(docs, tok.encode_batch([d.encode() for d in docs])):
            want = []
            for a, b in pretokenize(d, pattern):
                want += bpe(d[a:b].encode(), table)
            assert g.tolist() == want, repr(d)


@pytest.mark.parametrize("pattern", ["cl100k", "o200k"])
@pytest.mark.parametrize("bad", [b"\x80", b"\xc3", b"\xe4\xb8", b"\xf0\x9f\x98", b"\xc1\xbf", b"\xe0\x9f\xbf", b"\xed\xa0\x80",
                                 b"\xf4\x90\x80\x80", b"\xf5\x80\x80\x80", b"\xc3\xa9\xa9", b"\xff"])
def test_invalid_bytes_at_every_place_of_a_word(gpu, bad, pattern):
    """Also where the text or a document ends inside a character."""
    from paper_2607_29678_amd import TokTierError

    with _tok(pattern) as tok:
        for at in [0, 1, 2, 3, 30, 31, 32] + list(range(OWN - 5, OWN + 3)):
            for tail in (b"", b"x", "é".encode(), b"x" * 40, b"y" * OWN):
                with pytest.raises(TokTierError):
                    tok.pretokenize(b"a" * at + bad + tail)
            with pytest.raises(TokTierError):
                tok.encode_batch([b"a" * at + bad, "é".encode(), b"x"])
        cut = "x" * 7 + "😀"
        for k in (1, 2, 3):  # a character split between two documents
            with pytest.raises(TokTierError):
                tok.encode_batch([cut.encode()[:-k], cut.encode()[-k:]])
        assert np.array_equal(tok.pretokenize(cut.encode()), piece_byte_starts(cut, pattern))
