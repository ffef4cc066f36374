"""Piece starts by the library's rules (``tt_runs.h``), run on the CPU, against the oracle: what the rules take
from the 32 bytes before a tile, at the library's tile size and at small ones."""

import random

import pytest

from oracle.pretok import piece_byte_starts
from run_rules import HALO, starts, starts_and_operations

OWN = 1984


def _same(text, pattern, own=OWN, docs=None):
    if docs is None:
        want = piece_byte_starts(text, pattern)
    else:
        want, at = [], 0
        for d in docs:
            want += [at + x for x in piece_byte_starts(d, pattern)]
            at += len(d.encode())
    assert starts(text, pattern, own, docs) == want, (pattern, own, docs or text[-120:])


def _at(lead, edge):
    """Text that ends in ``lead``, whose last byte is the byte before ``edge``."""
    return ("w " * edge)[:edge - len(lead.encode())] + lead


# a window begins 32 bytes before its tile; a lead character on that byte, or cut by it
LEADS = ["!!", " !", "…!", "a!", "!", "。'", "😀#", "\x01'", "中!", "\n!", "é'", "1$"]


@pytest.mark.parametrize("own", [OWN, 64])
@pytest.mark.parametrize("lead", LEADS)
def test_lone_symbol_at_the_window_edge(own, lead):
    """DeepSeek: ASCII letters belong to an ASCII symbol before them unless a symbol or U+0020 precedes it, which a
    tile cannot see when the symbol is its window's first character."""
    edge = 2 * own - HALO
    for end in range(edge - 1, edge + 5):
        for run in (HALO - 2, HALO - 1, HALO, 40, HALO + own, HALO + 2 * own):
            for tail in ("é tail", "é", " x", "!é"):
                _same(_at(lead, end) + "a" * run + tail, "deepseek", own)
    for cut in (0, 1):  # a document starts at the symbol, or after it
        text = _at(lead, edge + 1)
        _same(None, "deepseek", own, [text[:len(text) - 1 + cut], text[len(text) - 1 + cut:] + "a" * (HALO - 1) + "é"])


@pytest.mark.parametrize("own", [OWN, 64])
@pytest.mark.parametrize("pattern", ["cl100k", "deepseek", "o200k"])
@pytest.mark.parametrize("lead", ["…", "😀", "！", "!", "!…", "é", "中", "٣", "　", "\u0301", "・", "\n", " "])
def test_line_breaks_behind_a_cut_character(own, pattern, lead):
    """A CR/LF run is the tail of a symbol piece when a symbol precedes it; the window may begin inside that symbol."""
    edge = 2 * own - HALO
    for end in range(edge - 1, edge + 5):
        for run in (HALO - 4, HALO - 2, HALO - 1, HALO, HALO + own):
            for tail in ("  \nx", "\t\r", "　\n", " x", "\nx"):
                _same(_at(lead, end) + "\n" * run + tail, pattern, own)
    text = _at(lead, edge + 1)
    n = len(text) - len(lead)
    for k in range(n, len(text) + 1):  # a document starts around the lead
        _same(None, pattern, own, [text[:k], text[k:] + "\r" * (HALO - 1) + "  \n"])


@pytest.mark.parametrize("pattern", ["cl100k", "o200k", "deepseek"])
def test_runs_past_the_window(pattern):
    """Whitespace after a line break, and capitals after a letter without case, up to what ends them: beyond the
    window, in steps of 1,024 bytes, 16 per lane, with characters that a lane's bytes cut."""
    rng = random.Random(7)
    ws = [" ", "\t", "\u3000", "\u00a0", "\u2028"]
    runs = [("\n", ws, ["\nx", "x", "é", "\r", "1", "中", ""])]
    if pattern == "o200k":
        runs.append(("中", ["A", "Я", "É", "\U00010400"], ["b", "я", "中", "\u0301", "1", " ", "'s", ""]))
    for lead, parts, tails in runs:
        for size in (10, 63, 64, 65, 200, 1020, 1025, 1090, 2100):
            for tail in tails:
                kinds = rng.sample(parts, rng.randint(1, len(parts)))
                run = ""
                while len(run.encode()) < size + rng.randint(0, 20):
                    run += rng.choice(kinds)
                text = "w" * rng.randint(0, 70) + lead + run
                _same(text + tail, pattern, 64)
                _same(None, pattern, 64, [text, tail, "\nx"])


@pytest.mark.parametrize("text,pattern", [("\n" + "\u3000" * 20_000, "cl100k"), ("\n" + "\u3000" * 20_000, "o200k"),
                                          ("\n" + "\u00a0\u3000" * 12_000, "deepseek"), ("中" + "Я" * 30_000, "o200k")])
def test_a_long_run_past_the_window_takes_few_steps(text, pattern):
    """A step of the wave takes the characters of 1,024 bytes, whatever their length."""
    got, ops = starts_and_operations(text, pattern)
    assert got == piece_byte_starts(text, pattern)
    assert ops < 400 + 4 * len(text.encode()) // 1024
