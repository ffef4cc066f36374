"""Piece starts by the library's rules (``tt_runs.h``), run on the CPU, against the oracle: what the rules take
from the 32 bytes before a tile, at the library's tile size and at small ones."""

import itertools
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


# representatives of every class a pattern tells apart
ALPHABET = {
    "gpt2": ["a", "s", "é", "1", "²", " ", "\t", "\n", "'", "!", "…"],
    "cl100k": ["a", "S", "é", "ſ", "1", "²", " ", "\u3000", "\n", "\r", "'", "!", "…"],
    "o200k": ["a", "s", "S", "É", "中", "\u0301", "1", " ", "\u3000", "\n", "'", "/", "!", "…", "ſ"],
    "deepseek": ["a", "é", "\u0301", "1", "٣", " ", "\u3000", "\n", "!", "'", "…", "中", "か", "・", "\u3097", "\x01"],
}


@pytest.mark.parametrize("pattern", sorted(ALPHABET))
@pytest.mark.parametrize("own,longest", [(OWN, 4), (32, 3)])
def test_all_short_strings(pattern, own, longest):
    """Side by side, as documents: the rules themselves, and that none looks across a document's start."""
    docs = ["".join(t) for n in range(1, longest + 1) for t in itertools.product(ALPHABET[pattern], repeat=n)]
    got = set(starts(None, pattern, own, docs))
    at = 0
    for d in docs:
        n = len(d.encode())
        assert [x for x in range(n) if at + x in got] == piece_byte_starts(d, pattern), (pattern, d)
        at += n


MORE = {
    "gpt2": ["'s", "'ll", "'v", "ſ", "😀", "S", "中", "٣", "\r", "\u3000"],
    "cl100k": ["'s", "'ll", "'v", "😀", "中", "٣", "\t"],
    "o200k": ["'s", "'ll", "'S", "'ſ", "é", "ʰ", "\u0e31", "٣", "\t", "\r", "😀"],
    "deepseek": ["S", "\t", "\r", "😀", "\u3099", "\u0e31", "\u200b"],
}


# units whose runs carry something along, and text that what precedes a run decides on
CARRY = ["\n", "a", "1", " ", "!", "中", "\u0301", "A", "/"]
DECIDED = ["  \nx", "\t\r", "\u3000\n", "é", "É", "x", "A", "1", "中", "!", "'s"]


def _edge_case(rng, pattern):
    """A short lead whose last bytes lie around a window's first one, a run up to about a tile's first byte or beyond,
    and what follows it; sometimes cut into documents near the lead."""
    parts = ALPHABET[pattern] + MORE[pattern]
    own, tile = rng.choice((32, 32, 64, 96)), rng.choice((1, 2, 2, 3))
    edge = own * tile - HALO if own * tile > HALO else own
    lead = "".join(rng.choice(parts) for _ in range(rng.choice((1, 2, 2, 3))))
    room = max(0, edge + rng.choice((-1, 0, 1, 1, 2, 3, 4, 5)) - len(lead.encode()))
    fill = rng.choice(("w ", "w", "1", " ", "\n", "!", "中", "S"))
    text = fill * (room // len(fill.encode()))
    text += "w" * (room - len(text.encode())) + lead
    at = len(text)
    unit = rng.choice(CARRY if rng.random() < 0.6 else parts) + (rng.choice(parts) if rng.random() < 0.15 else "")
    end = edge + HALO + rng.choice((-2, -1, 0, 0, 1, 2, 3, own, own + 1, 2 * own))
    text += unit * max(0, (end - len(text.encode())) // len(unit.encode()) + 1)
    text += rng.choice(DECIDED) if rng.random() < 0.5 else "".join(rng.choice(parts) for _ in range(rng.choice((1, 2, 3))))
    if rng.random() < 0.3:
        text += rng.choice(parts) * rng.randint(20, 80) + "".join(rng.choice(parts) for _ in range(2))
    docs = None
    if rng.random() < 0.25:
        cuts = sorted(min(len(text), max(0, at + rng.choice((-3, -2, -1, 0, 1, 20)))) for _ in range(2))
        docs = [text[a:b] for a, b in zip([0] + cuts, cuts + [len(text)])]
    return text, own, docs


@pytest.mark.parametrize("pattern", sorted(ALPHABET))
def test_random_strings_in_small_tiles(pattern):
    """What the rules take from the context before a tile, from the words of earlier tiles and from beyond the
    window."""
    rng = random.Random(41)
    for _ in range(6000):
        text, own, docs = _edge_case(rng, pattern)
        _same(text, pattern, own, docs)
