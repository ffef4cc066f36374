"""Units of 3..64 bytes, several to a wave (``bpe_lanes``).

A round of that engine merges, besides the unit's lowest rank, every pair whose
rank lies below the lowest rank of any merge across the boundaries on either
side of it.  The schedule is restated here and compared with greedy BPE on the
CPU; on the GPU, units at the edges of every width (8, 16, 32 and 64 bytes, and
the two-row engine after them) are compared with the oracle, in counts that
leave the last wave of a width partly filled.
"""

import random

import numpy as np
import pytest

from oracle.bpe import MergeTable, bpe
from tests.test_gpu_random_merges import _docs, _pack, random_merges


def _bounded_rounds(piece, merges, vocab):
    """IDs by rounds that merge the lowest rank (leftmost first, without overlap)
    and every pair below the junction bounds of its outer boundaries."""
    rank, low = {}, {}
    for r, (a, b, _) in enumerate(merges):
        rank[a, b] = r
        low.setdefault((vocab[a][-1], vocab[b][0]), r)  # (the first is the lowest)
    inf = len(merges)
    ids = list(piece)
    while True:
        r = [rank.get(p, inf) for p in zip(ids, ids[1:])]
        if not r or min(r) == inf:
            return ids
        j = [inf] + [low.get((vocab[a][-1], vocab[b][0]), inf) for a, b in zip(ids, ids[1:])] + [inf]
        take, m = set(), min(r)
        for i, x in enumerate(r):
            if x == m and i - 1 not in take:
                take.add(i)
        lowest = set(take)
        take |= {i for i, x in enumerate(r) if x < j[i] and x < j[i + 2]}
        assert all(i + 1 not in take for i in take), "two pairs share a token"
        out, i = [], 0
        while i < len(ids):
            if i in take:
                out.append(merges[r[i]][2])
                i += 2
            else:
                out.append(ids[i])
                i += 1
        assert lowest <= take
        ids = out


@pytest.mark.parametrize("seed,letters,n_merges,same", [(1, "ab", 400, False), (2, "abcd", 900, False),
                                                        (3, "abcdefgh", 1500, False), (4, "abc", 500, True)])
def test_bounded_rounds_equal_greedy(seed, letters, n_merges, same):
    merges, vocab = random_merges(seed, letters, n_merges, allow_same_spelling=same)
    table = MergeTable(merges, vocab)
    for d in _docs(500 + seed, letters, 400, lo=2, hi=64):
        assert _bounded_rounds(d, merges, vocab) == bpe(d, table), d


@pytest.mark.gpu
@pytest.mark.parametrize("letters,n_merges", [("ab", 500), ("abcdefgh", 2500)])
@pytest.mark.parametrize("count", [1, 3, 9])
def test_units_at_the_edges_of_every_width(gpu, letters, n_merges, count):
    from paper_2607_29678_amd import Tokenizer

    merges, vocab = random_merges(21, letters, n_merges)
    table = MergeTable(merges, vocab)
    vb, vo = _pack(vocab)
    rng = random.Random(77)
    with Tokenizer(np.array(merges, dtype=np.int32), vb, vo, "gpt2") as tok:
        for L in (3, 4, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129):
            docs = _docs(L * 100 + count, letters, count, lo=L, hi=L)
            docs += [letters[0].encode() * L, (letters[:2] * L).encode()[:L]]
            docs += _docs(L, letters, 5, lo=2, hi=140)
            rng.shuffle(docs)
            for d, g in zip(docs, tok.encode_batch(docs)):
                assert g.tolist() == bpe(d, table), (L, d)
