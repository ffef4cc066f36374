"""Units over 128 bytes on the block engine: rows of 64 tokens split over eight waves, runs of one pair that
cross rows and waves (the choice of every second pair continues from one wave's rows to the next), and rows that
a round leaves as they are beside rows that merge."""

import random

import pytest

from conftest import lib_tokenizer, oracle_ids, oracle_table, pattern_of
from test_gpu_long_units import _clique

pytestmark = pytest.mark.gpu


def _texts(k, seed):
    rng = random.Random(seed)
    letters = _clique(k, b"etaoinsrhldcumfpgwybvkxjqz")  # no unit of these is cut
    # lengths around one row, one row per wave, and both sides of the rows kept in LDS
    sizes = (129, 192, 193, 448, 449, 480, 481, 511, 512, 513, 575, 577, 1023, 1025, 4095, 4097, 9001)
    for n in sizes:
        for c in letters[:2]:
            yield bytes([c]) * n
            # the run's first pair falls on either parity, and other pairs stand inside it
            yield bytes([letters[-1]]) + bytes([c]) * n
            body = bytearray([c]) * n
            for _ in range(rng.randint(1, 6)):
                body[rng.randrange(n)] = rng.choice(letters)
            yield bytes(body)
        yield bytes(rng.choice(letters) for _ in range(n))


@pytest.mark.parametrize("k", [2, 4])
def test_block_units_id_parity(gpu, k):
    tok = lib_tokenizer(k)
    memo = {}
    for i, data in enumerate(_texts(k, 31 + k)):
        got = tok.encode(data).tolist()
        assert got == oracle_ids(data, oracle_table(k), pattern_of(k), memo), "case %d: %d bytes" % (i, len(data))
