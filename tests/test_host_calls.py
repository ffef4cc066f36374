"""The host code (``tt_api.hip``, ``tt_session.hip``) on the CPU: what it does when memory runs out, and which
documents it hands to the kernel.  The sources themselves, compiled for the host against a runtime with budgets for
device and pinned memory, whose kernel gives one token per byte (``tests/native/fake_hip.cpp``)."""

import ctypes
import functools
import os
import shutil
import subprocess
import tempfile

import numpy as np
import pytest

from paper_2607_29678_amd import Session, Tokenizer, TokTierError, _lib
from run_rules import CSRC, NATIVE, clang

ALL = (1 << 64) - 1


@functools.lru_cache(maxsize=None)
def _fake():
    tmp = tempfile.mkdtemp(prefix="fake_hip_")
    try:
        so = os.path.join(tmp, "fake.so")
        r = subprocess.run([clang(), "-O1", "-std=c++17", "-shared", "-fPIC", "-pthread", "-w", "-I" + NATIVE, "-I" + CSRC,
                            "-x", "c++"] + [os.path.join(CSRC, f) for f in ("tt_api.hip", "tt_session.hip", "tt_copy.cpp")]
                           + [os.path.join(NATIVE, "fake_hip.cpp"), "-o", so], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-4000:]
        lib = ctypes.CDLL(so)
    finally:
        shutil.rmtree(tmp)
    for name, (res, args) in _lib.SIGNATURES.items():
        if hasattr(lib, name):
            fn = getattr(lib, name)
            fn.restype, fn.argtypes = res, args
    lib.fake_budgets.argtypes = [ctypes.c_uint64, ctypes.c_uint64]
    lib.fake_used.restype = ctypes.c_uint64
    lib.fake_device.restype = ctypes.c_void_p
    lib.fake_device.argtypes = [ctypes.c_uint64]
    lib.fake_free.argtypes = [ctypes.c_void_p]
    return lib


@pytest.fixture
def fake(monkeypatch):
    lib = _fake()
    monkeypatch.setattr(_lib, "_lib", lib)
    yield lib
    lib.fake_budgets(ALL, ALL)


# IDs of 16, 24 and 32 bits (staged in as many bytes)
FIRST = {16: 0, 24: 70_000, 32: 1 << 24}


def _tok(bits=16, **opt):
    first = FIRST[bits]
    vocab = [b"??"] * first + [bytes([b]) for b in range(256)]
    offsets = np.concatenate([[0], np.cumsum([len(v) for v in vocab])]).astype(np.int64)
    return Tokenizer(np.zeros((0, 3), dtype=np.int32), np.frombuffer(b"".join(vocab), dtype=np.uint8), offsets, "gpt2", **opt)


def _ids(data, bits=16):
    return [FIRST[bits] + b for b in data]


def test_a_failed_allocation_does_not_fail_the_next_call(fake):
    """The runtime keeps its last error until it is read; a later call's launch does not take it for its own (and the
    tile tickets stay in step with the calls)."""
    with _tok() as tok:
        text, ids, n = (fake.fake_device(k) for k in (1 << 20, 4 << 20, 8))
        ctypes.memmove(text, b"x" * (1 << 20), 1 << 20)
        fake.fake_budgets(16 << 20, ALL)
        with pytest.raises(TokTierError) as e:
            tok.encode_device(text, 1 << 20, ids, n)
        assert e.value.status == -8
        for _ in range(2):
            tok.encode_device(text, 3, ids, n)
        assert ctypes.cast(n, ctypes.POINTER(ctypes.c_int64))[0] == 3
        assert ctypes.cast(ids, ctypes.POINTER(ctypes.c_int32))[:3] == _ids(b"xxx")
        for p in (text, ids, n):
            fake.fake_free(p)


def test_a_failed_allocation_leaves_no_error_behind(fake):
    """The status says what failed; the program's own check of the runtime after the call finds nothing."""
    data, spans = b"x" * (1 << 20), 5 << 20
    with _tok() as tok:
        for device, pinned, call in ((16 << 20, ALL, lambda: tok.encode(data)), (ALL, 1 << 20, lambda: tok.encode(data)),
                                     (180 << 20, ALL, lambda: tok.encode_spans(b"x" * spans))):
            fake.fake_budgets(device, pinned)
            with pytest.raises(TokTierError) as e:
                call()
            assert e.value.status == -8
            assert fake.fake_last_error() == 0
    fake.fake_budgets(1 << 18, ALL)
    with pytest.raises(TokTierError) as e:
        _tok()
    assert e.value.status == -8 and fake.fake_last_error() == 0


TEXT = "".join("wörd %d, 中文 – x%d\n" % (i, i * i) for i in range(9000))


def _docs(n):
    data = TEXT.encode()
    cuts, at = [0], 0
    for k in range(n):
        at = min(len(data), at + (k * 7919) % (2 * len(data) // n + 1))
        while at < len(data) and (data[at] & 0xC0) == 0x80:
            at += 1
        cuts.append(at)
    return [data[a:b] for a, b in zip(cuts, cuts[1:])] + [b"", data[at:], b""]


def _spans(data):
    chars, out = 0, []
    for i, b in enumerate(data):
        chars += (b & 0xC0) != 0x80
        out.append([i, i + 1, chars - 1, chars])
    return out


# no pinned memory but the length word; room for the documents' words, not for the IDs; room for the staged
# IDs, not for the spans; all
@pytest.mark.parametrize("bits,pinned", [(b, p) for b in (16, 24) for p in (8, 64 << 10, 3 << 20, ALL)] + [(32, 8), (32, ALL)])
def test_calls_without_pinned_memory(fake, bits, pinned):
    """Batches, span export and sessions that find no pinned memory give the same results through copies."""
    docs, data = _docs(300), TEXT.encode()
    with _tok(bits) as tok:
        fake.fake_budgets(ALL, pinned)
        for batch in (docs, [b"a", b"", b"bc"], docs[:40]):
            assert [g.tolist() for g in tok.encode_batch(batch)] == [_ids(d, bits) for d in batch]
        with pytest.raises(TokTierError) as e:
            tok.encode_batch([b"ab", b"\x80"])
        assert e.value.status == -5
        ids, spans = tok.encode_spans(data)
        assert ids.tolist() == _ids(data, bits) and spans.tolist() == _spans(data)
        with Session(tok, 16) as s:
            step = len(TEXT) // 5 + 1
            for k in range(0, len(TEXT), step):
                s.append(TEXT[k:k + step].encode())
            ids, spans = s.tokens()
        assert ids.tolist() == _ids(data, bits) and spans.tolist() == _spans(data)
        assert fake.fake_last_error() == 0
        before = fake.fake_used(0)
        assert [g.tolist() for g in tok.encode_batch(docs)] == [_ids(d, bits) for d in docs]
        assert fake.fake_used(0) == before  # (what a call without pinned memory took is given back)
    # literals: their segments go the way of a batch
    fake.fake_budgets(ALL, ALL)
    with _tok(bits, added=[("<|x|>", 999)]) as tok:
        fake.fake_budgets(ALL, fake.fake_used(1) + pinned if pinned != ALL else ALL)
        want = _ids(b"ab", bits) + [999] + _ids(data, bits)
        assert tok.encode(b"ab<|x|>" + data).tolist() == want
        assert [g.tolist() for g in tok.encode_batch([b"ab<|x|>", data])] == [want[:3], want[3:]]


@pytest.mark.parametrize("docs", [[b"", b"ab", b"", b"", b"c" * 5000, b""], [b"a", b"b"], [b"", b"", b"x"], [b"x", b"", b""],
                                  [b"ab"] + [b""] * 700 + [b"cd"] * 3 + [b""] * 40 + ["é".encode() * 3000] + [b""] * 2])
@pytest.mark.parametrize("pinned", [8, ALL])
def test_empty_documents_stay_on_the_host(fake, docs, pinned):
    """One block has all documents of its bytes: the kernel gets one per position, however many are empty."""
    with _tok() as tok:
        fake.fake_budgets(ALL, pinned)
        assert [g.tolist() for g in tok.encode_batch(docs)] == [_ids(d) for d in docs]
        assert fake.fake_documents() == sum(1 for d in docs if d)
        with pytest.raises(TokTierError) as e:
            tok.encode_batch(docs + [b"", b"\xff", b""])
        assert e.value.status == -5


def _pairs_of_results(vocab, n):
    for a in range(n):
        for b in range(n):
            yield a, b
    first = len(vocab)
    for i in range(256, min(first, 256 + 8 * n)):
        for j in range(256, min(first, 256 + 8 * n)):
            yield i, j


def _letters_then(vocab, n):
    for a in range(97, 97 + n):
        for b in range(97, 97 + n):
            yield a, b
    for r in range(256, len(vocab)):
        for b in range(97, 97 + n):
            yield r, b


def _one_letter(vocab, n):
    yield 97, 97
    for _ in range(n - 1):
        yield len(vocab) - 1, 97


@pytest.mark.parametrize("pairs,n", [(_letters_then, 2), (_letters_then, 26), (_pairs_of_results, 8), (_pairs_of_results, 32),
                                     (_pairs_of_results, 256), (_one_letter, 1500)])
def test_merge_tables_of_neighbouring_pairs(fake, pairs, n):
    """The merge table's hashes are sums of products: lists whose pairs are neighbours in both operands, which such
    hashes put side by side, are accepted too, in tables of a few times the load of others."""
    vocab, merges, seen = [bytes([b]) for b in range(256)], [], set()
    for a, b in pairs(vocab, n):
        if (a, b) not in seen:
            seen.add((a, b))
            merges.append((a, b, len(vocab)))
            vocab.append(vocab[a] + vocab[b])
            if len(merges) >= 80_000:
                break
    offsets = np.concatenate([[0], np.cumsum([len(v) for v in vocab])]).astype(np.int64)
    before = fake.fake_used(0)
    with Tokenizer(np.array(merges, dtype=np.int32), np.frombuffer(b"".join(vocab), dtype=np.uint8), offsets, "gpt2"):
        # (besides the merge table: the byte pairs and junctions, the dictionaries, 8 bytes per ID)
        assert fake.fake_used(0) - before < (1 << 20) + (8 + 4 * 16 + 4 * 32) * len(merges)
