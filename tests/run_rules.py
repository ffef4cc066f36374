"""The library's piece-start rules (``csrc/tt_runs.h``) on the CPU: the header itself, compiled for the host by
clang and run on a wave of 64 fibers (``tests/native``), for tiles of a chosen size."""

import ctypes
import functools
import os
import re
import shutil
import subprocess
import tempfile

import numpy as np
import pytest

from oracle.classes import BO, L, LO, MK, N, UP, W, char_class, is_mark, is_punct_or_symbol, o200k_class
from oracle.pretok import ASCII_LETTERS, ASCII_PUNCT, in_kana_cjk

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_29678_amd", "csrc")
NATIVE = os.path.join(ROOT, "tests", "native")
IDS = {"gpt2": 0, "cl100k": 1, "o200k": 2, "deepseek": 3}
HALO = 32


def clang():
    for c in ("/opt/rocm/bin/amdclang++", shutil.which("amdclang++"), shutil.which("clang++")):
        if c and os.path.exists(c):
            return c
    pytest.skip("clang++ not found")


@functools.lru_cache(maxsize=None)
def rules(own=1984):
    """The rules for tiles that own ``own`` bytes (a multiple of 32; 1,984 in the library)."""
    tmp = tempfile.mkdtemp(prefix="run_rules_")
    try:
        os.makedirs(os.path.join(tmp, "package", "csrc"))
        os.makedirs(os.path.join(tmp, "include"))
        shutil.copy(os.path.join(ROOT, "include", "toktier.h"), os.path.join(tmp, "include"))
        for f in os.listdir(CSRC):
            if f.endswith(".h"):
                src = open(os.path.join(CSRC, f)).read()
                # (a tile is smaller than a wave's bitmap: the words past it stay empty)
                if f == "tt_internal.h":
                    src, k = re.subn(r"constexpr int PT_THREADS = 512;", "constexpr int PT_THREADS = %d;" % ((own + 2 * HALO) // 4), src)
                    assert k == 1
                if f == "tt_runs.h":
                    src, k = re.subn(r"static_assert\(BM_WORDS == 64", "static_assert(BM_WORDS <= 64", src)
                    assert k == 1
                open(os.path.join(tmp, "package", "csrc", f), "w").write(src)
        so = os.path.join(tmp, "rules.so")
        r = subprocess.run([clang(), "-O2", "-std=c++17", "-shared", "-fPIC", "-w", "-I" + NATIVE,
                            "-I" + os.path.join(tmp, "package", "csrc"), os.path.join(NATIVE, "run_rules.cpp"), "-o", so],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-4000:]
        lib = ctypes.CDLL(so)
        assert lib.run_rules_own() == own
        lib.run_rules.restype = ctypes.c_uint64
        return lib
    finally:
        shutil.rmtree(tmp)


@functools.lru_cache(maxsize=None)
def class_letter(ch, pattern):
    """The class of a character as ``native/run_rules.cpp`` names it."""
    cp = ord(ch)
    k = char_class(cp)
    if ch in "\r\n":
        return "R"
    if pattern == "deepseek":
        if k == N:
            return "N"
        letter, ps = k == L or is_mark(cp), is_punct_or_symbol(cp)
        if in_kana_cjk(cp):
            return "K" if letter else "k" if ps else "o"
        if ch in ASCII_LETTERS:
            return "a"
        if letter:
            return "L"
        if ps:
            return "p" if ch in ASCII_PUNCT else "P"
        return "S" if ch == " " else "W" if k == W else "O"
    if pattern == "o200k" and o200k_class(cp) in (UP, LO, BO, MK):
        return {UP: "U", LO: "l", BO: "X", MK: "M"}[o200k_class(cp)]
    if k in (L, N):
        return "L" if k == L else "N"
    if k == W:
        return "S" if ch == " " else "W"
    return "A" if ch == "'" else "/" if ch == "/" and pattern == "o200k" else "O"


def starts(text, pattern, own=1984, docs=None):
    """Byte offsets of the piece starts of ``text``, or of the documents ``docs`` side by side."""
    return starts_and_operations(text, pattern, own, docs)[0]


def starts_and_operations(text, pattern, own=1984, docs=None):
    """The same, and the cross-lane operations of the tile that takes the most."""
    parts = [text] if docs is None else docs
    whole = "".join(parts)
    data = whole.encode()
    cls = "".join(class_letter(c, pattern) + "." * (len(c.encode()) - 1) for c in whole).encode()
    flags = None
    if docs is not None:
        flags = np.zeros(len(data) + 1, dtype=np.uint8)
        flags[np.cumsum([0] + [len(d.encode()) for d in docs])] = 1
    out = np.zeros(max(1, len(data)), dtype=np.uint8)
    ops = rules(own).run_rules(IDS[pattern], data, cls, len(data),
                               None if flags is None else flags.ctypes.data_as(ctypes.c_void_p),
                               out.ctypes.data_as(ctypes.c_void_p))
    return np.flatnonzero(out[:len(data)]).tolist(), ops
