"""An error of an earlier runtime call that nobody has read does not fail a later call of the library."""

import ctypes

import pytest

from conftest import config_bytes, lib_tokenizer, oracle_config_ids

pytestmark = pytest.mark.gpu


def test_calls_after_an_unread_error(gpu):
    from paper_2607_29678_amd import _lib

    hip = ctypes.CDLL(_lib.LIB_PATH)  # (the runtime's entry points, through the library that links to it)
    data, want = config_bytes(1), list(oracle_config_ids(1))
    tok = lib_tokenizer(1)
    d_in = gpu.frombuffer(bytearray(data), dtype=gpu.uint8).to("cuda")
    ids = gpu.zeros(len(data), dtype=gpu.int32, device="cuda")
    n = gpu.zeros(1, dtype=gpu.int64, device="cuda")
    gpu.cuda.synchronize()
    assert hip.hipSetDevice(1 << 20) != 0  # no such device
    try:
        for call in (tok.encode_device, tok.encode_device_noalloc):
            for _ in range(3):
                call(d_in, len(data), ids, n)
                assert hip.hipDeviceSynchronize() == 0
    finally:
        hip.hipGetLastError()
    assert ids[:int(n.item())].tolist() == want
    assert tok.encode(data).tolist() == want
