"""Which attention kernel a call goes to (host logic only, for 256 CUs): the lines lie where the measured times cross, and
the tests of the 64-row kernel assert by the same functions that they reach it."""
import ctypes

import pytest

import paper_2605_12825_amd as orthrus

_lib = ctypes.CDLL(orthrus.library_path())
_decode = getattr(_lib, "_ZN7orthrus14attn_wide_paysEiiili")
_decode.restype, _decode.argtypes = ctypes.c_bool, [ctypes.c_int] * 3 + [ctypes.c_int64, ctypes.c_int]
_prefill = getattr(_lib, "_ZN7orthrus18prefill_wide_wavesEiiliii")
_prefill.restype, _prefill.argtypes = ctypes.c_int, [ctypes.c_int] * 2 + [ctypes.c_int64] + [ctypes.c_int] * 3
_merge = getattr(_lib, "_ZN7orthrus11merge_wavesEli")
_merge.restype, _merge.argtypes = ctypes.c_int, [ctypes.c_int64, ctypes.c_int]


def decode_is_wide(head_dim, rows, max_seq_len, units):
    """True if an unsplit decode-mode call of these sizes takes the 64-row kernel."""
    return _decode(head_dim, rows, max_seq_len, units, 256)


def prefill_waves(head_dim, group, units, max_new, max_seq_len):
    """Waves of 64 rows per workgroup of a prefill call, 0 for the 32-row kernel's form."""
    return _prefill(head_dim, group, units, max_new, max_seq_len, 256)


@pytest.mark.parametrize("wide,head_dim,rows,max_seq_len,units", [
    (True, 128, 128, 2048, 8192), (True, 128, 112, 1000, 512), (False, 128, 112, 180, 512), (True, 128, 128, 180, 512),
    (False, 128, 128, 256, 768), (True, 128, 128, 400, 768), (True, 128, 128, 180, 896), (False, 128, 96, 2048, 8192),
    (False, 128, 128, 1000, 256), (False, 128, 128, 1000, 640), (True, 128, 112, 2035, 568), (True, 128, 128, 1000, 768),
    (False, 128, 224, 4000, 4096), (True, 128, 256, 2500, 384), (False, 128, 256, 1000, 384), (False, 128, 256, 3000, 256),
    (False, 64, 128, 3000, 512), (False, 64, 128, 2048, 640), (True, 64, 128, 2048, 704), (True, 64, 128, 400, 1024), (False, 64, 128, 180, 768), (True, 64, 112, 256, 768),
    (True, 64, 256, 512, 320), (False, 64, 256, 300, 320), (True, 64, 256, 1024, 256), (False, 64, 256, 700, 256),
    (True, 64, 224, 1024, 384), (False, 64, 224, 700, 384), (False, 64, 224, 4000, 352),
])
def test_decode_route(wide, head_dim, rows, max_seq_len, units):
    assert decode_is_wide(head_dim, rows, max_seq_len, units) == wide


@pytest.mark.parametrize("waves,head_dim,group,units,max_new,max_seq_len", [
    # empty cache, from one short prompt to many long ones
    (0, 128, 4, 8, 128, 128), (0, 128, 4, 2, 7000, 7000), (4, 128, 4, 8, 8192, 8192), (2, 128, 4, 8, 4000, 4000),
    (0, 128, 3, 2, 7000, 7000), (0, 128, 2, 8, 2000, 2000), (2, 128, 2, 8, 4093, 4093), (0, 128, 1, 8, 4000, 4000),
    (2, 128, 1, 8, 7000, 7000), (0, 64, 1, 8, 9000, 9000), (0, 64, 4, 8, 2000, 2000), (4, 64, 4, 8, 4000, 4000),
    # behind a longer cache
    (0, 128, 1, 32, 700, 3700), (2, 128, 1, 32, 1021, 3521), (0, 128, 2, 8, 2000, 5000), (0, 128, 4, 8, 700, 3700),
    (2, 128, 4, 8, 2000, 5000), (0, 128, 3, 32, 700, 3700), (4, 128, 3, 32, 677, 3177), (0, 64, 1, 32, 700, 3700),
    (4, 64, 2, 32, 700, 3700),
    # more than four query heads per KV head
    (2, 128, 5, 1, 16, 16), (2, 128, 7, 4, 700, 700), (4, 64, 8, 2, 16, 5000), (4, 128, 7, 32, 700, 3700),
])
def test_prefill_route(waves, head_dim, group, units, max_new, max_seq_len):
    assert prefill_waves(head_dim, group, units, max_new, max_seq_len) == waves


@pytest.mark.parametrize("waves,wgs,num_cus", [(1, 64, 256), (1, 127, 256), (4, 128, 256), (4, 64, 32), (1, 15, 32)])
def test_merge_form(waves, wgs, num_cus):
    """A workgroup per wave while half the CUs of this device, whatever part of the chip it is, would have none."""
    assert _merge(wgs, num_cus) == waves
