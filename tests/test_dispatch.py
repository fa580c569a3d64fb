"""Which kernel takes a call: the rule's lines, by the library's own functions
(host code, looked up by their C++ names), so that a change of the rule cannot
quietly move a test elsewhere off the kernel it is there for."""
import ctypes

import pytest

FULL, ANCHOR, RELAY = 0, 1, 3
F32, BF16 = 0, 1


def shape(n_k, k, m=0, r=0, n_mand=0):
    from paper_2609_07306_amd import routerelay as rr
    f = rr.lib["_ZN2rr14resident_shapeEiiiii"]
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_int] * 5
    return f(n_k, k, m, r, n_mand)


def pays(mode, dtype, d, heads, n_q, n_k, causal, T, one_pass=False):
    from paper_2609_07306_amd import routerelay as rr
    f = rr.lib["_ZN2rr13resident_paysEiiiiiibib"]
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_int] * 6 + [ctypes.c_bool, ctypes.c_int, ctypes.c_bool]
    return f(mode, dtype, d, heads, n_q, n_k, causal, T, one_pass)


def test_resident_shapes():
    assert [shape(n, 32, 16) for n in (1, 256, 257, 512, 513, 1024, 1025, 2048)] == [42, 42, 44, 44, 48, 48, 88, 88]
    assert [shape(n, 64, 32) for n in (512, 513, 1024, 1025, 2048)] == [82, 84, 84, 88, 88]
    assert shape(2049, 64, 64) == shape(4096, 64, 64) == 386
    assert shape(4097, 8) == 0 and shape(100, 64, 65) == 0
    # a tile of several panels stages up to 440 slots a row
    assert shape(2500, 64, 32, 144) == 386 and shape(2500, 1, 0, 255) == 0 and shape(2048, 1, 0, 255) == 88


# mode, dtype, d, heads, n_q, n_k, causal, T (one pass), resident
LINES = [
    # bf16, up to 256-byte rows: from 1025 keys and a 128-row tile per compute unit, T <= 52
    (FULL, BF16, 128, 32, 1024, 1024, False, 48, True), (FULL, BF16, 128, 32, 1024, 1025, False, 48, False),
    (ANCHOR, BF16, 32, 32, 1024, 2048, False, 52, False), (RELAY, BF16, 64, 32, 1024, 2048, False, 53, True),
    (RELAY, BF16, 128, 31, 1024, 1280, False, 48, True), (RELAY, BF16, 128, 32, 897, 1280, False, 48, False),
    # ... two per unit, T <= 56
    (RELAY, BF16, 128, 32, 2048, 1536, False, 56, False), (RELAY, BF16, 128, 32, 2048, 1536, False, 57, True),
    # ... and relays of 64-byte rows only up to 1536 keys without two tiles per unit
    (RELAY, BF16, 32, 32, 1024, 1536, False, 48, False), (RELAY, BF16, 32, 32, 1024, 1537, False, 48, True),
    (RELAY, BF16, 32, 32, 2048, 1537, False, 48, False), (ANCHOR, BF16, 32, 32, 1024, 1537, False, 48, False),
    (RELAY, BF16, 128, 32, 2048, 1536, True, 48, True), (RELAY, F32, 128, 32, 2048, 1536, False, 48, True),
    # 512-byte rows: from 513 keys, T <= 24, a relay from two tiles per unit
    (FULL, BF16, 256, 32, 1024, 512, False, 24, True), (FULL, BF16, 256, 32, 1024, 513, False, 24, False),
    (FULL, BF16, 256, 32, 1024, 2048, False, 25, True), (RELAY, BF16, 256, 32, 1024, 1024, False, 24, True),
    (RELAY, BF16, 256, 32, 2048, 1024, False, 24, False), (FULL, BF16, 256, 32, 1024, 2049, False, 24, True),
    # panels: bf16 of T <= 64 where 128-row tiles are few, wider ones under the mask or with few tiles
    (ANCHOR, BF16, 128, 32, 1024, 2049, False, 48, False), (ANCHOR, BF16, 128, 16, 1024, 2049, False, 48, True),
    (RELAY, BF16, 128, 32, 2100, 2100, True, 48, False), (RELAY, BF16, 128, 32, 4096, 4096, True, 96, True),
    (RELAY, BF16, 128, 32, 1024, 4096, False, 96, False), (RELAY, BF16, 128, 32, 960, 4096, False, 96, True),
    (RELAY, BF16, 256, 32, 2048, 4096, False, 96, True),
    # binary32 relays of up to 256-byte rows over panels with two tiles per unit
    (RELAY, F32, 64, 32, 2048, 2049, False, 56, False), (RELAY, F32, 64, 32, 2048, 2049, False, 57, True),
    (RELAY, F32, 128, 32, 2048, 2049, False, 48, True), (RELAY, F32, 32, 32, 1920, 2049, False, 48, True),
    (ANCHOR, F32, 64, 32, 2048, 2049, False, 56, True), (RELAY, F32, 64, 32, 2048, 2048, False, 56, True),
]


@pytest.mark.parametrize("line", LINES, ids=["-".join(map(str, x)) for x in LINES])
def test_dispatch_lines(line):
    *args, want = line
    assert pays(*args) == want


def test_a_forced_one_pass_does_not_compare_with_the_split_schedule():
    assert pays(RELAY, BF16, 128, 32, 2048, 1536, False, 48, True)
    assert pays(RELAY, F32, 64, 32, 2048, 2049, False, 48, True)
    assert not pays(RELAY, BF16, 128, 32, 2100, 2100, False, 48, True)


@pytest.mark.parametrize("kw,status", [
    # by the resident tile, where the two-sweep tile's bitmaps end at 1920 (d = 256; binary32 d = 128) ...
    (dict(n_k=2048, d=256, dtype="bf16"), -1), (dict(n_k=4096, d=128), -1),
    # ... or 3072 chunks
    (dict(n_k=4096, d=128, dtype="bf16"), -1),
    # two-sweep tiles: routes that stage more slots than a tile of several panels holds, wide routes past 4096
    (dict(n_k=3072, d=128, dtype="bf16", k=1, m=0, r=255), -1), (dict(n_k=4608, d=64, k=64, m=32), -1),
    # neither
    (dict(n_k=4097, d=128, dtype="bf16"), -5), (dict(n_k=3073, d=128, dtype="bf16", k=1, m=0, r=255), -5),
    (dict(n_k=4609, d=64, k=64, m=32), -5),
])
def test_one_pass_relays_are_refused_where_no_tile_takes_them(kw, status):
    """Null pointers are refused (-1) after the configuration (-5) has been
    looked at, and before anything is launched."""
    from paper_2609_07306_amd import routerelay as rr
    cfg = rr.Config(**{**dict(n_heads=2, n_kv_heads=1, n_q=64, n_k=64, d=64, k=8, m=4, r=4, relay="one_pass"), **kw})
    got = rr.lib.rr_relay_layer_static(ctypes.byref(cfg.c()), 1, *([None] * 11))
    assert got == status, rr.lib.rr_last_error()
