"""Parity of the resident-score route kernel (n_k <= 2048) with the oracle at
the edges of its shapes: key counts around the stage and wave limits (32 waves'
keys, 256, 512, 1024, 2048), ragged last tiles, the widest routes of each class
(k + m = 64, 65, 128), one and many random sentinels (more than the parallel
draws take), routes as wide as the key range, and every input type and width.
Step mode (the oracle's ledger imported before every relay layer), with the
tie bands of parity_util."""
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2609_07306_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.set_device(0)
    yield


def _w(n, d, dtype, k, m, r, causal=False, heads=2, kv=1, nk=0, **kw):
    return synth.preset("drift", n_heads=heads, n_kv_heads=kv, n=n, n_keys=nk, d=d, dtype=dtype, k=k, m=m, r=r,
                        causal=causal, n_layers=3, anchor_every=0, **kw)


CASES = [
    _w(1, 64, "f32", 1, 0, 0, heads=1),
    _w(31, 32, "bf16", 8, 4, 4, causal=True),
    _w(33, 32, "f32", 5, 3, 2, nk=128),
    _w(97, 64, "bf16", 12, 6, 6, causal=True),
    _w(64, 128, "f32", 33, 31, 40, nk=256),            # T = 64, more draws than half the pool
    _w(96, 128, "bf16", 33, 32, 16, nk=257),           # T = 65: eight waves
    _w(65, 64, "f32", 16, 8, 70, nk=512),              # r past the parallel draws
    _w(130, 128, "bf16", 32, 16, 16, causal=True, heads=4, kv=2),
    _w(513, 128, "bf16", 64, 64, 16, causal=True, heads=1),
    _w(40, 256, "bf16", 20, 12, 9, nk=1023),
    _w(70, 128, "f32", 30, 30, 17, nk=1024),
    _w(50, 64, "bf16", 17, 7, 7, nk=1025),
    _w(36, 256, "bf16", 100, 28, 33, nk=2048),
    _w(34, 32, "bf16", 3, 2, 130, nk=2047, n_sink=3, n_recent=2),
    _w(257, 32, "f32", 64, 0, 3, causal=True, n_sink=1, n_recent=4, min_reuse=1),
]


@pytest.mark.parametrize("w", CASES, ids=[f"n{w.n}x{w.nk}-d{w.d}-{w.dtype}-T{w.k + w.m}-r{w.r}{'-causal' if w.causal else ''}"
                                          for w in CASES])
def test_resident_step_parity(w):
    from parity_util import step_compare
    print(w, flush=True)
    st = step_compare(w, note=lambda s: (print(s, flush=True), sys.stdout.flush()))
    assert st["compared"] >= 0.8 * st["rows"]


@pytest.mark.parametrize("n,nk,k,m,r", [(40, 300, 20, 10, 6), (33, 2048, 90, 38, 12), (64, 64, 64, 0, 0)])
def test_resident_exact_ties(n, nk, k, m, r):
    """Small-integer inputs: every score is exact in binary32, rows hold many
    equal scores, more than a row's candidate list takes, and every row has to
    match (lower id first)."""
    from parity_util import dev, ledger_np
    from paper_2609_07306_amd import routerelay as rr
    rng = np.random.default_rng(n + nk)
    for dtype in ("f32", "bf16"):
        print(n, nk, k, m, r, dtype, flush=True)
        Q = rng.integers(-2, 3, size=(2, n, 32)).astype(np.float32)
        Q[:, 1] = 0.0
        K = rng.integers(-1, 2, size=(2, nk, 32)).astype(np.float32)
        Qd, Kd = (synth.bf16_round(Q), synth.bf16_round(K)) if dtype == "bf16" else (Q, K)
        p = oracle.Problem(2, 2, n, nk, 32, k, m, r)
        led = rr.Ledger(rr.Config(2, 2, n, nk, 32, k, m, r, dtype))
        led.anchor(0, dev(Qd, dtype), dev(Kd, dtype))
        ref = oracle.new_ledger(p)
        oracle.anchor(p, 0, Q, K, ref)
        got = ledger_np(led)
        for key in ("routes", "sent", "build", "age"):
            np.testing.assert_array_equal(got[key], ref[key], err_msg=key)
        led.close()


def test_resident_relay_routes_to_unaligned_rows():
    """routes handed out by a relay: rows of an odd width and a buffer that is
    not 16-byte aligned take the element-wise copies."""
    from paper_2609_07306_amd import routerelay as rr
    for k, off in ((7, 0), (8, 1), (8, 0)):
        w = _w(70, 64, "bf16", k, 4, 5, rho=0.05)
        L = [(rr.to_device(q, w.dtype), rr.to_device(kk, w.dtype)) for _, _, _, q, kk in synth.Generator(w)]
        led = rr.Ledger(rr.Config.of(w))
        led.anchor(0, *L[0])
        buf = torch.full((w.rows * k + off,), -7, dtype=torch.int32, device="cuda")
        out = buf[off:].view(w.rows, k)
        for layer in (1, 2):
            led.relay(layer, *L[layer], routes=out)
            assert torch.equal(out, led.export()["routes"]), (k, off, layer)
        led.close()
