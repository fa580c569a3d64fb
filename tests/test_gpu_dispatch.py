"""Parity of what the dispatch leaves to the 128-row two-sweep tiles and the
split relays at key counts the resident-score tile takes as well, on a subset
of the heads (the tests of that tile and the small cases of the two-sweep
kernels have too few rows to get here; tests/test_dispatch.py pins the rule)."""
import sys

import pytest
import torch

from paper_2609_07306_amd import synth
from test_dispatch import ANCHOR, BF16, F32, RELAY, pays

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.set_device(0)
    yield


def note(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _w(n, nk, d, dtype, k, m, r, causal=False, heads=32, kv=32, **kw):
    return synth.preset("drift", n_heads=heads, n_kv_heads=kv, n=n, n_keys=nk, d=d, dtype=dtype, k=k, m=m, r=r,
                        causal=causal, n_layers=3, anchor_every=0, **kw)


def _pays(w, mode):
    return pays(mode, BF16 if w.dtype == "bf16" else F32, w.d, w.n_heads, w.n, w.nk, w.causal, w.k + w.m)


MANY_ROWS = [
    # (workload, anchors by the resident tile)
    (_w(1024, 1025, 128, "bf16", 32, 16, 16), False),
    (_w(1030, 2047, 32, "bf16", 36, 16, 16, heads=30, kv=15, rho=0.01), False),
    (_w(2048, 513, 256, "bf16", 16, 8, 8), False),
    (_w(2000, 2100, 64, "f32", 32, 24, 16, rho=0.02), True),
]


@pytest.mark.parametrize("w,anchor", MANY_ROWS, ids=[f"{w.n}x{w.nk}-d{w.d}-{w.dtype}-T{w.k + w.m}" for w, _ in MANY_ROWS])
def test_many_rows_relay_by_the_split_schedule(w, anchor):
    from parity_util import step_compare
    assert _pays(w, ANCHOR) == anchor and not _pays(w, RELAY)
    note(w)
    st = step_compare(w, heads=[1, w.n_heads - 2], note=note)
    assert st["compared"] >= 0.8 * st["rows"] and st["rerouted"] > 0


def test_static_relay_past_the_split_schedules_scratch():
    """More rows than the static area holds threshold seeds for: the relay runs
    as one pass there, with the ledger's results (small integers, exact)."""
    from paper_2609_07306_amd import routerelay as rr
    heads, n, nk, d = 32, 8192, 1100, 32
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    draw = lambda *s: torch.randint(-3, 4, s, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    Q, K, Q2 = draw(heads, n, d), draw(heads, nk, d), draw(heads, n, d)
    cfg = rr.Config(heads, heads, n, nk, d, 8, 4, 4, "bf16")
    assert not pays(RELAY, BF16, d, heads, n, nk, False, 12)
    led = rr.Ledger(cfg)
    led.anchor(0, Q, K)
    own = led.export()
    mask, mask2 = (torch.empty(cfg.rows, dtype=torch.uint8, device="cuda") for _ in range(2))
    led.relay(1, Q2, K, mask=mask)
    out = torch.empty(cfg.rows, cfg.k, dtype=torch.int32, device="cuda")
    rr.relay_static(cfg, 1, Q2, K, own, routes=out, mask=mask2)
    want = led.export()
    assert 0 < int(mask.sum()) and torch.equal(mask, mask2)
    for key in want:
        assert torch.equal(want[key], own[key]), key
    assert torch.equal(out, want["routes"])
    led.close()


ONE_PASS = [_w(70, 2000, 256, "bf16", 32, 16, 16, heads=2, kv=1), _w(1024, 3200, 128, "bf16", 32, 16, 16)]


@pytest.mark.parametrize("w", ONE_PASS, ids=[f"{w.n}x{w.nk}-d{w.d}" for w in ONE_PASS])
def test_forced_one_pass_where_only_the_resident_tile_fits(w):
    from parity_util import step_compare
    note(w)
    st = step_compare(w, heads=[0, w.n_heads - 1], relay="one_pass", note=note)
    # (by the oracle's scores alone 84 of the 140 rows of the d = 256 case's first
    # layer lie outside the tie bands, which grow with d: 2 d 2^-24 sum |q k|)
    assert st["compared"] >= 0.55 * st["rows"] and st["rerouted"] > 0
