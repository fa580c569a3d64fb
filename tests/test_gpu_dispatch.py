"""Parity of what the dispatch leaves to the 128-row two-sweep tiles and the
split relays at key counts the resident-score tile takes as well, on a subset
of the heads (the tests of that tile and the small cases of the two-sweep
kernels have too few rows to get here; tests/test_dispatch.py pins the rule)."""
import sys

import pytest
import torch

from paper_2609_07306_amd import synth
from test_dispatch import ANCHOR, BF16, F32, FULL, RELAY, pays, shape

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
    (_w(1030, 2047, 64, "bf16", 36, 16, 16, heads=30, kv=15, rho=0.01), False),
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


TWO_SWEEP = [
    # one-pass relays over two-sweep tiles: 128-row; 64-row past 4096 chunks; 32-row (more staged slots than
    # a tile of several panels holds)
    (_w(2100, 2100, 128, "bf16", 32, 16, 16, causal=True, heads=16, kv=4, rho=0.1), [3, 14], "relay"),
    (_w(4200, 4200, 64, "bf16", 64, 32, 16, causal=True, heads=2, kv=1, rho=0.1), [1], "relay"),
    (_w(2100, 2100, 64, "f32", 1, 0, 255, causal=True, heads=1, kv=1), [0], "relay"),
    # 128-row anchors, split relays, without and (past the bitmaps) with the mask
    (_w(1024, 4096, 128, "bf16", 32, 16, 16), [0, 31], "rescore"),
    (_w(4096, 4096, 128, "bf16", 32, 16, 16, causal=True, heads=16, kv=16), [9], "rescore"),
]


@pytest.mark.parametrize("w,heads,kind", TWO_SWEEP,
                         ids=[f"{w.n}x{w.nk}-T{w.k + w.m}{'-causal' if w.causal else ''}" for w, _, _ in TWO_SWEEP])
def test_two_sweep_tiles_that_the_resident_tile_leaves(w, heads, kind):
    from parity_util import step_compare
    from paper_2609_07306_amd import routerelay as rr
    applies = shape(w.nk, w.k, w.m, w.r) != 0
    assert not applies or not (_pays(w, ANCHOR) or _pays(w, RELAY))
    note(w)
    rr.profile_start()
    st = step_compare(w, heads=heads, note=note)
    launched = {k for k, (_, n) in rr.profile_stop().items() if n}
    assert launched == {"anchor", "relay"} if kind == "relay" else launched == {"anchor", "rescore", "reroute"}
    assert st["compared"] >= 0.5 * st["rows"] and st["rerouted"] > 0


@pytest.mark.parametrize("nk,k", [(1500, 32), (2100, 48), (4097, 20)])
def test_full_routing_by_128_row_tiles(nk, k):
    """Every row of 32 heads, on small integers (scores exact, ties to the lower id)."""
    from paper_2609_07306_amd import routerelay as rr
    heads, n, d = 32, 1000, 64
    assert nk > 4096 or not pays(FULL, BF16, d, heads, n, nk, False, k)
    g = torch.Generator(device="cuda")
    g.manual_seed(nk)
    Q, K = (torch.randint(-3, 4, (heads, x, d), generator=g, device="cuda").float() for x in (n, nk))
    routes = torch.empty(heads * n, k, dtype=torch.int32, device="cuda")
    scores = torch.empty(heads * n, k, device="cuda")
    rr.full_route(rr.Config(heads, heads, n, nk, d, k, 0, 0, "bf16"), Q.bfloat16(), K.bfloat16(), routes, scores=scores)
    for h in range(heads):
        S = Q[h] @ K[h].t().contiguous()
        ids = torch.sort(torch.sort(S, dim=1, descending=True, stable=True).indices[:, :k], dim=1).values
        assert torch.equal(routes[h * n:(h + 1) * n].long(), ids), h
        assert torch.equal(scores[h * n:(h + 1) * n], torch.gather(S, 1, ids)), h


def test_two_sweep_rows_stopped_at_the_cap():
    """At a cap of one sweep the rows of equal scores keep no candidate and are
    counted, the others are exact (more chunks than the resident tile takes)."""
    from paper_2609_07306_amd import routerelay as rr
    n, nk, k = 33, 4200, 16
    assert shape(nk, k) == 0
    Q = torch.zeros(1, n, 32, device="cuda")
    K = torch.zeros(1, nk, 32, device="cuda")
    Q[:, ::2, 0] = 1.0
    K[:, :, 0] = torch.arange(nk, device="cuda") / 64.0
    routes = torch.empty(n, k, dtype=torch.int32, device="cuda")
    before = rr.unconverged_rows()
    try:
        rr.set_sweep_cap(1)
        rr.full_route(rr.Config(1, 1, n, nk, 32, k, 0, 0, "f32"), Q, K, routes)
        torch.cuda.synchronize()
    finally:
        rr.set_sweep_cap(0)
    got = routes.cpu()
    stopped = (got == -1).all(1)
    assert rr.unconverged_rows() - before == int(stopped.sum()) and bool(stopped[1::2].all())
    want = torch.arange(nk - k, nk, dtype=torch.int32)
    assert all(torch.equal(row, want) for row in got[~stopped])


def test_two_sweep_zeros_of_both_signs():
    """-0 equals +0: every score is a zero, the +0 ones just as many as the
    threshold sweep keeps (two per register slot of each of four key segments),
    the others products that underflow to -0.  Ties to the lower id."""
    from paper_2609_07306_amd import routerelay as rr
    n, nk, d, k = 40, 4352, 32, 40
    assert shape(nk, k) == 0
    Q = torch.full((1, n, d), 2.0 ** -100, device="cuda")
    K = torch.full((1, nk, d), -2.0 ** -100, device="cuda")
    stage = torch.arange(nk, device="cuda") % (nk // 4) // 16
    K[0, (stage == 3) | (stage == 7)] = 0.0
    routes = torch.empty(n, k, dtype=torch.int32, device="cuda")
    scores = torch.empty(n, k, device="cuda")
    rr.full_route(rr.Config(1, 1, n, nk, d, k, 0, 0, "f32"), Q, K, routes, scores=scores)
    assert bool((scores == 0).all())
    assert torch.equal(routes.cpu(), torch.arange(k, dtype=torch.int32).expand(n, k))
