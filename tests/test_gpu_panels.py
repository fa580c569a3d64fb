"""Parity of the resident-score route kernel over several panels of keys (2048 <
n_k <= 4096) with the oracle: key counts at the ends of the range and of a
panel, causal tiles of one, two and three panels, the widest routes, few and
many random sentinels (also more than the parallel draws take, and more staged
slots than a tile of several panels holds), every input type and width, equal scores
across the panels, and a row that stops at the collection cap."""
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


# (workload, least share of rows compared).  Rows inside the tie bands are left
# out, which the inputs alone decide (by the oracle's scores): near the boundary
# of 4096 normal scores neighbours lie about 1 / (4096 * 0.05) = 5e-3 standard
# deviations apart, closer in a row's own cluster; the band is 1e-4 of the score
# plus the product's rounding bound 2 d 2^-24 sum |q k|, at two boundaries (k and
# T).  So wide rows and wide routes lose up to four tenths, narrow ones few.
CASES = [
    (_w(40, 128, "bf16", 64, 32, 32, nk=2049), 0.75),
    (_w(33, 64, "bf16", 8, 4, 4, nk=2304), 0.9),        # nine stages: three panels of three
    (_w(65, 128, "f32", 32, 16, 16, nk=3000), 0.75),
    (_w(31, 32, "f32", 100, 28, 40, nk=4095), 0.75),
    (_w(36, 256, "bf16", 20, 108, 9, nk=4096), 0.55),
    (_w(34, 32, "bf16", 3, 2, 130, nk=4000, n_sink=3, n_recent=2), 0.95),  # r past the parallel draws
    (_w(34, 64, "f32", 1, 0, 255, nk=2500), 0.99),      # more slots than several panels stage
    (_w(2100, 128, "bf16", 64, 32, 32, causal=True, heads=1), 0.9),
    (_w(4096, 32, "bf16", 16, 8, 8, causal=True, heads=1, n_sink=1, n_recent=4, min_reuse=1), 0.9),
]


@pytest.mark.parametrize("w,floor", CASES, ids=[f"n{w.n}x{w.nk}-d{w.d}-{w.dtype}-T{w.k + w.m}-r{w.r}{'-causal' if w.causal else ''}"
                                                for w, _ in CASES])
def test_panels_step_parity(w, floor):
    from parity_util import step_compare
    print(w, flush=True)
    st = step_compare(w, note=lambda s: (print(s, flush=True), sys.stdout.flush()))
    assert st["compared"] >= floor * st["rows"]


@pytest.mark.parametrize("nk,k,m,r,ones", [(4096, 90, 38, 12, None), (2500, 64, 0, 40, None), (4096, 64, 32, 8, "late"),
                                           (4096, 64, 32, 8, "last")])
def test_panels_exact_ties(nk, k, m, r, ones):
    """Small-integer inputs: every score is exact in binary32, and the boundary
    rank falls among equal scores of all three panels (4096 keys: 1536, 1536 and
    1024 of them), lower id first.  `late`: among scores that the second and the
    third panel hold above the first's; `last`: among the third's alone, with
    fewer, higher ones that the list carries over from the first two."""
    from parity_util import dev, ledger_np
    from paper_2609_07306_amd import routerelay as rr
    n = 40
    rng = np.random.default_rng(nk + k)
    Q = rng.integers(-2, 3, size=(2, n, 32)).astype(np.float32)
    Q[:, 1] = 0.0
    K = rng.integers(-1, 2, size=(2, nk, 32)).astype(np.float32)
    if ones:
        Q[:, 2:] = 1.0
        K[:] = 0.0
    if ones == "late":
        K[:, 3000:, 0] = 1.0
        K[:, 3500:3530, 1] = 1.0
    elif ones == "last":
        K[:, 3100:, 0] = 1.0
        K[:, 700:720, :2] = 1.0
        K[:, 2000:2015, :3] = 1.0
    p = oracle.Problem(2, 2, n, nk, 32, k, m, r)
    led = rr.Ledger(rr.Config(2, 2, n, nk, 32, k, m, r, "bf16"))
    led.anchor(0, dev(synth.bf16_round(Q), "bf16"), dev(synth.bf16_round(K), "bf16"))
    ref = oracle.new_ledger(p)
    oracle.anchor(p, 0, Q, K, ref)
    got = ledger_np(led)
    for key in ("routes", "sent", "build", "age"):
        np.testing.assert_array_equal(got[key], ref[key], err_msg=key)
    led.close()


def test_panels_scores_and_budgets():
    """Full routing with slot scores and per-row widths."""
    from paper_2609_07306_amd import routerelay as rr
    rng = np.random.default_rng(5)
    n, nk, k = 45, 3333, 60
    Q = rng.standard_normal((2, n, 64)).astype(np.float32)
    K = rng.standard_normal((1, nk, 64)).astype(np.float32)
    kr = rng.integers(1, k + 1, size=2 * n).astype(np.int32)
    cfg = rr.Config(2, 1, n, nk, 64, k, 0, 0, "f32", k_rows=torch.from_numpy(kr).cuda())
    routes = torch.empty(2 * n, k, dtype=torch.int32, device="cuda")
    scores = torch.empty(2 * n, k, device="cuda")
    rr.full_route(cfg, torch.from_numpy(Q).cuda(), torch.from_numpy(K).cuda(), routes, scores=scores)
    S = (Q.astype(np.float64) @ K[0].astype(np.float64).T).reshape(2 * n, nk)
    # binary32 sums of 64 products: |error| <= 64 * 2^-24 * sum |q k|
    bound = 64 * 2.0 ** -24 * (np.abs(Q).astype(np.float64) @ np.abs(K[0]).astype(np.float64).T).reshape(2 * n, nk)
    R, F = routes.cpu().numpy(), scores.cpu().numpy()
    for i in range(2 * n):
        ids = R[i][R[i] >= 0]
        assert len(ids) == kr[i] and np.all(np.diff(ids) > 0) and np.all(np.isneginf(F[i][kr[i]:]))
        assert np.all(np.abs(F[i][:kr[i]] - S[i, ids]) <= bound[i, ids])
        rest = np.setdiff1d(np.arange(nk), ids)
        assert S[i, ids].min() >= S[i, rest].max() - 2 * bound[i].max()


def test_panels_sweep_cap_counts_rows_once():
    """Rows whose first panel overflows its list at a cap of one sweep keep no
    candidate, and count once."""
    from paper_2609_07306_amd import routerelay as rr
    n, nk, k = 33, 4096, 16
    Q = torch.zeros(1, n, 32, device="cuda")
    K = torch.zeros(1, nk, 32, device="cuda")
    Q[:, ::2, 0] = 1.0
    K[:, :, 0] = torch.arange(nk, device="cuda") / 64.0
    routes = torch.empty(n, k, dtype=torch.int32, device="cuda")
    cfg = rr.Config(1, 1, n, nk, 32, k, 0, 0, "f32")
    before = rr.unconverged_rows()
    try:
        rr.set_sweep_cap(1)
        rr.full_route(cfg, Q, K, routes)
        torch.cuda.synchronize()
        assert rr.unconverged_rows() - before == n // 2  # the rows of equal scores
    finally:
        rr.set_sweep_cap(0)
    got = routes.cpu().numpy()
    assert (got[1::2] == -1).all()
    np.testing.assert_array_equal(got[::2], np.tile(np.arange(nk - k, nk), ((n + 1) // 2, 1)))
