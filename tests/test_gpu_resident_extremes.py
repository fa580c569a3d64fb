"""Scores at the ends of binary32 through the resident-score route kernel, one
panel of keys and several: zeros of both signs, NaN, ranges wider than the
largest float, infinities; past 4096 keys the two-sweep tiles and the split
relay (without NaN).

The inputs are scaled unit vectors or constants, so that every score is known
exactly; the expected routes are the k highest scores, -0 equal to +0, ties to
the lower id."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.set_device(0)
    yield


def _top(scores, width):
    """Ids of the `width` highest scores of each row, highest first (equal: lower id)."""
    return np.argsort(-scores, axis=1, kind="stable")[:, :width]


def _expected(scores, k, m):
    ids = _top(scores, k + m)
    return np.sort(ids[:, :k], axis=1), np.sort(ids[:, k:k + m], axis=1)


def _check_routing(Q, K, scores, k, m, r, dtype="f32"):
    """Full routing, an anchor, and a relay that refreshes every row, against
    the exact scores [n, n_k] of one head."""
    from parity_util import dev, ledger_np
    from paper_2609_07306_amd import routerelay as rr
    from paper_2609_07306_amd import synth
    n, nk, d = Q.shape[1], K.shape[1], Q.shape[2]
    as_dev = lambda x: dev(synth.bf16_round(x) if dtype == "bf16" else x, dtype)  # noqa: E731
    Qd, Kd = as_dev(Q), as_dev(K)
    R, N = _expected(scores, k, m)
    full = torch.full((n, k), -7, dtype=torch.int32, device="cuda")
    fs = torch.zeros(n, k, device="cuda")
    rr.full_route(rr.Config(1, 1, n, nk, d, k, 0, 0, dtype), Qd, Kd, full, scores=fs)
    np.testing.assert_array_equal(full.cpu().numpy(), R, err_msg="full")
    np.testing.assert_array_equal(fs.cpu().numpy(), np.take_along_axis(scores, R, 1), err_msg="scores")
    led = rr.Ledger(rr.Config(1, 1, n, nk, d, k, m, r, dtype, gamma=np.inf))
    for what in ("anchor", "relay"):
        out = torch.full((n, k), -7, dtype=torch.int32, device="cuda")
        if what == "anchor":
            led.anchor(0, Qd, Kd, routes=out)
        else:
            mask = torch.zeros(n, dtype=torch.uint8, device="cuda")
            led.relay(1, Qd, Kd, routes=out, mask=mask)
            assert bool(mask.all()) or not np.isfinite(scores).all()  # (-inf + gamma is not above anything)
        got = ledger_np(led)
        np.testing.assert_array_equal(out.cpu().numpy(), R, err_msg=f"{what}: routes out")
        np.testing.assert_array_equal(got["routes"], R, err_msg=f"{what}: ledger routes")
        np.testing.assert_array_equal(got["sent"][:, :m], N, err_msg=f"{what}: near misses")
        draws = got["sent"][:, m:]
        assert ((draws >= 0) & (draws < nk)).all(), what
        assert all(len(set(a) | set(b)) == k + m + r for a, b in zip(got["sent"], R)), what
    led.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("nk", [256, 2304])
def test_zeros_of_both_signs(nk, dtype):
    """Products that underflow to -0 beside +0: every second block of 16 keys.
    The blocks are a stage apart, so each kept maximum is a +0 and so is the
    row's threshold, which the -0 scores reach as well."""
    n, d, k, m, r = 40, 32, 40, 20, 8
    Q = np.full((1, n, d), 2.0 ** -100, np.float32)
    K = np.zeros((1, nk, d), np.float32)
    K[0, (np.arange(nk) >> 4) % 2 == 1] = -2.0 ** -100
    s = np.zeros((n, nk), np.float32)
    _check_routing(Q, K, s, k, m, r, dtype)


@pytest.mark.parametrize("nk,good", [(700, 600), (700, 12), (2304, 2000), (2304, 0)])
def test_nan_scores_are_not_routed(nk, good):
    """Chunks whose representation holds a NaN rank with those of -inf: no row
    routes to them while it has others, and every id handed out is one of the
    head's chunks."""
    n, d, k, m, r = 40, 32, 30, 10, 16
    rng = np.random.default_rng(nk)
    Q = rng.integers(-2, 3, size=(1, n, d)).astype(np.float32)
    Q[:, :, 0] = 1.0
    K = rng.integers(-1, 2, size=(1, nk, d)).astype(np.float32)
    s = (Q[0] @ K[0].T).astype(np.float32)  # small integers: exact
    bad = rng.choice(nk, nk - good, replace=False)
    K[0, bad, 0] = np.where(np.arange(len(bad)) % 2, np.nan, -np.nan)
    s[:, bad] = -np.inf
    _check_routing(Q, K, s, k, m, r)


def _column(nk, values):
    """Keys whose only component is `values`: a query (q, 0, ...) scores q * values."""
    K = np.zeros((1, nk, 32), np.float32)
    K[0, :, 0] = values
    return K


def _queries(n, q):
    Q = np.zeros((1, n, 32), np.float32)
    Q[0, :, 0] = q
    return Q


@pytest.mark.parametrize("nk", [100, 600, 2304, 4200])
def test_finite_scores_wider_than_the_largest_float(nk):
    """Rows whose highest and lowest scores lie further apart than the largest
    finite float, the highest T close together or not."""
    n, k, m, r = 40, 30, 10, 8
    rng = np.random.default_rng(nk)
    v = np.where(rng.random(nk) < 0.5, 1.0, -1.0) * (2e38 + 1e32 * rng.permutation(nk))
    v[::7] *= 1e-3
    q = np.where(np.arange(n) % 3 == 0, -1.0, 1.0) * np.where(np.arange(n) % 5 == 0, 1e-38, 1.0)
    K, Q = _column(nk, v.astype(np.float32)), _queries(n, q.astype(np.float32))
    s = Q[0, :, :1] * K[0, :, 0][None, :]
    assert np.isfinite(s).all()
    _check_routing(Q, K, s, k, m, r)


@pytest.mark.parametrize("nk,hot", [(100, 50), (600, 45), (600, 500), (2304, 60), (2304, 1500), (4200, 60), (4200, 2500)])
def test_infinite_scores(nk, hot):
    """Products that overflow to +inf: as many as a row selects and more, in a
    row's list or past it, beside rows where the same chunks are finite."""
    n, k, m, r = 40, 30, 10, 8
    rng = np.random.default_rng(nk + hot)
    v = rng.permutation(nk).astype(np.float32)
    v[rng.choice(nk, hot, replace=False)] = 3e38
    K, Q = _column(nk, v), _queries(n, np.where(np.arange(n) % 3 == 1, 1.0, 4.0).astype(np.float32))
    with np.errstate(over="ignore"):
        s = Q[0, :, :1] * K[0, :, 0][None, :]
    assert np.isposinf(s[0]).sum() == hot and np.isfinite(s[1]).all()
    _check_routing(Q, K, s, k, m, r)


@pytest.mark.parametrize("nk,finite", [(100, 20), (600, 0), (600, 39), (2304, 5), (4096, 0), (4200, 0), (4200, 36)])
def test_valid_chunks_of_minus_infinity(nk, finite):
    """Rows with fewer finite scores than they select (products that overflow to
    -inf) take the lowest ids of the others, beside rows of finite scores."""
    n, k, m, r = 40, 30, 10, 8
    rng = np.random.default_rng(nk + finite)
    v = np.full(nk, -3e38, np.float32)
    v[rng.choice(nk, finite, replace=False)] = rng.permutation(finite).astype(np.float32) - 3
    K, Q = _column(nk, v), _queries(n, np.where(np.arange(n) % 3 == 1, 1.0, 4.0).astype(np.float32))
    with np.errstate(over="ignore"):
        s = Q[0, :, :1] * K[0, :, 0][None, :]
    assert np.isfinite(s[0]).sum() == finite and np.isfinite(s[1]).all()
    _check_routing(Q, K, s, k, m, r)


@pytest.mark.parametrize("n", [300, 2200, 4200])
def test_minus_infinity_under_the_causal_mask(n):
    """... and never a chunk past the row's position, which the mask also gives -inf."""
    from paper_2609_07306_amd import routerelay as rr
    k = 40
    v = np.full(n, -3e38, np.float32)
    v[::11] = np.arange(len(v[::11]))
    Q, K = _queries(n, np.full(n, 4.0, np.float32)), _column(n, v)
    with np.errstate(over="ignore"):
        s = np.tile(4.0 * v, (n, 1))
    routes = torch.full((n, k), -7, dtype=torch.int32, device="cuda")
    rr.full_route(rr.Config(1, 1, n, n, 32, k, 0, 0, "f32", True), torch.from_numpy(Q).cuda(), torch.from_numpy(K).cuda(),
                  routes)
    want = np.full((n, k), -1, np.int32)
    for i in range(n):
        ids = np.sort(np.argsort(-s[i, :i + 1], kind="stable")[:k])
        want[i, :len(ids)] = ids
    np.testing.assert_array_equal(routes.cpu().numpy(), want)
