"""Token expansion against the oracle at the edges of its launch: one-token
and very long chunks, chunks that no piece of four aligns with, slots at the
span limits, short outputs, unaligned output buffers, empty and out-of-range
slots."""
import numpy as np
import pytest
import torch

from oracle import consumer as oc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.set_device(0)
    yield


@pytest.mark.parametrize("rows,k,chunk,n_tok", [(1, 1, 1, 1), (3, 5, 1, 7), (7, 3, 3, 100), (65, 9, 5, 333), (41, 7, 48, 1000),
                                                (3, 2, 1025, 5000), (2, 3, 70001, 200000), (700, 16, 64, 4096),
                                                (8300, 32, 33, 16384)])
@pytest.mark.parametrize("offset", [0, 1])
def test_expand_edges(rows, k, chunk, n_tok, offset):
    from paper_2609_07306_amd import routerelay as rr
    rng = np.random.default_rng(rows * 7 + k)
    nc = oc.n_chunks(n_tok, chunk)
    routes = rng.integers(-1, nc + 2, size=(rows, k)).astype(np.int32)
    print(rows, k, chunk, n_tok, offset, flush=True)
    buf = torch.full((rows * k * chunk + offset + 8,), -9, dtype=torch.int32, device="cuda")
    out = buf[offset:offset + rows * k * chunk].view(rows, k * chunk)
    rr.expand_tokens(torch.from_numpy(routes).cuda(), chunk, n_tok, out=out)
    np.testing.assert_array_equal(out.cpu().numpy(), oc.expand_tokens(routes, chunk, n_tok))
    assert (buf[:offset] == -9).all() and (buf[offset + rows * k * chunk:] == -9).all()
