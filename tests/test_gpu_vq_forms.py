"""VQ assignment at the edges of its forms: few rows (one row set per wave, buffers of four chunks)
and many, rows that load as float4 and rows that do not, codebooks around whole chunks and buffers.
Indices and distances equal the FP64 definition bit for bit."""
import numpy as np
import pytest

from paper_2604_26799_amd import mgs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    mgs.lib()
    return _t


def check(torch, orc, x, cb):
    idx, dist, _ = mgs.vq_assign(torch.from_numpy(x).cuda(), torch.from_numpy(cb).cuda())
    wi, wd = orc.vq_assign(x, cb)[:2]
    assert np.array_equal(idx.cpu().numpy(), wi)
    assert np.array_equal(dist.cpu().numpy(), wd)


@pytest.mark.parametrize("D", [1, 3, 8, 14, 15, 16, 30, 31, 36, 45, 46, 47, 60, 63, 64])
@pytest.mark.parametrize("N,K", [(1, 1), (127, 63), (129, 64), (300, 255), (1000, 257), (777, 513)])
def test_few_rows(torch, orc, D, N, K):
    rng = np.random.default_rng(D * 1000 + N)
    x = rng.laplace(0, 0.03, (N, D)).astype(np.float32)
    cb = rng.laplace(0, 0.03, (K, D)).astype(np.float32)
    cb[K // 2] = cb[0]  # a tie: the smaller index
    check(torch, orc, x, cb)


@pytest.mark.parametrize("D,N", [(36, 65536), (36, 65537), (45, 65537), (64, 32768), (64, 32769), (63, 32769)])
def test_form_boundary(torch, orc, D, N):
    rng = np.random.default_rng(N + D)
    x = rng.laplace(0, 0.03, (N, D)).astype(np.float32)
    x[-1] *= 1e6  # a row far larger than the codebook: exact scan
    check(torch, orc, x, np.ascontiguousarray(x[rng.choice(N - 1, 130, replace=False)]))


def test_unaligned_rows(torch, orc):
    """D % 4 == 0 with rows and codewords that start off a 16-byte boundary."""
    rng = np.random.default_rng(1)
    x, cb = rng.laplace(0, 0.03, (70_000, 12)).astype(np.float32), rng.laplace(0, 0.03, (99, 12)).astype(np.float32)
    for n in (500, 70_000):
        gx = torch.empty(n * 12 + 1, device="cuda")[1:].view(n, 12).copy_(torch.from_numpy(x[:n]))
        gc = torch.empty(99 * 12 + 1, device="cuda")[1:].view(99, 12).copy_(torch.from_numpy(cb))
        idx, dist, _ = mgs.vq_assign(gx, gc)
        wi, wd = orc.vq_assign(x[:n], cb)[:2]
        assert np.array_equal(idx.cpu().numpy(), wi) and np.array_equal(dist.cpu().numpy(), wd)


@pytest.mark.parametrize("D", [1, 2, 3, 4, 5, 6, 7, 8, 9])
@pytest.mark.parametrize("N,K", [(700, 65), (3000, 1000), (70_000, 300)])
def test_short_rows(torch, orc, D, N, K):
    """Rows of few values, which leave several candidates each (repeated codewords among them), at
    and off 16-byte boundaries."""
    rng = np.random.default_rng(10 * D + K)
    x = rng.laplace(0, 0.03, (N, D)).astype(np.float32)
    cb = rng.laplace(0, 0.03, (K, D)).astype(np.float32)
    cb[K // 3] = cb[K - 1] = cb[2]
    x[::5] = cb[rng.integers(0, K, x[::5].shape[0])]
    wi, wd = orc.vq_assign(x, cb)[:2]
    for xs, cs in ((0, 0), (1, 0), (0, 1), (1, 1)):
        gx = torch.empty(N * D + xs, device="cuda")[xs:].view(N, D).copy_(torch.from_numpy(x))
        gc = torch.empty(K * D + cs, device="cuda")[cs:].view(K, D).copy_(torch.from_numpy(cb))
        idx, dist, _ = mgs.vq_assign(gx, gc)
        assert np.array_equal(idx.cpu().numpy(), wi) and np.array_equal(dist.cpu().numpy(), wd), (xs, cs)
