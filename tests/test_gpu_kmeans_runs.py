"""Mini-batch k-means: the grouping of a batch by center at the edges of its tiles, of its key bits
and of the counters in LDS (more centers take the radix sort), and runs around the row chunks of
the center update.  Centers, counts and assignments equal the oracle's batched running mean bit for
bit."""
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


def check(torch, orc, x, cb, counts, batch, shift=0):
    n, D = x.shape
    xd = torch.empty(n * D + shift, device="cuda")[shift:].view(n, D).copy_(torch.from_numpy(x))
    cd, vd = torch.from_numpy(cb).cuda(), torch.from_numpy(counts).cuda()
    a = mgs.kmeans_step(xd, cd, vd, torch.from_numpy(batch).cuda())
    wc, wv, wa = orc.kmeans_step_batched(x, cb, counts, batch)
    assert np.array_equal(a.cpu().numpy(), wa)
    assert np.array_equal(vd.cpu().numpy(), wv)
    assert np.array_equal(cd.cpu().numpy(), wc)


@pytest.mark.parametrize("B", [1, 63, 255, 256, 257, 65536, 65537])
@pytest.mark.parametrize("D,K,shift", [(1, 1, 0), (8, 3, 0), (8, 16, 1), (45, 17, 0), (64, 64, 0)])
def test_tiles(torch, orc, B, D, K, shift):
    rng = np.random.default_rng(B + D)
    x = rng.laplace(0, 1, (5000, D)).astype(np.float32)
    cb = rng.laplace(0, 1, (K, D)).astype(np.float32)
    check(torch, orc, x, cb, rng.integers(0, 9, K), rng.integers(0, 5000, B), shift)


@pytest.mark.parametrize("K", [255, 256, 16383, 16384, 16385])
def test_many_centers(torch, orc, K):
    rng = np.random.default_rng(K)
    x = rng.laplace(0, 1, (4000, 4)).astype(np.float32)
    cb = rng.laplace(0, 1, (K, 4)).astype(np.float32)
    check(torch, orc, x, cb, np.zeros(K, np.int64), rng.integers(0, 4000, 3000))


def test_run_lengths(torch, orc):
    """Centers far apart whose runs are 0, 1, .. rows around the chunks of 32 and 64, in mixed order."""
    lens = [0, 1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 2000]
    rng = np.random.default_rng(3)
    cb = (np.arange(len(lens))[:, None] * np.full((1, 12), 50.0)).astype(np.float32)
    own = rng.permutation(np.repeat(np.arange(len(lens)), lens))
    x = (cb[own] + rng.normal(0, 1, (own.size, 12))).astype(np.float32)
    check(torch, orc, x, cb, np.arange(len(lens), dtype=np.int64), rng.permutation(own.size))


@pytest.mark.parametrize("B,K,B1,K1", [
    (65536, 64, 65537, 64),     # the tile grows: fewer tiles, a smaller table in use
    (300, 16384, 300, 16385),   # the last codebook of the counting sort, the first of the radix sort
])
def test_workspace_of_a_larger_call(torch, B, K, B1, K1):
    """A workspace sized for a larger batch or codebook serves the smaller call."""
    L = mgs.lib()
    g = torch.Generator(device="cuda").manual_seed(B)
    x = torch.randn(1000, 4, device="cuda", generator=g)
    batch = torch.randint(0, 1000, (B,), device="cuda", generator=g)
    ws = mgs.workspace(L.mgs_kmeans_step_ws_bytes(B1, 4, K1), x.device)
    out = []
    for held in (True, False):
        cb = torch.randn(K, 4, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
        counts = torch.zeros(K, dtype=torch.int64, device="cuda")
        if held:
            assert L.mgs_kmeans_step(x.data_ptr(), 1000, 4, batch.data_ptr(), B, cb.data_ptr(), K,
                                     counts.data_ptr(), None, ws.data_ptr(), ws.numel(),
                                     torch.cuda.current_stream().cuda_stream) == mgs.OK
            assert mgs.status(ws) == mgs.OK
        else:
            mgs.kmeans_step(x, cb, counts, batch)
        out.append((cb, counts))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("K", [1, 2, 3, 64, 65])
def test_places_shared_by_lanes(torch, orc, K):
    """Wavefronts of 64 rows whose centers repeat in every pattern of lanes (all one center, two in
    turn, 64 of them, ..), in one and in several steps of a wavefront: the rows of a center that meet
    in a wavefront take consecutive places, in batch order."""
    cb = (np.arange(K)[:, None] * np.full((1, 5), 40.0)).astype(np.float32)
    rng = np.random.default_rng(K)
    for B in (64, 1024, 5000):
        own = np.concatenate([np.arange(B // 2) % K, np.repeat(np.arange(K), -(-B // K))])[:B]
        x = (cb[own] + rng.normal(0, 1, (B, 5)) * np.float32(10.0) ** rng.integers(-6, 1, (B, 1))).astype(np.float32)
        check(torch, orc, x, cb, np.zeros(K, np.int64), np.arange(B))
