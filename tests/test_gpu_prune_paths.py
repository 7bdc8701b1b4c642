"""Prune select around the sizes where its form changes (one kernel with 16 or 64 keys per thread,
the general path), with ties across thresholds, shared digits and more counts than LDS rows.
Kept sets are exact."""
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


def importance(kind, n, seed):
    rng = np.random.default_rng(seed)
    if kind == "spread":
        return rng.lognormal(0, 2, n).astype(np.float32)
    if kind == "tied":
        return np.round(rng.lognormal(0, 1, n) * 2).astype(np.float32)
    if kind == "constant":
        return np.full(n, 0.75, np.float32)
    if kind == "close":  # one first digit, few last ones
        return (np.float32(1.0) + rng.integers(0, 3000, n).astype(np.float32) * np.float32(2 ** -23)).astype(np.float32)
    v = rng.normal(0, 1, n).astype(np.float32)  # both signs, both zeros
    v[rng.random(n) < 0.2] = 0.0
    v[rng.random(n) < 0.2] = -0.0
    return v


@pytest.mark.parametrize("n", [1, 63, 64, 1023, 1025, 16383, 16384, 16385, 65535, 65536, 65537, 262_147, 1_000_001])
@pytest.mark.parametrize("kind", ["spread", "tied", "constant", "close", "signed"])
def test_sizes_and_ties(torch, orc, n, kind):
    imp = importance(kind, n, n)
    rng = np.random.default_rng(n + 1)
    k = np.concatenate([[0, n, 1, n - 1, n // 2, n // 2], rng.integers(0, n + 1, 6)]).clip(0, n).astype(np.int64)
    got = mgs.prune_select(torch.from_numpy(imp).cuda(), k).cpu().numpy()
    np.testing.assert_array_equal(got, orc.prune_select(imp, k))


@pytest.mark.parametrize("kind", ["spread", "tied", "close"])
@pytest.mark.parametrize("T", [1, 32, 33, 58, 59, 64])
def test_many_counts(torch, orc, kind, T):
    n = 120_007
    imp = importance(kind, n, T)
    k = np.random.default_rng(T).integers(0, n + 1, T).astype(np.int64)
    got = mgs.prune_select(torch.from_numpy(imp).cuda(), k).cpu().numpy()
    np.testing.assert_array_equal(got, orc.prune_select(imp, k))


@pytest.mark.parametrize("n", [70_001, 300_000])
def test_unaligned_importance(torch, orc, n):
    """An importance array that starts 4, 8 or 12 bytes past a 16-byte boundary."""
    imp = importance("spread", n + 3, 5)
    base = torch.from_numpy(imp).cuda()
    for off in (1, 2, 3):
        k = np.array([n // 3, n // 7], np.int64)
        got = mgs.prune_select(base[off:off + n], k).cpu().numpy()
        np.testing.assert_array_equal(got, orc.prune_select(imp[off:off + n], k))


@pytest.mark.parametrize("n", [300, 50_000, 90_000])
@pytest.mark.parametrize("bad", [np.nan, -np.nan, np.inf, -np.inf])
def test_nonfinite_then_clean(torch, orc, n, bad):
    """Non-finite importance raises the flag, nothing is written past the kept sets, and the next call
    on the same workspace is clean."""
    imp = importance("spread", n, 3)
    k = np.array([n // 2, n], np.int64)
    ws = mgs.workspace(mgs.lib().mgs_prune_select_ws_bytes(n, 2))
    out = torch.full((int(k.sum()) + 64,), -7, dtype=torch.int32, device="cuda")
    spoilt = imp.copy()
    spoilt[n // 3] = bad
    with pytest.raises(mgs.MgsError) as e:
        mgs.prune_select(torch.from_numpy(spoilt).cuda(), k, ws=ws, out=out)
    assert e.value.code == mgs.ENONFINITE
    assert (out[int(k.sum()):] == -7).all()
    got = mgs.prune_select(torch.from_numpy(imp).cuda(), k, ws=ws, out=out[:int(k.sum())]).cpu().numpy()
    np.testing.assert_array_equal(got, orc.prune_select(imp, k))


@pytest.mark.parametrize("n", [64, 700, 16384, 16385, 50_000, 65_536])
@pytest.mark.parametrize("crowd", [1, 7, 8, 9, 40, 64])
def test_crowded_bins(torch, orc, n, crowd):
    """Up to `crowd` of every 64 keys in one bin (equal, or close together), in the first lanes or from
    the middle on; thresholds inside the crowd, beside it and at its edges."""
    rng = np.random.default_rng(n + crowd)
    for shift in (0, 32):
        imp = rng.lognormal(0, 2, n).astype(np.float32)
        lane = (np.arange(n) - shift) % 64
        hit = (lane < crowd) & (rng.random(n) < 0.95)
        imp[hit] = np.float32(0.5)
        near = hit & (rng.random(n) < 0.3)
        imp[near] += rng.integers(0, 5, int(near.sum())).astype(np.float32) * np.float32(2 ** -24)
        above, below = int((imp > 0.6).sum()), int((imp >= 0.5).sum())
        k = np.array([0, n, above, below, (above + below) // 2, n // 2, max(below - 1, 0)], np.int64)
        got = mgs.prune_select(torch.from_numpy(imp).cuda(), k).cpu().numpy()
        np.testing.assert_array_equal(got, orc.prune_select(imp, k))
