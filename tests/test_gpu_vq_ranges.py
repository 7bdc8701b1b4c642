"""VQ assignment over the whole range of FP32: values whose squares underflow or overflow in FP32,
subnormal values, and codebooks whose norms exceed the largest FP32 number.  Indices and distances
equal the FP64 definition bit for bit."""
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
    idx, dist, nfb = mgs.vq_assign(torch.from_numpy(x).cuda(), torch.from_numpy(cb).cuda())
    wi, wd = orc.vq_assign(x, cb)[:2]
    wrong = np.flatnonzero(idx.cpu().numpy() != wi)
    assert wrong.size == 0, f"{wrong.size} wrong indices"
    assert np.array_equal(dist.cpu().numpy(), wd)
    return int(nfb.item())


@pytest.mark.parametrize("D", [3, 36])
@pytest.mark.parametrize("scale", [1e-44, 1e-40, 1e-30, 1e-27, 1e-24, 3e-24, 1e-20, 1e-15, 1e15, 1e20, 1e30, 1e36])
def test_scales(torch, orc, D, scale):
    rng = np.random.default_rng(D)
    x = (rng.laplace(0, 1, (4000, D)) * scale).astype(np.float32)
    cb = (rng.laplace(0, 1, (1024, D)) * scale).astype(np.float32)
    # no row leaves FP16 at its codebook's scale; only ties (subnormal values) may fill a row's list
    fallback = check(torch, orc, x, cb)
    assert fallback == 0 or scale < 1e-38


@pytest.mark.parametrize("D", [3, 36])
def test_rows_far_below_the_codebook(torch, orc, D):
    """Rows of every magnitude down to zero and subnormal values, against one codebook."""
    rng = np.random.default_rng(D + 1)
    x = (rng.laplace(0, 1, (3000, D)) * 10.0 ** rng.uniform(-45, 0, (3000, 1))).astype(np.float32)
    x[::97] = 0.0
    check(torch, orc, x, rng.laplace(0, 1, (300, D)).astype(np.float32))


@pytest.mark.parametrize("D", [36, 64])
def test_codebook_norms_past_fp32(torch, orc, D):
    rng = np.random.default_rng(D)
    cb = (rng.uniform(-1, 1, (130, D)) * 3e38).astype(np.float32)
    x = (rng.uniform(-1, 1, (500, D)) * 3e38).astype(np.float32)
    x[:100] *= np.float32(1e-30)
    x[100:200] *= np.float32(1e-37)  # (these rows are inside FP16 without a scale)
    x[200:230] = 0.0
    check(torch, orc, x, cb)
