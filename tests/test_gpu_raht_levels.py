"""The attribute transform's levels: tiles of 256 leaves, groups of 16 lists, and groups whose
lists hold more nodes than fit in LDS.  Coefficients are FP64 results rounded to FP32 and match the
step-by-step definition bit for bit, so the inverse of exact FP64 coefficients is off by their
rounding alone."""
import numpy as np
import pytest

from paper_2604_26799_amd import mgs, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    mgs.lib()
    return _t


def dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def steps(codes, depth):
    """The definition, step by step over the live nodes: (first slots, second slots, weights)."""
    code, slot = codes.astype(np.uint64), np.arange(codes.size)
    w = np.ones(codes.size)
    for s in range(3 * depth):
        above = code >> np.uint64(s + 1)
        i = np.nonzero(above[1:] == above[:-1])[0]
        if i.size:
            yield slot[i], slot[i + 1], w[i].copy(), w[i + 1].copy()
            w[i] += w[i + 1]
            keep = np.ones(code.size, bool)
            keep[i + 1] = False
            code, slot, w = code[keep], slot[keep], w[keep]


def forward(codes, attr, depth):
    val = attr.astype(np.float64)
    out, at = np.empty(attr.shape), 1
    for sa, sb, w1, w2 in steps(codes, depth):
        s1, s2, sw = np.sqrt(w1), np.sqrt(w2), np.sqrt(w1 + w2)
        a1, a2 = val[:, sa], val[:, sb]
        out[:, at:at + sa.size] = (s1 * a2 - s2 * a1) / sw
        val[:, sa] = (s1 * a1 + s2 * a2) / sw
        at += sa.size
    out[:, 0] = val[:, 0]
    return out.astype(np.float32)


def inverse(codes, coef, depth):
    every = list(steps(codes, depth))
    val, at = np.empty(coef.shape), coef.shape[1]
    val[:, 0] = coef[:, 0]
    for sa, sb, w1, w2 in reversed(every):
        at -= sa.size
        s1, s2, sw = np.sqrt(w1), np.sqrt(w2), np.sqrt(w1 + w2)
        low, high = val[:, sa], coef[:, at:at + sa.size].astype(np.float64)
        val[:, sa] = (s1 * low - s2 * high) / sw
        val[:, sb] = (s2 * low + s1 * high) / sw
    return val.astype(np.float32)


def comb(pieces):
    """Codes at depth 21 whose subtrees are zigzag combs of 41 leaves (20 single leaves on either side
    of the deepest pair), one across every multiple of 256 leaves: each tile keeps about 45 nodes."""
    def zigzag(bits):
        lo, hi, left, right = 0, 1 << bits, [], []
        for b in range(bits - 1, -1, -1):
            if b % 2:
                left.append(lo)
                lo += 1 << b
            else:
                right.append(hi - 1)
                hi -= 1 << b
        return left + [lo] + right[::-1]
    z = np.array(zigzag(40), np.uint64)
    fill = np.arange(256 - z.size, dtype=np.uint64)
    out = [np.arange(256 - z.size // 2, dtype=np.uint64)]
    for p in range(1, pieces):
        out += [z + (np.uint64(2 * p) << np.uint64(40)), fill + (np.uint64(2 * p + 1) << np.uint64(40))]
    return np.concatenate(out)


def check(torch, codes, depth, C, seed):
    rng = np.random.default_rng(seed)
    attr = rng.normal(0, 1, (C, codes.size)).astype(np.float32)
    attr[0, ::3] = 0.0
    if C > 2:
        attr[1] *= np.float32(1e-38)  # subnormal values among them
        attr[2] = np.float32(1e35) * np.sign(attr[2])
    cd = dev(torch, codes.astype(np.int64))
    want = forward(codes, attr, depth)
    got = mgs.raht(cd, dev(torch, attr), depth)
    assert np.array_equal(got.cpu().numpy(), want)
    assert np.array_equal(mgs.raht(cd, got, depth, inverse=True).cpu().numpy(), inverse(codes, want, depth))


@pytest.mark.parametrize("n,depth,C", [
    (1, 1, 1), (2, 1, 3), (8, 1, 2), (64, 2, 5),                     # a full grid: every step merges
    (255, 6, 1), (256, 6, 5), (257, 6, 6), (512, 7, 20),             # one tile, two tiles
    (1023, 8, 11), (1024, 8, 4), (1025, 8, 7), (4096, 9, 20), (4097, 9, 21),   # one group, two groups
    (32768, 5, 3),                                                   # a full grid over three levels
    (65537, 12, 11), (130001, 10, 2),                                # three levels
])
def test_levels(torch, n, depth, C):
    if n == 1 << (3 * depth):
        codes = np.arange(n, dtype=np.uint64)
    elif 2 * n > 1 << (3 * depth):
        codes = np.sort(np.random.default_rng(n).permutation(1 << (3 * depth))[:n]).astype(np.uint64)
    else:
        codes, _ = synth.voxel_codes(synth.voxels(n, depth, seed=n), depth)
    check(torch, codes, depth, C, n)


def test_definition_matches_the_oracle(orc):
    coords = synth.voxels(700, 6, seed=3)
    codes, order = synth.voxel_codes(coords, 6)
    attr = np.random.default_rng(0).normal(0, 1, (3, 700)).astype(np.float32)
    assert np.array_equal(forward(codes, attr, 6), orc.raht_forward(coords[order], attr, 6))


@pytest.mark.parametrize("pieces,C", [(3, 2), (40, 6), (300, 3)])
def test_combs(torch, pieces, C):
    """Groups with more nodes than the LDS holds, at one and at two levels."""
    check(torch, comb(pieces), 21, C, pieces)


@pytest.mark.parametrize("bad", ["equal", "falling", "outside"])
def test_bad_codes_are_flagged(torch, bad):
    codes, _ = synth.voxel_codes(synth.voxels(9000, 9, seed=1), 9)
    codes = codes.astype(np.int64)
    if bad == "equal":
        codes[5000:5600] = codes[5000]
    elif bad == "falling":
        codes[:] = codes[::-1].copy()
    else:
        codes[-700:] += 1 << 27
    for inv in (False, True):
        with pytest.raises(mgs.MgsError) as e:
            mgs.raht(dev(torch, codes), torch.ones((2, 9000), device="cuda"), 9, inverse=inv)
        assert e.value.code == mgs.ENONFINITE


@pytest.mark.parametrize("C", [1, 4, 16, 17, 32, 33, 70])
def test_channels(torch, C):
    """Chunks of four channels: one or more wavefronts per group, and groups spread over blocks."""
    codes, _ = synth.voxel_codes(synth.voxels(70_001, 11, seed=C), 11)
    check(torch, codes, 11, C, C)


def test_values_without_a_quotient(torch):
    """Infinities, NaN, zeros of both signs and the largest values pass through a merge as the
    division passes them."""
    codes, _ = synth.voxel_codes(synth.voxels(5000, 8, seed=5), 8)
    rng = np.random.default_rng(5)
    attr = rng.normal(0, 1, (6, 5000)).astype(np.float32)
    attr[0, rng.integers(0, 5000, 40)] = np.inf
    attr[1, rng.integers(0, 5000, 40)] = -np.inf
    attr[2, rng.integers(0, 5000, 40)] = np.nan
    attr[3] = rng.choice(np.array([0.0, -0.0, np.finfo(np.float32).max, -np.finfo(np.float32).max], np.float32), 5000)
    attr[4] = 0.25
    attr[5] = -0.0
    cd = dev(torch, codes.astype(np.int64))
    with np.errstate(all="ignore"):
        want = forward(codes, attr, 8)
        back = inverse(codes, want, 8)
    got = mgs.raht(cd, dev(torch, attr), 8)
    again = mgs.raht(cd, dev(torch, want), 8, inverse=True)
    for g, w in ((got.cpu().numpy(), want), (again.cpu().numpy(), back)):
        assert np.array_equal(g, w, equal_nan=True)
        finite = np.isfinite(w)
        assert np.array_equal(np.signbit(g[finite]), np.signbit(w[finite]))


def call(torch, name, codes, values, out, ld, depth, C):
    n = codes.numel()
    ws = mgs.workspace(mgs.lib().mgs_raht_ws_bytes(n, C, depth))
    code = getattr(mgs.lib(), name)(codes.data_ptr(), n, C, depth, values, ld, out, ws.data_ptr(), ws.numel(),
                                    torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return code


@pytest.mark.parametrize("n,C,pad", [(300, 1, 0), (70_001, 5, 0), (70_001, 5, 7)])
def test_in_place(torch, n, C, pad):
    """Input and output in one buffer, also with a stride and one row further on."""
    codes, _ = synth.voxel_codes(synth.voxels(n, 11, seed=n), 11)
    cd, ld = dev(torch, codes.astype(np.int64)), n + pad
    attr = np.random.default_rng(n).normal(0, 1, (C, ld)).astype(np.float32)
    want = forward(codes, attr[:, :n], 11)
    back = inverse(codes, want, 11)
    buf = dev(torch, np.concatenate([attr, np.zeros((1, ld), np.float32)]))
    step = 4 * ld if C > 1 else 0
    assert call(torch, "mgs_raht_forward", cd, buf.data_ptr(), buf.data_ptr() + step, ld, 11, C) == 0
    got = buf.cpu().numpy()[1 if step else 0:][:C]
    assert np.array_equal(got[:, :n], want)
    assert call(torch, "mgs_raht_inverse", cd, buf.data_ptr() + step, buf.data_ptr() + step, ld, 11, C) == 0
    assert np.array_equal(buf.cpu().numpy()[1 if step else 0:][:C, :n], back)


def test_largest(torch):
    """The largest size that the counts hold, and one more."""
    n = 2048 * 4096 + 1
    codes = torch.arange(n + 1, device="cuda")
    attr = torch.randn((1, n), generator=torch.Generator("cuda").manual_seed(0), device="cuda")
    got = mgs.raht(codes[:n], attr, 8)
    want = forward(np.arange(n, dtype=np.uint64), attr.cpu().numpy(), 8)
    assert np.array_equal(got.cpu().numpy(), want)
    with pytest.raises(mgs.MgsError) as e:
        mgs.raht(codes, torch.zeros((1, n + 1), device="cuda"), 8)
    assert e.value.code == mgs.EINVAL
