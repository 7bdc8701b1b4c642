"""Edges of the sweep kernel's variants: workgroups of half the width that keep the wide
shape's sums, repeated elements past a ragged end, NaN pairs, rows beyond 32-bit offsets.
Tolerances as in test_gpu_parity.py (loss 4e-6 relative, sizes 1e-9)."""
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


def sweep(torch, attr, imp, kept, k, G, bits, check=True):
    out = mgs.quant_sweep(dev(torch, attr), dev(torch, imp), dev(torch, kept.astype(np.int32)), k, G, bits,
                          check=check)
    torch.cuda.synchronize()
    return {key: out[key].cpu().numpy() for key in ("err", "bits", "gmin", "gmax")}


def assert_tables(got, want):
    ok = ~np.isnan(want["err"])
    assert np.array_equal(np.isnan(got["err"]), ~ok)
    np.testing.assert_allclose(got["err"][ok], want["err"][ok], rtol=4e-6, atol=1e-300)
    np.testing.assert_allclose(got["bits"][ok], want["bits"][ok], rtol=1e-9, atol=1e-6)
    g = ~np.isnan(want["gmin"])
    assert np.array_equal(got["gmin"][g], want["gmin"][g]) and np.array_equal(got["gmax"][g], want["gmax"][g])


@pytest.mark.parametrize("G,wide,half", [
    (2049, (512, 8), (256, 16)),    # the smallest and largest groups of each half-width shape,
    (4096, (512, 8), (256, 16)),    # and one whose last elements are spread over few lanes
    (4097, (1024, 8), (512, 16)),
    (7777, (1024, 8), (512, 16)),
    (8192, (1024, 8), (512, 16)),
])
@pytest.mark.parametrize("scale", [1.0, 1e-38])  # (tiny weights: the FP64 recomputation of the sums)
def test_half_width_shapes(torch, orc, G, wide, half, scale):
    attr, imp = synth.scene(30011, 20, seed=G)
    attr = np.ascontiguousarray(attr[:5])
    attr[4] = attr[4] * np.float32(1e-30)  # literal division at the largest bit-widths
    imp = (imp / imp.max() * np.float32(scale)).astype(np.float32)
    k = np.array([30011, 2 * G + 1, G - 1, 1], np.int64)
    bits = [1, 4, 8, 12, 15, 16]
    kept = orc.prune_select(imp, k)
    want = orc.quant_sweep(attr, imp, kept, k, G, bits)
    got = []
    try:
        for nt, ept in (wide, half):
            for persist in (0, 1):
                mgs.sweep_set_shape(G, len(bits), max(bits), nt, ept, 98304, 0, persist)
                got.append(sweep(torch, attr, imp, kept, k, G, bits))
    finally:
        mgs.sweep_set_shape(G, len(bits), max(bits), 0, 0, 0, 0)
    for one in got:
        assert_tables(one, want)
        for key in ("err", "gmin", "gmax"):  # the half-width shape adds the same terms in the same order
            assert np.array_equal(one[key], got[0][key], equal_nan=True), key


@pytest.mark.parametrize("G", [1, 2, 255, 1025, 5000, 16384, 20000])  # 20000: the chunked kernel
def test_nan_and_ragged_ends(torch, orc, G):
    """One NaN in the last, ragged group (in turn in its last and its first element) makes that
    group NaN and leaves every other one, and its bounds are those of its other values."""
    n = 2 * G + max(1, G // 2)
    attr, imp = synth.scene(n, 11, seed=G)
    attr = np.ascontiguousarray(attr[:3])
    k, bits = np.array([n], np.int64), [2, 7, 13]
    kept = np.arange(n, dtype=np.int32)
    want = orc.quant_sweep(attr, imp, kept, k, G, bits)
    for at in (n - 1, 2 * G):
        bad = attr.copy()
        bad[1, at] = np.nan
        got = sweep(torch, bad, imp, kept, k, G, bits, check=False)
        assert np.isnan(got["err"][0, 1, -1]).all() and np.isnan(got["bits"][0, 1, -1]).all()
        rest = np.delete(bad[1, 2 * G:], at - 2 * G)
        if rest.size:
            assert got["gmin"][0, 1, -1] == rest.min() and got["gmax"][0, 1, -1] == rest.max()
        for key in ("err", "bits", "gmin", "gmax"):
            got[key][0, 1, -1] = want[key][0, 1, -1]
        assert_tables(got, want)


def test_rows_beyond_32_bit_offsets(torch, orc):
    """Rows with a stride above 2^30 floats are gathered by index, others by 32-bit byte offset."""
    n, G, bits = 5000, 2048, [3, 9]
    attr, imp = synth.scene(n, 11, seed=3)
    k = np.array([n, 3333], np.int64)
    kept = orc.prune_select(imp, k)
    want = orc.quant_sweep(attr[:1], imp, kept, k, G, bits)
    for ld in (1 << 30, (1 << 30) + 64):
        wide = torch.zeros((1, ld), dtype=torch.float32, device="cuda")
        wide[0, :n] = dev(torch, attr[0])
        scene = {"attr": wide, "n": n, "imp": dev(torch, imp), "kept": dev(torch, kept.astype(np.int32)), "k": k}
        (out,) = mgs.quant_sweep_multi([scene], G, bits)
        assert_tables({key: out[key].cpu().numpy() for key in ("err", "bits", "gmin", "gmax")}, want)
        del wide, scene


@pytest.mark.parametrize("G,n,C,T,wide", [
    (200, 3000, 3, 2, (256, 8)), (256, 60000, 11, 4, (256, 8)), (257, 60000, 5, 4, (256, 8)),
    (513, 60000, 5, 4, (256, 8)), (1024, 60000, 11, 6, (256, 8)), (1025, 60000, 11, 2, (256, 8)),
    (2048, 60000, 3, 1, (256, 8)), (2049, 60000, 20, 6, (512, 8)), (4096, 60000, 11, 2, (512, 8)),
    (4097, 120000, 20, 6, (1024, 8)), (8192, 9000, 2, 1, (1024, 8)), (8192, 300000, 20, 4, (1024, 8)),
    (8193, 60000, 20, 3, (1024, 16)), (16384, 20000, 1, 1, (1024, 16)), (16385, 60000, 11, 3, (512, 16)),
])
def test_default_shape_keeps_the_tables(torch, G, n, C, T, wide):
    """The default launch shape follows the launch's size; its losses and bounds are bit for bit those
    of the wide shape in plain one-workgroup-per-tile form, its sizes the same to FP64 rounding."""
    attr, imp = synth.scene(n, 20, seed=n + G)
    attr = np.ascontiguousarray(attr[:C])
    k = np.linspace(n // 3, n, T).astype(np.int64)
    order = np.argsort(-imp, kind="stable")
    kept = np.concatenate([np.sort(order[:kt]) for kt in k]).astype(np.int32)
    bits = [2, 6, 11, 16]
    got = sweep(torch, attr, imp, kept, k, G, bits)
    try:
        mgs.sweep_set_shape(G, len(bits), max(bits), *wide, 0, 0, 0)
        want = sweep(torch, attr, imp, kept, k, G, bits)
    finally:
        mgs.sweep_set_shape(G, len(bits), max(bits), 0, 0, 0, 0)
    for key in ("err", "gmin", "gmax"):
        assert np.array_equal(got[key], want[key], equal_nan=True), key
    ok = ~np.isnan(want["bits"])
    np.testing.assert_allclose(got["bits"][ok], want["bits"][ok], rtol=1e-12, atol=1e-9)
    # and bit for bit, sizes too, those of the same scene in a batch with a larger one
    big = 400_000
    attr2, imp2 = synth.scene(big, 20, seed=1)
    k2 = np.array([big, big // 2], np.int64)
    scenes = [{"attr": dev(torch, attr), "imp": dev(torch, imp), "kept": dev(torch, kept), "k": k},
              {"attr": dev(torch, attr2), "imp": dev(torch, imp2), "k": k2,
               "kept": dev(torch, np.concatenate([np.arange(v) for v in k2]).astype(np.int32))}]
    both = mgs.quant_sweep_multi(scenes, G, bits)[0]
    for key in ("err", "bits", "gmin", "gmax"):
        assert np.array_equal(both[key].cpu().numpy(), got[key], equal_nan=True), key


@pytest.mark.parametrize("G,n,C,bits", [
    (64, 200_000, 3, [8]), (64, 200_000, 3, list(range(1, 17))),    # whole groups: plain, persistent
    (1000, 300_000, 20, [1, 2]), (1000, 300_000, 20, [2, 9, 16]),   # runs of channels: plain, persistent
])
def test_short_tiles(torch, orc, G, n, C, bits):
    """Launches of many tiles on both sides of the line between plain and persistent grids: the oracle's
    tables, and those of one-channel tiles in a plain grid, bit for bit."""
    attr, imp = synth.scene(n, 20, seed=G)
    attr = np.ascontiguousarray(attr[:C])
    k = np.array([n, n // 2 + 1], np.int64)
    kept = orc.prune_select(imp, k)
    got = sweep(torch, attr, imp, kept, k, G, bits)
    nt, ept, cap = 256, (1 if G <= 256 else 4), 40960
    try:
        mgs.sweep_set_shape(G, len(bits), max(bits), nt, ept, cap, 1, 0)
        want = sweep(torch, attr, imp, kept, k, G, bits)
    finally:
        mgs.sweep_set_shape(G, len(bits), max(bits), 0, 0, 0, 0)
    for key in ("err", "bits", "gmin", "gmax"):
        assert np.array_equal(got[key], want[key], equal_nan=True), key
    few = slice(0, 2)  # (the oracle takes its time over two channels)
    ref = orc.quant_sweep(np.ascontiguousarray(attr[few]), imp, kept, k, G, bits)
    assert_tables({key: got[key][:, few] for key in got}, ref)


@pytest.mark.parametrize("G,shapes", [
    (300, [(256, 2)]), (2048, [(256, 8)]), (3000, [(512, 8), (256, 16)]), (4096, [(512, 8), (256, 16)]),
    (5000, [(1024, 8), (512, 16)]), (8192, [(1024, 8), (512, 16)]),
])
def test_sizes_do_not_depend_on_the_plan(torch, orc, G, shapes):
    """A small launch and a large one of the same groups differ in the workgroup's width and in the LDS
    that its histograms are planned in: the tables are the same bit for bit, sizes too, and so are
    those of a call that also returns the histograms."""
    n = 3 * G + G // 3
    attr, imp = synth.scene(n, 11, seed=G)
    attr = np.ascontiguousarray(attr[:6])
    attr[5] = np.round(attr[5] * 2)  # few values: bins of many elements
    k, bits = np.array([n, 2 * G], np.int64), [1, 3, 4, 5, 7, 8, 9, 12, 14, 15, 16]
    kept = orc.prune_select(imp, k)
    want = orc.quant_sweep(attr, imp, kept, k, G, bits)
    first = sweep(torch, attr, imp, kept, k, G, bits)  # (the default of a small launch)
    assert_tables(first, want)
    d = [dev(torch, a) for a in (attr, imp, kept.astype(np.int32))]
    try:
        for nt, ept in shapes:
            for cap in (0, 81920, 40960):
                mgs.sweep_set_shape(G, len(bits), max(bits), nt, ept, cap, 1, 0)
                for hist in (False, True):
                    got = mgs.quant_sweep(*d, k, G, bits, want_hist=hist)
                    for key in ("err", "bits", "gmin", "gmax"):
                        assert np.array_equal(got[key].cpu().numpy(), first[key], equal_nan=True), (nt, cap, hist, key)
    finally:
        mgs.sweep_set_shape(G, len(bits), max(bits), 0, 0, 0, 0)
