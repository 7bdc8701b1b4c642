"""The work that a user of this library has it do, case by case: what is timed when a kernel changes.

One case is one call (or one pair of calls that a program always makes together) of the public
Python entry points in ``paper_2604_26799_amd.mgs``:

* ``prune``: the kept sets of a scene's reserve ratios;
* ``sweep``: the loss and size tables of one scene over ratios, channels, groups and bit-widths;
* ``served``: one iteration of a compression server: the kept sets of every scene that is ready,
  then one batched sweep over all of them;
* ``codes``: the final codes at a chosen bit allocation, and their reconstruction;
* ``vq``: nearest-codeword assignment of higher-degree SH vectors;
* ``kmeans``: one mini-batch iteration of the codebook's refinement;
* ``raht``: the attribute transform, forward (encode) or inverse (decode).

Sizes are those of the repository's own workloads (small, medium and large scenes of the tests and
the benchmark, the served stream's job sizes, the benchmark's codebook and voxel grid), and odd and
ragged ones of the same ranges.  Inputs follow the seeded distributions of
``paper_2604_26799_amd.synth`` but are drawn on the GPU, which is quick.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2604_26799_amd import mgs

DEVICE = "cuda"
EVALS_EXACT_HIST = 6_000_000_000  # histograms of more codes than this take too long to count a second time


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest calls of a search over a small scene (the tests' small workload): a few
        # launches each, with the buffers and the status check that the plain call makes itself
        {"name": "prune_small", "kind": "prune", "n": 50_000, "ratios": 4, "lo": 0.3, "hi": 0.9, "held": False},
        {"name": "sweep_small", "kind": "sweep", "n": 50_000, "channels": 11, "ratios": 4, "lo": 0.3, "hi": 0.9,
         "group": 4096, "b0": 4, "b1": 8, "pad": 0, "held": False},
        # an ordinary scene (the medium workload)
        {"name": "sweep_medium", "kind": "sweep", "n": 1_000_000, "channels": 20, "ratios": 16, "lo": 0.2,
         "hi": 0.95, "group": 8192, "b0": 2, "b1": 16, "pad": 0, "held": True},
        # a full-size outdoor scene (the benchmark's large workload): kept sets, then the tables
        {"name": "prune_large", "kind": "prune", "n": 5_300_000, "ratios": 32, "lo": 0.1, "hi": 0.95, "held": True},
        {"name": "sweep_large", "kind": "sweep", "n": 5_300_000, "channels": 20, "ratios": 32, "lo": 0.1, "hi": 0.95,
         "group": 16384, "b0": 1, "b1": 16, "pad": 0, "held": True},
        # three jobs of the served stream that became ready together, ragged sizes
        {"name": "served_three", "kind": "served", "n0": 200_003, "n1": 731_111, "n2": 262_147, "channels": 20,
         "ratios": 16, "lo": 0.2, "hi": 0.95, "group": 8192, "b0": 2, "b1": 16},
        # the final codes of the large scene at the ratio its search picks, and the decoder's side
        {"name": "codes_large", "kind": "codes", "n": 5_300_000, "channels": 20, "tau": 0.1, "group": 16384},
        # every SH vector of a scene against the full codebook (the benchmark's VQ workload)
        {"name": "vq_large", "kind": "vq", "n": 3_000_000, "dim": 36, "k": 4096, "held": True},
        # the retained part of a small scene: few rows, odd vector length, a codebook that is no
        # multiple of any tile; the plain call with its own buffers and status check
        {"name": "vq_small", "kind": "vq", "n": 10_007, "dim": 45, "k": 1000, "held": False},
        # one refinement step of the codebook (the benchmark's batch)
        {"name": "kmeans_batch", "kind": "kmeans", "n": 1_000_000, "dim": 36, "k": 4096, "batch": 262_144},
        # encode: the transform of a full-size scene's attributes; decode: that of a medium one
        {"name": "raht_forward", "kind": "raht", "n": 5_300_000, "channels": 20, "depth": 14, "inverse": False},
        {"name": "raht_inverse", "kind": "raht", "n": 1_000_003, "channels": 20, "depth": 14, "inverse": True},
    ]


def _log_int(rng, lo, hi):
    """A whole number, uniform in its logarithm; odd more often than not."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.6:
        v |= 1
    return max(lo, min(hi, v))


def draw(rng):
    kind = rng.choice(["prune", "sweep", "sweep", "served", "codes", "vq", "kmeans", "raht", "raht"])
    if kind == "prune":
        return {"kind": kind, "n": _log_int(rng, 10_000, 5_300_000), "ratios": rng.randint(1, 32),
                "lo": round(rng.uniform(0.05, 0.4), 3), "hi": round(rng.uniform(0.5, 0.98), 3),
                "held": rng.random() < 0.7}
    if kind == "sweep":
        b0 = rng.randint(1, 5)
        return {"kind": kind, "n": _log_int(rng, 20_000, 3_000_000), "channels": rng.choice([11, 20]),
                "ratios": rng.randint(1, 16), "lo": round(rng.uniform(0.1, 0.4), 3),
                "hi": round(rng.uniform(0.5, 0.95), 3),
                "group": rng.choice([1024, 4096, 8192, 16384, _log_int(rng, 500, 32_768)]),
                "b0": b0, "b1": rng.randint(max(b0 + 1, 8), 16), "pad": rng.choice([0, 0, 13]),
                "held": rng.random() < 0.7}
    if kind == "served":
        b0 = rng.randint(1, 3)
        return {"kind": kind, "n0": _log_int(rng, 100_000, 1_500_000), "n1": _log_int(rng, 100_000, 1_500_000),
                "n2": _log_int(rng, 100_000, 1_500_000), "channels": 20, "ratios": rng.randint(4, 16), "lo": 0.2,
                "hi": 0.95, "group": rng.choice([4096, 8192, 16384]), "b0": b0, "b1": rng.randint(12, 16)}
    if kind == "codes":
        return {"kind": kind, "n": _log_int(rng, 50_000, 5_300_000), "channels": rng.choice([11, 20]),
                "tau": round(rng.uniform(0.08, 0.95), 3),
                "group": rng.choice([4096, 8192, 16384, _log_int(rng, 500, 32_768)])}
    if kind == "vq":
        k = _log_int(rng, 200, 8192)
        return {"kind": kind, "n": _log_int(rng, max(2 * k, 1_000), 2_000_000),
                "dim": rng.choice([9, 15, 24, 27, 36, 45, 48, 64]), "k": k, "held": rng.random() < 0.7}
    if kind == "kmeans":
        return {"kind": kind, "n": _log_int(rng, 100_000, 1_000_000), "dim": rng.choice([24, 36, 45]),
                "k": _log_int(rng, 200, 8192), "batch": _log_int(rng, 10_000, 400_000)}
    return {"kind": kind, "n": _log_int(rng, 20_000, 5_300_000), "channels": rng.choice([11, 20, 3]),
            "depth": rng.randint(12, 16), "inverse": rng.random() < 0.5}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed) * 1_000_003 + 17)
    return g


def _normal(g, shape, mean, std):
    return torch.empty(shape, dtype=torch.float32, device=DEVICE).normal_(mean, std, generator=g)


def _laplace(g, shape, scale):
    # the difference of two exponentials
    a = torch.empty(shape, dtype=torch.float32, device=DEVICE).exponential_(1.0, generator=g)
    b = torch.empty(shape, dtype=torch.float32, device=DEVICE).exponential_(1.0, generator=g)
    return a.sub_(b).mul_(scale)


def _importance(g, n):
    return _normal(g, (n,), 0.0, 2.0).exp_()


def _scene(g, n, channels, ld=None):
    """Importance [n] and attributes [channels][ld]: colour, opacity, log-scale, rotation, SH degree 1, in
    turn; a scene of other channel counts (the transform's) takes its first ones."""
    ld = ld or n
    imp = _importance(g, n)
    attr = torch.zeros((channels, ld), dtype=torch.float32, device=DEVICE)
    rows = [_normal(g, (3, n), 0.0, 0.5), _normal(g, (1, n), 0.0, 2.0), _normal(g, (3, n), -4.0, 1.0)]
    rot = _normal(g, (4, n), 0.0, 1.0)
    rows += [rot / rot.square().sum(0, keepdim=True).sqrt()]
    if channels > 11:
        rows.append(_laplace(g, (9, n), 0.05))
    attr[:, :n] = torch.cat(rows)[:channels]
    return attr, imp


def _keep_counts(case, n):
    taus = np.linspace(case["lo"], case["hi"], case["ratios"]) if case["ratios"] > 1 else np.array([case["hi"]])
    return np.floor(n * taus).astype(np.int64)


def _kept(imp, k):
    """The kept sets, concatenated: the k most important (equal ones: lower index), ascending."""
    order = torch.sort(imp, descending=True, stable=True).indices.to(torch.int32)
    return torch.cat([torch.sort(order[:int(kt)]).values for kt in k])


def _bits(case):
    return list(range(case["b0"], case["b1"] + 1))


def _voxels(g, n, depth):
    """Sorted Morton codes of n distinct voxels in eight blobs of a 2^depth grid (bit 3l + a: bit l of axis a)."""
    side = 1 << depth
    centers = torch.randint(0, side, (8, 3), generator=g, device=DEVICE)
    have = None
    while have is None or have.numel() < n:
        m = n + n // 4 + 1024
        c = centers[torch.randint(0, 8, (m,), generator=g, device=DEVICE)]
        p = (c + _normal(g, (m, 3), 0.0, side / 8).round_().to(torch.int64)) % side
        code = torch.zeros(m, dtype=torch.int64, device=DEVICE)
        for l in range(depth):
            for a in range(3):
                code |= ((p[:, a] >> l) & 1) << (3 * l + a)
        have = torch.unique(code if have is None else torch.cat([have, code]))
    pick = torch.randperm(have.numel(), generator=g, device=DEVICE)[:n]
    return torch.sort(have[pick]).values


def _merges(codes, depth):
    """The transform's merges, step by step: (first slots, second slots, their weights as doubles)."""
    n = codes.numel()
    code, slot = codes, torch.arange(n, device=codes.device)
    w = torch.ones(n, dtype=torch.float64, device=codes.device)
    for s in range(3 * depth):
        above = code >> (s + 1)
        same = above[1:] == above[:-1]
        i = same.nonzero(as_tuple=True)[0]
        if i.numel() == 0:
            continue
        yield slot[i], slot[i + 1], w[i], w[i + 1]
        keep = torch.ones(code.numel(), dtype=torch.bool, device=codes.device)
        keep[i + 1] = False
        w = w.clone()
        w[i] += w[i + 1]
        code, slot, w = code[keep], slot[keep], w[keep]


def _raht_plain(codes, attr, depth):
    """The forward transform of attr [C][N] in doubles."""
    val = attr.double().t().contiguous()
    coef = torch.empty_like(val)
    at = 1
    for sa, sb, w1, w2 in _merges(codes, depth):
        s1, s2, sw = w1.sqrt()[:, None], w2.sqrt()[:, None], (w1 + w2).sqrt()[:, None]
        a1, a2 = val[sa], val[sb]
        coef[at:at + sa.numel()] = (s1 * a2 - s2 * a1) / sw
        val[sa] = (s1 * a1 + s2 * a2) / sw
        at += sa.numel()
    coef[0] = val[0]
    return coef.t().contiguous()


def _raht_plain_inverse(codes, coef, depth):
    src = coef.double().t()
    steps = list(_merges(codes, depth))
    val = torch.empty(src.shape, dtype=torch.float64, device=src.device)
    val[0] = src[0]
    at = src.shape[0]
    for sa, sb, w1, w2 in reversed(steps):
        at -= sa.numel()
        s1, s2, sw = w1.sqrt()[:, None], w2.sqrt()[:, None], (w1 + w2).sqrt()[:, None]
        low, high = val[sa], src[at:at + sa.numel()]
        val[sa] = (s1 * low - s2 * high) / sw
        val[sb] = (s2 * low + s1 * high) / sw
    return val.t().contiguous()


def _inputs(case, seed):
    """What the case's program is given (the same for every implementation)."""
    g, kind = _gen(seed), case["kind"]
    if kind == "prune":
        return {"imp": _importance(g, case["n"]), "k": _keep_counts(case, case["n"])}
    if kind == "sweep":
        attr, imp = _scene(g, case["n"], case["channels"])
        k = _keep_counts(case, case["n"])
        s = {"attr": attr, "imp": imp, "k": k, "kept": _kept(imp, k)}
        if case["pad"]:  # rows with a stride, as a scene inside a larger allocation has them
            wide = torch.zeros((case["channels"], case["n"] + case["pad"]), dtype=torch.float32, device=DEVICE)
            wide[:, :case["n"]] = attr
            s["wide"] = wide
        return s
    if kind == "served":
        out = []
        for key in ("n0", "n1", "n2"):
            attr, imp = _scene(g, case[key], case["channels"])
            out.append({"attr": attr, "imp": imp, "k": _keep_counts(case, case[key])})
        return {"scenes": out}
    if kind == "codes":
        attr, imp = _scene(g, case["n"], case["channels"])
        k = int(case["n"] * case["tau"])
        ng = (k + case["group"] - 1) // case["group"]
        bw = torch.randint(4, 14, (case["channels"] * ng,), generator=g, device=DEVICE).to(torch.uint8)
        return {"attr": attr, "kept": _kept(imp, [k]), "bw": bw}
    if kind in ("vq", "kmeans"):
        x = _laplace(g, (case["n"], case["dim"]), 0.03)
        pick = torch.randperm(case["n"], generator=g, device=DEVICE)[:case["k"]]
        s = {"x": x, "cb": x[pick].contiguous()}
        if kind == "kmeans":
            s["batches"] = [torch.randint(0, case["n"], (case["batch"],), generator=g, device=DEVICE) for _ in range(4)]
        return s
    codes = _voxels(g, case["n"], case["depth"])
    attr, _ = _scene(g, case["n"], case["channels"])
    if case["inverse"]:
        attr = _raht_plain(codes, attr, case["depth"]).float()
    return {"codes": codes, "values": attr}


# ------------------------------------------------------------------ the calls
def _table_space(case, k):
    gm = mgs.gmax_groups(k, case["group"])
    return mgs.sweep_tables(len(k), case["channels"], gm, len(_bits(case)), DEVICE)


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    L, kind = mgs.lib(), case["kind"]
    if kind == "prune" and case["held"]:
        s["ws"] = mgs.workspace(L.mgs_prune_select_ws_bytes(case["n"], len(s["k"])))
        s["out"] = torch.empty(int(s["k"].sum()), dtype=torch.int32, device=DEVICE)
    elif kind == "sweep" and (case["held"] or case["pad"]):
        s["out"] = _table_space(case, s["k"])
        if case["pad"]:  # rows of a wider allocation go through the batched form, alone
            scene = {"attr": s["wide"], "n": case["n"], "imp": s["imp"], "kept": s["kept"], "k": s["k"], "out": s["out"]}
            s["jobs"], _ = mgs.sweep_jobs([scene], case["group"], _bits(case))
            s["scenes"] = [scene]
            s["ws"] = mgs.workspace(L.mgs_quant_sweep_multi_ws_bytes(s["jobs"], 1))
        else:
            d = mgs.sweep_desc(case["n"], case["channels"], s["k"], case["group"], _bits(case))
            s["ws"] = mgs.workspace(L.mgs_quant_sweep_ws_bytes(mgs.ct.byref(d)))
    elif kind == "served":
        for sc in s["scenes"]:
            n, k = sc["imp"].numel(), sc["k"]
            sc["ws"] = mgs.workspace(L.mgs_prune_select_ws_bytes(n, len(k)))
            sc["kept"] = torch.empty(int(k.sum()), dtype=torch.int32, device=DEVICE)
            sc["out"] = _table_space(case, k)
        jobs, _ = mgs.sweep_jobs(s["scenes"], case["group"], _bits(case))
        s["ws"] = mgs.workspace(L.mgs_quant_sweep_multi_ws_bytes(jobs, len(s["scenes"])))
    elif kind == "vq" and case["held"]:
        s["ws"] = mgs.workspace(L.mgs_vq_assign_ws_bytes(case["n"], case["dim"], case["k"]))
    elif kind == "kmeans":
        s["ws"] = mgs.workspace(L.mgs_kmeans_step_ws_bytes(case["batch"], case["dim"], case["k"]))
        s["counts"] = torch.zeros(case["k"], dtype=torch.int64, device=DEVICE)
        s["step"] = 0
    elif kind == "raht":
        s["ws"] = mgs.workspace(L.mgs_raht_ws_bytes(case["n"], case["channels"], case["depth"]))
    return s


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "prune":
        if case["held"]:
            return mgs.prune_select(state["imp"], state["k"], ws=state["ws"], out=state["out"], check=False)
        return mgs.prune_select(state["imp"], state["k"])
    if kind == "sweep":
        if case["pad"]:
            mgs.quant_sweep_multi(state["scenes"], case["group"], _bits(case), ws=state["ws"], check=False,
                                  jobs=state["jobs"])
            out = state["out"]
        elif case["held"]:
            out = mgs.quant_sweep(state["attr"], state["imp"], state["kept"], state["k"], case["group"], _bits(case),
                                  ws=state["ws"], out=state["out"], check=False)
        else:
            out = mgs.quant_sweep(state["attr"], state["imp"], state["kept"], state["k"], case["group"], _bits(case))
        return {key: out[key] for key in ("err", "bits", "gmin", "gmax")}
    if kind == "served":
        for sc in state["scenes"]:
            mgs.prune_select(sc["imp"], sc["k"], ws=sc["ws"], out=sc["kept"], check=False)
        outs = mgs.quant_sweep_multi(state["scenes"], case["group"], _bits(case), ws=state["ws"], check=False)
        return [{"kept": sc["kept"], **{key: o[key] for key in ("err", "bits", "gmin", "gmax")}}
                for sc, o in zip(state["scenes"], outs)]
    if kind == "codes":
        codes, mn, mx = mgs.quantize(state["attr"], state["kept"], case["group"], state["bw"])
        back = mgs.dequantize(codes, case["group"], state["bw"], mn, mx)
        return {"codes": codes, "gmin": mn, "gmax": mx, "values": back}
    if kind == "vq":
        if case["held"]:
            return list(mgs.vq_assign(state["x"], state["cb"], ws=state["ws"], check=False))
        return list(mgs.vq_assign(state["x"], state["cb"]))
    if kind == "kmeans":
        batch = state["batches"][state["step"] % len(state["batches"])]
        state["step"] += 1
        assign = mgs.kmeans_step(state["x"], state["cb"], state["counts"], batch, ws=state["ws"], check=False)
        return {"assign": assign, "centers": state["cb"], "counts": state["counts"]}
    return mgs.raht(state["codes"], state["values"], case["depth"], inverse=case["inverse"], ws=state["ws"],
                    check=False)


# ------------------------------------------------------------------ what a pass cannot do without
def _sweep_work(case, n):
    k = _keep_counts(case, n)
    nb, C, G = case["b1"] - case["b0"] + 1, case["channels"], case["group"]
    gm = (int(k.max()) + G - 1) // G
    # the largest kept set holds all others: its attributes and weights once, every index once, the tables once
    nbytes = int(k.max()) * 4 * (C + 1) + int(k.sum()) * 4 + len(k) * C * gm * (16 * nb + 8)
    # per kept Gaussian, channel and bit-width: quantize, clamp, round, dequantize, difference, weighted square
    return nbytes, 7 * int(k.sum()) * C * nb


def work(case):
    kind = case["kind"]
    if kind == "prune":
        return {"bytes": 4 * case["n"] + 4 * int(_keep_counts(case, case["n"]).sum()), "flops": 0}
    if kind == "sweep":
        b, f = _sweep_work(case, case["n"])
        return {"bytes": b, "flops": f}
    if kind == "served":
        b = f = 0
        for key in ("n0", "n1", "n2"):
            bi, fi = _sweep_work(case, case[key])
            b, f = b + bi + 4 * case[key], f + fi
        return {"bytes": b, "flops": f}
    if kind == "codes":
        k = int(case["n"] * case["tau"])
        return {"bytes": k * case["channels"] * (4 + 2 + 2 + 4) + 4 * k, "flops": 8 * k * case["channels"]}
    if kind == "vq":
        return {"bytes": case["n"] * (4 * case["dim"] + 12) + 4 * case["k"] * case["dim"],
                "flops": 2 * case["n"] * case["k"] * case["dim"]}
    if kind == "kmeans":
        return {"bytes": case["batch"] * (4 * case["dim"] + 12) + case["k"] * (8 * case["dim"] + 16),
                "flops": 2 * case["batch"] * case["k"] * case["dim"]}
    return {"bytes": case["n"] * (8 + 8 * case["channels"]), "flops": 8 * case["n"] * case["channels"]}


# ------------------------------------------------------------------ the same in 64 bits
def _quantizer(mn, mx, b):
    """Step and zero point: the definition is in single precision, operation by operation."""
    P = float(1 << b)
    S = (mx - mn) / P
    one = torch.ones_like(S)
    Z = torch.where(S != 0, torch.round(P - mx / torch.where(S != 0, S, one)), torch.zeros_like(S))
    return P, S, Z


def _tables_plain(attr, imp, kept, k, G, bits):
    C, dev = attr.shape[0], attr.device
    gm = (int(max(k)) + G - 1) // G
    T, nb = len(k), len(bits)
    err = torch.full((T, C, gm, nb), math.nan, dtype=torch.float64, device=dev)
    size = torch.full((T, C, gm, nb), math.nan, dtype=torch.float64, device=dev)
    lo = torch.full((T, C, gm), math.nan, dtype=torch.float64, device=dev)
    hi = torch.full((T, C, gm), math.nan, dtype=torch.float64, device=dev)
    count = int(sum(k)) * C * nb <= EVALS_EXACT_HIST
    off = 0
    for t, kt in enumerate(int(v) for v in k):
        if kt == 0:
            continue
        ids = kept[off:off + kt].long()
        off += kt
        ng = (kt + G - 1) // G
        # the last group filled up with copies of the last element, which weigh nothing
        fill = torch.arange(ng * G, device=dev).clamp_(max=kt - 1)
        w = imp[ids].double()[fill]
        w[kt:] = 0.0
        w = w.view(ng, G)
        group = torch.arange(ng, device=dev).repeat_interleave(G)[:kt]
        n_in = torch.full((ng,), float(G), dtype=torch.float64, device=dev)
        n_in[-1] = kt - (ng - 1) * G
        for c in range(C):
            x = attr[c][ids][fill].view(ng, G)
            mn, mx = x.amin(1, keepdim=True), x.amax(1, keepdim=True)
            lo[t, c, :ng], hi[t, c, :ng] = mn[:, 0].double(), mx[:, 0].double()
            x64 = x.double()
            for i, b in enumerate(bits):
                P, S, Z = _quantizer(mn, mx, b)
                q = torch.round(torch.clamp(x / torch.where(S != 0, S, torch.ones_like(S)) + Z, 0.0, P - 1.0))
                q = torch.where(S != 0, q, torch.zeros_like(q))
                back = torch.where(S != 0, (q - Z) * S, mn)
                err[t, c, :ng, i] = (w * (back.double() - x64).square()).sum(1)
                if count:
                    h = torch.bincount(group * (1 << b) + q.view(-1)[:kt].long(), minlength=ng << b).view(ng, 1 << b)
                    h = h.double()
                    size[t, c, :ng, i] = n_in * n_in.log2() - torch.special.xlogy(h, h).sum(1) / math.log(2.0)
    return {"err": err, "bits": size if count else None, "gmin": lo, "gmax": hi}


def exact(case, seed):
    kind = case["kind"]
    if kind == "prune":
        return None  # indices
    s = _inputs(case, seed)
    if kind == "sweep":
        return _tables_plain(s["attr"], s["imp"], s["kept"], s["k"], case["group"], _bits(case))
    if kind == "served":
        out = []
        for sc in s["scenes"]:
            kept = _kept(sc["imp"], sc["k"])
            out.append({"kept": None, **_tables_plain(sc["attr"], sc["imp"], kept, sc["k"], case["group"], _bits(case))})
        return out
    if kind == "codes":
        C, G, kept = case["channels"], case["group"], s["kept"].long()
        k = kept.numel()
        ng = (k + G - 1) // G
        fill = torch.arange(ng * G, device=kept.device).clamp_(max=k - 1)
        bw = s["bw"].view(C, ng)
        lo = torch.empty((C, ng), dtype=torch.float64, device=kept.device)
        hi, back = torch.empty_like(lo), torch.empty((C, k), dtype=torch.float64, device=kept.device)
        for c in range(C):
            x = s["attr"][c][kept][fill].view(ng, G)
            mn, mx = x.amin(1, keepdim=True), x.amax(1, keepdim=True)
            lo[c], hi[c] = mn[:, 0].double(), mx[:, 0].double()
            P = torch.pow(2.0, bw[c].float())[:, None]
            S = (mx - mn) / P
            safe = torch.where(S != 0, S, torch.ones_like(S))
            Z = torch.round(P - mx / safe)
            q = torch.round(torch.minimum(torch.clamp(x / safe + Z, min=0.0), P - 1.0))
            back[c] = torch.where(S != 0, (q - Z) * S, mn).double().view(-1)[:k]
        return {"codes": None, "gmin": lo, "gmax": hi, "values": back}
    if kind in ("vq", "kmeans"):
        cb = s["cb"].double()
        x = s["x"] if kind == "vq" else s["x"][s["batches"][0]]
        idx = torch.empty(x.shape[0], dtype=torch.int64, device=x.device)
        dist = torch.empty(x.shape[0], dtype=torch.float64, device=x.device)
        c2 = cb.square().sum(1)
        rows = 1 << 17
        for r in range(0, x.shape[0], rows):
            xd = x[r:r + rows].double()
            near = torch.argmin(c2 - 2.0 * (xd @ cb.t().contiguous()), 1)
            idx[r:r + rows] = near
            dist[r:r + rows] = (xd - cb[near]).square().sum(1)
        if kind == "vq":
            return [None, dist, None]
        n = torch.bincount(idx, minlength=case["k"]).double()[:, None]
        total = torch.zeros_like(cb).index_add_(0, idx, x.double())
        # the counts start at zero: a center with rows becomes their mean
        return {"assign": None, "centers": torch.where(n > 0, total / n.clamp(min=1.0), cb), "counts": None}
    plain = _raht_plain_inverse if case["inverse"] else _raht_plain
    return plain(s["codes"], s["values"], case["depth"])
