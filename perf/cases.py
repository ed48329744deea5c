"""The measured work of this framework: whole ABX scorings through the public API.

A pass of every case but one is what a program does per feature set (say one
layer of one model): build the task from the attribute table, score every cell,
collapse to the error rate.  The dataset (features resident in HBM, offsets,
attributes) is in hand before the pass.  The serving case submits a batch of
jobs to a running server and waits for all of them.

Inputs are Gaussian stand-ins for self-supervised speech features, as in
bench.py and tests/: frame = label centroid + speaker (or group) offset + noise.
``centroid`` is the spread of the label centroids: 1.0 separates labels
completely, 0.1 gives an error of several percent, as trained models do, so
that near ties meet the FP64 recheck.  Some pairs of labels are confusable
whatever that spread (as m and n are): their centroids are 0.1 apart.

The attribute table and the item lengths of a case are fixed (``table`` seeds
them), as one item file serves many feature sets; the features come from the
seed of the pass.
"""
from __future__ import annotations

import numpy as np
import torch

import paper_2505_02692_amd as fx


# ---------------------------------------------------------------- the cases

def _triphones(name, items, dim, **kw):
    """ON phone BY prev, next and speaker ("within") or ACROSS speaker ("across")."""
    c = dict(kind="triphones", items=items, dim=dim, labels=40, contexts=40, speakers=40, across=False,
             len_median=9.0, len_sigma=0.45, len_lo=5, len_hi=25, centroid=1.0, dtype="f32", mode="dtw",
             precision="bf16", distance="angular", norm="path", table=1)
    c.update(kw)
    return dict(name=name, **c) if name else c


def _groups(name, groups, dim, **kw):
    """ON label BY group: uneven groups of two labels, sizes Zipf(1.1) on [2, size_hi]."""
    c = dict(kind="groups", groups=groups, dim=dim, size_hi=2000, len_lo=1, len_hi=60, centroid=1.0,
             dtype="bf16", mode="dtw", precision="bf16", distance="angular", norm="path", table=1)
    c.update(kw)
    return dict(name=name, **c) if name else c


def _serving(name, jobs, items_lo, items_hi, **kw):
    c = dict(kind="serving", jobs=jobs, items_lo=items_lo, items_hi=items_hi, streams=4, centroid=1.0,
             dtype="bf16", mode="dtw", precision="bf16", distance="angular", norm="path", table=1)
    c.update(kw)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest call: a quick check of a feature set on a few hundred items, launches and latency
        _triphones("tiny", 400, 64, labels=20, contexts=2, speakers=1, len_median=7.0, len_sigma=0.4, len_lo=3,
                   len_hi=12, centroid=0.3),
        # within-speaker triphone ABX of one layer (the bench's size), labels well separated
        _triphones("within", 100_000, 768),
        # the same with an error rate of several percent, as trained models have: many near ties
        _triphones("within-hard", 100_000, 768, centroid=0.1),
        # across-speaker triphone ABX: many small cells per context
        _triphones("across", 40_000, 1024, speakers=100, across=True, len_sigma=0.55, len_lo=3, len_hi=40,
                   centroid=0.3),
        # few contexts, large uneven cells, features stored as bfloat16: the heaviest use
        _groups("batched", 1200, 512),
        # time-pooled scoring (one vector per item) of large cells
        _groups("batched-pooled", 400, 512, mode="pooled", centroid=0.3),
        # single-precision scoring, the form to compare with
        _triphones("within-fp32", 60_000, 768, centroid=0.3, precision="fp32"),
        # 39 cepstral features with the Euclidean distance, in the precision that the item-file
        # front end takes for it
        _triphones("cepstra-euclidean", 30_000, 39, len_lo=3, len_hi=40, len_sigma=0.55, centroid=0.3,
                   distance="euclidean", precision="fp32"),
        # the Euclidean distance in the BF16 form, raw alignment cost, a ragged feature width
        _triphones("euclidean-cost", 30_000, 250, speakers=10, centroid=0.3, distance="euclidean", norm="none"),
        # word-length items: most pairs have an item of more than 64 frames
        _groups("words", 60, 256, size_hi=60, len_lo=10, len_hi=200, centroid=0.3),
        # discrete units: one code per frame
        _triphones("units", 60_000, 1, len_lo=3, len_hi=40, len_sigma=0.55, dtype="units", distance="units",
                   precision="fp32"),
        # a server working off a burst of jobs of mixed sizes and widths
        _serving("serving", 8, 1000, 8000, centroid=0.3),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    """A case of the same ranges that has at least one cell."""
    while True:
        case = dict(_draw(rng), table=rng.randrange(1 << 30))
        if all(any(_group_cells(c, t["across"]) for _, c in _cells(t)) for t in _tables(case)):
            return case


def _draw(rng):
    dims = lambda hi: rng.choice([d for d in (64, 100, 256, 333, 512, 768, 1024) if d <= hi])
    # few cells need labels that overlap to have an error at all
    cent = lambda n, few: 0.1 if n < few else rng.choice([0.1, 0.3, 1.0])
    kind = rng.choice(["triphones", "triphones", "across", "groups", "groups", "pooled", "fp32", "euclidean", "words",
                       "units", "serving"])
    if kind == "triphones":
        n = _log_int(rng, 300, 100_000)
        return _triphones(None, n, dims(1024), speakers=_log_int(rng, 1, 60), contexts=_log_int(rng, 5, 60),
                          centroid=cent(n, 30_000), dtype=rng.choice(["f32", "bf16"]),
                          norm=rng.choice(["path", "path", "none"]), len_hi=rng.choice([25, 33, 40]))
    if kind == "across":
        n = _log_int(rng, 500, 40_000)
        return _triphones(None, n, dims(1024), speakers=rng.randint(3, 100), across=True, len_lo=3,
                          len_hi=rng.choice([25, 40]), centroid=0.1 if n < 8000 else 0.3)
    if kind == "groups":
        # labels that overlap send most pairs of a large cell to the FP64 recheck: smaller cells there
        dim, c = dims(1024), rng.choice([0.1, 1.0])
        n_lo, n_hi, size_hi = (200, 1200 * 512 // max(dim, 512), 2000) if c == 1.0 else (8, 100, 100)
        return _groups(None, _log_int(rng, n_lo, n_hi), dim, size_hi=_log_int(rng, 20, size_hi),
                       len_hi=rng.choice([17, 40, 60, 64]), centroid=c, dtype=rng.choice(["f32", "bf16"]))
    if kind == "pooled":
        n = _log_int(rng, 8, 400)
        return _groups(None, n, dims(512), size_hi=_log_int(rng, 20, 2000), mode="pooled", centroid=cent(n, 200),
                       dtype=rng.choice(["f32", "bf16"]), precision=rng.choice(["bf16", "bf16", "fp32"]),
                       distance=rng.choice(["angular", "angular", "euclidean"]))
    if kind == "fp32":
        n = _log_int(rng, 300, 60_000)
        return _triphones(None, n, dims(768), precision="fp32", centroid=cent(n, 30_000), contexts=_log_int(rng, 5, 40),
                          norm=rng.choice(["path", "none"]), dtype=rng.choice(["f32", "bf16"]))
    if kind == "euclidean":
        n = _log_int(rng, 300, 30_000)
        return _triphones(None, n, rng.choice([13, 39, 80, 250, 512]), centroid=0.1, len_lo=3, len_hi=40,
                          speakers=_log_int(rng, 1, 40), distance="euclidean", contexts=_log_int(rng, 5, 40),
                          precision=rng.choice(["bf16", "fp32"]), norm=rng.choice(["path", "none"]))
    if kind == "words":
        return _groups(None, _log_int(rng, 8, 60), dims(256), size_hi=_log_int(rng, 16, 60), len_lo=10,
                       len_hi=rng.choice([100, 151, 200]), centroid=0.03, dtype=rng.choice(["f32", "bf16"]),
                       precision=rng.choice(["bf16", "bf16", "fp32"]))
    if kind == "units":
        return _triphones(None, _log_int(rng, 300, 60_000), 1, len_lo=3, len_hi=rng.choice([25, 40, 90]),
                          contexts=_log_int(rng, 5, 40), dtype="units", distance="units", precision="fp32",
                          norm=rng.choice(["path", "none"]))
    return _serving(None, rng.randint(2, 8), 1000, _log_int(rng, 1500, 8000), centroid=0.3)


# ---------------------------------------------------------------- the inputs

def _rng(seed):
    return np.random.Generator(np.random.Philox(seed))


def _zipf(rng, s, lo, hi, n):
    p = np.arange(lo, hi + 1, dtype=np.float64) ** -s
    return lo + np.searchsorted(np.cumsum(p) / p.sum(), rng.random(n), side="right").clip(0, hi - lo)


def _lognormal_lengths(case, rng, n):
    l = np.rint(np.exp(rng.normal(np.log(case["len_median"]), case["len_sigma"], size=n)))
    return l.clip(case["len_lo"], case["len_hi"]).astype(np.int64)


def _triphone_table(case):
    rng = _rng(case["table"])
    n = case["items"]
    label = _zipf(rng, 1.0, 1, case["labels"], n) - 1
    prev = _zipf(rng, 1.0, 1, case["contexts"], n) - 1
    nxt = _zipf(rng, 1.0, 1, case["contexts"], n) - 1
    spk = rng.integers(0, case["speakers"], size=n)
    by, across = ([1, 2], [3]) if case["across"] else ([1, 2, 3], [])
    return dict(lengths=_lognormal_lengths(case, rng, n), attrs=np.stack([label, prev, nxt, spk], 1).astype(np.int32),
                by=by, across=across, levels=[[1, 2], [3]], label=label, offset=spk, n_labels=case["labels"],
                n_offsets=case["speakers"], confusable=range(6, case["labels"] - 1, 8))


def _group_table(case):
    rng = _rng(case["table"])
    sizes = _zipf(rng, 1.1, 2, case["size_hi"], case["groups"]).astype(np.int64)
    group = np.repeat(np.arange(len(sizes)), sizes)
    pos = np.arange(len(group)) - np.repeat(np.cumsum(sizes) - sizes, sizes)
    l1 = rng.integers(0, 64, size=len(sizes))
    l2 = (l1 + 1 + rng.integers(0, 63, size=len(sizes))) % 64
    # labels 2k and 2k + 1 are confusable: together in one small group of eight, apart in the others
    l2 = np.where(l2 == l1 ^ 1, (l1 + 2) % 64, l2)
    l2 = np.where((sizes <= 32) & (rng.random(len(sizes)) < 0.125), l1 ^ 1, l2)
    label = np.where(pos < np.repeat((sizes + 1) // 2, sizes), l1[group], l2[group])
    lengths = rng.integers(case["len_lo"], case["len_hi"] + 1, size=len(group)).astype(np.int64)
    return dict(lengths=lengths, attrs=np.stack([label, group], 1).astype(np.int32), by=[1], across=[], levels=[[1]],
                label=label, offset=group, n_labels=64, n_offsets=len(sizes), confusable=range(0, 64, 2))


def _job_tables(case):
    """Jobs of a serving stream: sizes log-uniform, mixed widths, within or across speakers."""
    rng = _rng(case["table"])
    out = []
    for _ in range(case["jobs"]):
        n = int(round(np.exp(rng.uniform(np.log(case["items_lo"]), np.log(case["items_hi"])))))
        dim = int(rng.choice([256, 512, 768, 1024, 1280]))
        label = _zipf(rng, 1.0, 1, 40, n) - 1
        ctx = _zipf(rng, 1.0, 1, 16, n) - 1
        spk = rng.integers(0, 20, size=n)
        by, across = ([1], [2]) if rng.random() < 0.5 else ([1, 2], [])
        out.append(dict(lengths=rng.integers(1, 61, size=n).astype(np.int64),
                        attrs=np.stack([label, ctx, spk], 1).astype(np.int32), by=by, across=across,
                        levels=[[1], [2]], label=label, offset=spk, n_labels=40, n_offsets=20, dim=dim,
                        confusable=range(6, 39, 8)))
    return out


def _tables(case):
    if case["kind"] == "serving":
        return _job_tables(case)
    t = _triphone_table(case) if case["kind"] == "triphones" else _group_table(case)
    return [dict(t, dim=case["dim"])]


def _features(case, t, seed):
    """The frames of a table on the GPU (int32 codes for discrete units)."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed * 1000003 + 17)
    n = int(t["lengths"].sum())
    lengths = torch.as_tensor(t["lengths"], device=dev)
    label = torch.repeat_interleave(torch.as_tensor(np.asarray(t["label"], np.int64), device=dev), lengths)
    if case["dtype"] == "units":  # a label's frames favour a few of 100 codes
        rnd = torch.randint(0, 100, (n,), generator=gen, device=dev)
        own = (label * 7 + torch.randint(0, 5, (n,), generator=gen, device=dev)) % 100
        keep = torch.rand((n,), generator=gen, device=dev) < 0.6
        return torch.where(keep, own, rnd).to(torch.int32)
    dim = t["dim"]
    cent = torch.randn((t["n_labels"], dim), generator=gen, device=dev) * case["centroid"]
    for k in t["confusable"]:
        cent[k + 1] = cent[k] + torch.randn((dim,), generator=gen, device=dev) * min(0.1, case["centroid"])
    off = torch.randn((t["n_offsets"], dim), generator=gen, device=dev) * 0.4
    offset = torch.repeat_interleave(torch.as_tensor(np.asarray(t["offset"], np.int64), device=dev), lengths)
    out = torch.empty((n, dim), dtype=torch.bfloat16 if case["dtype"] == "bf16" else torch.float32, device=dev)
    for f0 in range(0, n, 1 << 20):
        f1 = min(n, f0 + (1 << 20))
        x = torch.randn((f1 - f0, dim), generator=gen, device=dev).mul_(0.6)
        x += cent[label[f0:f1]]
        x += off[offset[f0:f1]]
        out[f0:f1] = x
    return out


def _offsets(lengths):
    return np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)


def prepare(case, seed):
    ctx = fx.Context(0)
    jobs = []
    for k, t in enumerate(_tables(case)):
        ds = fx.Dataset(ctx, _features(case, t, seed + 7919 * k), _offsets(t["lengths"]), t["attrs"])
        jobs.append(dict(ds=ds, by=t["by"], across=t["across"], levels=t["levels"]))
    opts = dict(mode=case["mode"], precision=case["precision"], distance=case["distance"], norm=case["norm"])
    state = dict(ctx=ctx, jobs=jobs, opts=opts)
    if case["kind"] == "serving":
        state["server"] = fx.Server(ctx, 48 << 30, case["streams"])
    return state


# ---------------------------------------------------------------- the pass

def run(state):
    if "server" in state:
        srv = state["server"]
        ids = [srv.submit(j["ds"], 0, j["by"], j["across"], **state["opts"]) for j in state["jobs"]]
        out = []
        for i in ids:
            keys, half_units, n_triplets, scores = srv.wait(i)
            out.append(dict(half_units=half_units, scores=scores))
        return out
    j = state["jobs"][0]
    res = fx.Task(j["ds"], 0, j["by"], j["across"]).score(**state["opts"])
    return dict(half_units=res.half_units, scores=res.scores, error=res.collapse(j["levels"]))


# ------------------------------------------- what a pass cannot do without

def _cells(t):
    """Cells of a table in key order, as (group items, A, B, X, exclude_self) positions: groups by BY
    values, classes by (ON, ACROSS) values."""
    attrs, by, across = t["attrs"], t["by"], t["across"]
    order = np.lexsort(tuple(attrs[:, c] for c in reversed(by + [0] + across)))
    key = attrs[order][:, by]
    cuts = np.flatnonzero((key[1:] != key[:-1]).any(1)) + 1
    for g in np.split(order, cuts):
        cls = attrs[g][:, [0] + across]
        b = np.concatenate([[0], np.flatnonzero((cls[1:] != cls[:-1]).any(1)) + 1, [len(g)]])
        classes = [(tuple(int(v) for v in cls[b[k]]), int(b[k]), int(b[k + 1])) for k in range(len(b) - 1)]
        yield g, classes


def _group_cells(classes, across):
    """The cells of one group in ascending key order (on_ax, on_b, across_ab, across_x)."""
    out = []
    if not across:
        for (ka, a0, a1) in classes:
            for (kb, b0, b1) in classes:
                if ka[0] != kb[0] and a1 - a0 > 1:
                    out.append((ka[0], kb[0], (), (), a0, a1, b0, b1, a0, a1, True))
        return out
    at = {k: (lo, hi) for k, lo, hi in classes}
    for (ka, a0, a1) in classes:
        for (kb, b0, b1) in classes:
            if kb[0] == ka[0] or kb[1:] != ka[1:]:
                continue
            for (kx, x0, x1) in classes:
                if kx[0] == ka[0] and all(p != q for p, q in zip(kx[1:], ka[1:])):
                    out.append((ka[0], kb[0], ka[1:], kx[1:], a0, a1, b0, b1, x0, x1, False))
    return sorted(out)


def work(case):
    """bytes: the features of the items that take part, read once, and 16 bytes per cell out.  flops: two
    per feature of each frame pair (pooled: item pair) of the unordered item pairs of each group that has
    cells, one DTW update of three operations per frame pair, one comparison per triple of within tasks."""
    size = {"f32": 4, "bf16": 2, "units": 4}[case["dtype"]]
    bytes_, flops = 0.0, 0.0
    for t in _tables(case):
        for g, classes in _cells(t):
            on = {}
            for k, lo, hi in classes:
                on.setdefault(k[0], []).append((k[1:], lo, hi))
            if len(on) < 2 or (t["across"] and len({k[1:] for k, _, _ in classes}) < 2):
                continue
            L = t["lengths"][g].astype(np.float64)
            bytes_ += L.sum() * t["dim"] * size
            n = L.sum() if case["mode"] == "dtw" else float(len(g))
            self_pairs = (L * L).sum() if case["mode"] == "dtw" else float(len(g))
            pairs = (n * n - self_pairs) / 2
            flops += pairs * (2.0 * t["dim"] + (3.0 if case["mode"] == "dtw" else 0.0))
            if not t["across"]:
                sizes = np.array([hi - lo for _, lo, hi in classes], np.float64)
                tri = sum(s * (s - 1) * (sizes.sum() - s) for s in sizes)
                flops += tri
                bytes_ += 16.0 * len(on) * (len(on) - 1)
    return {"bytes": float(bytes_), "flops": float(flops)}


# ------------------------------------------------- the same in 64 bits

def _dtw64(d, N, M, norm):
    """DTW of a batch of frame-distance matrices d [p, n, m] (float64) with N rows and M columns in use:
    diagonal before left before up on ties; the cost, divided by its path's length for norm "path"."""
    p, n, m = d.shape
    inf = torch.full((p, 1), float("inf"), dtype=torch.float64, device=d.device)
    out = torch.zeros(p, dtype=torch.float64, device=d.device)
    # anti-diagonals t = i + j, all rows at once
    c1 = torch.full((p, n + 1), float("inf"), dtype=torch.float64, device=d.device)  # diagonal t - 1, index i + 1
    c2 = c1.clone()
    l1 = torch.zeros((p, n + 1), dtype=torch.float64, device=d.device)
    l2 = l1.clone()
    rows = torch.arange(n, device=d.device)
    fin = (N - 1 + M - 1)
    for t in range(n + m - 1):
        j = t - rows
        ok = (j >= 0) & (j < m)
        dv = d[:, rows, j.clamp(0, m - 1)]
        diag, left, up = c2[:, :-1], c1[:, 1:], c1[:, :-1]
        ld, ll, lu = l2[:, :-1], l1[:, 1:], l1[:, :-1]
        use_d = (diag <= left) & (diag <= up)
        use_l = ~use_d & (left <= up)
        best = torch.where(use_d, diag, torch.where(use_l, left, up))
        length = torch.where(use_d, ld, torch.where(use_l, ll, lu)) + 1
        if t == 0:
            best[:, 0] = 0.0
            length[:, 0] = 1.0
        c = torch.where(ok, dv + best, float("inf"))
        hit = (fin == t).nonzero().flatten()
        if len(hit):
            i = N[hit] - 1
            out[hit] = c[hit, i] / length[hit, i] if norm == "path" else c[hit, i]
        c2, l2 = c1, l1
        c1, l1 = torch.cat([inf, c], 1), torch.cat([torch.zeros_like(inf), length], 1)
    return out


def _distances64(case, t, x, xs, ys):
    """Distances of the item pairs (xs, ys) in float64, from the widened features x."""
    dev = x.device
    lengths = torch.as_tensor(t["lengths"], device=dev)
    start = torch.as_tensor(_offsets(t["lengths"])[:-1], device=dev)
    xs, ys = torch.as_tensor(xs, device=dev), torch.as_tensor(ys, device=dev)

    def frame_dist(u, v):
        if case["distance"] == "euclidean":
            return torch.cdist(u, v, compute_mode="donot_use_mm_for_euclid_dist")
        u = u / u.norm(dim=-1, keepdim=True).clamp_min(1e-300)
        v = v / v.norm(dim=-1, keepdim=True).clamp_min(1e-300)
        return torch.acos(torch.matmul(u, v.transpose(-1, -2).contiguous()).clamp(-1, 1)) / np.pi

    out = torch.zeros(len(xs), dtype=torch.float64, device=dev)
    if case["mode"] == "pooled":
        seg = torch.repeat_interleave(torch.arange(len(lengths), device=dev), lengths)
        mean = torch.zeros((len(lengths), x.shape[1]), dtype=torch.float64, device=dev)
        mean.index_add_(0, seg, x.double())
        mean /= lengths[:, None]
        for k in range(0, len(xs), 1 << 16):
            u, v = mean[xs[k:k + (1 << 16)]], mean[ys[k:k + (1 << 16)]]
            out[k:k + (1 << 16)] = frame_dist(u[:, None], v[:, None])[:, 0, 0]
        return out
    order = torch.argsort(lengths[xs] * 4096 + lengths[ys])
    k = 0
    while k < len(order):
        step = 4096
        while True:
            o = order[k:k + step]
            N, M = lengths[xs[o]], lengths[ys[o]]
            n, m = int(N.max()), int(M.max())
            if step <= 64 or len(o) * (n + m) * t["dim"] + len(o) * n * m * 4 <= 1 << 27:
                break
            step //= 2
        fi = start[xs[o]][:, None] + torch.minimum(torch.arange(n, device=dev)[None], N[:, None] - 1)
        fj = start[ys[o]][:, None] + torch.minimum(torch.arange(m, device=dev)[None], M[:, None] - 1)
        if case["dtype"] == "units":
            d = (x[fi][:, :, None] != x[fj][:, None, :]).double()
        else:
            d = frame_dist(x[fi].double(), x[fj].double())
        out[o] = _dtw64(d, N, M, case["norm"])
        k += step
    return out


def _exact_table(case, t, seed):
    groups = [(g, _group_cells(c, t["across"])) for g, c in _cells(t)]
    groups = [(g, c) for g, c in groups if c]
    cells = sum(len(c) for _, c in groups)
    pairs = sum(len(g) ** 2 for g, _ in groups)
    cost = sum(float(t["lengths"][g].sum()) ** 2 for g, _ in groups)
    if cells > 60_000 or pairs > 400_000 or cost * (t["dim"] + 60) > 6e10:
        return None
    x = _features(case, t, seed)
    need = [np.unique(np.concatenate([(np.r_[c[8]:c[9]][:, None] * len(g) + np.r_[c[4]:c[5], c[6]:c[7]][None]).ravel()
                                      for c in cs])) for g, cs in groups]
    xs = np.concatenate([g[q // len(g)] for (g, _), q in zip(groups, need)])
    ys = np.concatenate([g[q % len(g)] for (g, _), q in zip(groups, need)])
    dist = _distances64(case, t, x, xs, ys).cpu().numpy()
    half, total, keys, at = [], [], [], 0
    for (g, cs), q in zip(groups, need):
        mat = np.zeros(len(g) ** 2)
        mat[q] = dist[at:at + len(q)]
        at += len(q)
        mat = mat.reshape(len(g), len(g))
        byv = [int(v) for v in t["attrs"][g[0]][t["by"]]]
        for (oa, ob, ka, kx, a0, a1, b0, b1, x0, x1, self_) in cs:
            da, db = mat[x0:x1, a0:a1, None], mat[x0:x1, None, b0:b1]
            w = 2 * (da < db).astype(np.int64) + (da == db)
            if self_:
                w[np.arange(x1 - x0), np.arange(x1 - x0)] = 0
            half.append(int(w.sum()))
            total.append((a1 - a0) * (b1 - b0) * ((x1 - x0) - (1 if self_ else 0)))
            keys.append([oa, ob] + byv + list(ka) + list(kx))
    half, total = np.array(half, np.int64), np.array(total, np.int64)
    scores = half / (2.0 * total)
    # collapse: level by level, unweighted means over the rows that share the remaining columns
    attr = [0, 0] + t["by"] + t["across"] + t["across"]
    rows, vals = np.array(keys), scores
    for level in t["levels"]:
        keep = [k for k, a in enumerate(attr) if a not in level]
        attr = [attr[k] for k in keep]
        rows, inv = np.unique(rows[:, keep], axis=0, return_inverse=True)
        inv = inv.ravel()
        vals = np.bincount(inv, vals) / np.bincount(inv)
    return dict(half_units=half, scores=scores, error=1.0 - float(vals.mean()))


def exact(case, seed):
    if case["kind"] == "serving":
        outs = [_exact_table(case, t, seed + 7919 * k) for k, t in enumerate(_tables(case))]
        return [dict(half_units=o["half_units"], scores=o["scores"]) if o else dict(half_units=None, scores=None)
                for o in outs]
    return _exact_table(case, _tables(case)[0], seed)
