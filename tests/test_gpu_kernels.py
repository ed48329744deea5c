"""Kernels against the FP64 oracle at the sizes where they can go wrong: tile
edges, remainders, the ends of a dispatch rule's range."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from test_gpu_parity import all_oracle_pairs, gpu_score

pytestmark = pytest.mark.gpu


# Every pair goes to the FP64 recheck (margin above any distance gap).  The
# classes by the longer item: 16 frames (four pairs a wave from about 12,000
# pairs on, else one), 32 (a wave per pair from 2,048 pairs on, else a block),
# 64 (a block per pair), longer (chunks of 64 rows).  Dims: whole chunks of 16
# features, remainders, rows off a 16-byte boundary.
RECHECK = {
    "16-many": dict(n_groups=10, size_lo=60, size_hi=60, len_lo=1, len_hi=16, dim=20, dtype=torch.float32),
    "16-few": dict(n_groups=5, size_lo=9, size_hi=9, len_lo=14, len_hi=16, dim=16, dtype=torch.float32),
    "32-many": dict(n_groups=6, size_lo=40, size_hi=40, len_lo=10, len_hi=32, dim=5, dtype=torch.bfloat16),
    "32-few": dict(n_groups=4, size_lo=8, size_hi=8, len_lo=15, len_hi=33, dim=33, dtype=torch.float32),
    "64": dict(n_groups=4, size_lo=8, size_hi=8, len_lo=31, len_hi=64, dim=50, dtype=torch.bfloat16),
    "long": dict(n_groups=4, size_lo=6, size_hi=6, len_lo=60, len_hi=131, dim=17, dtype=torch.float32),
}


@pytest.mark.parametrize("distance,norm", [("angular", "path"), ("angular", "none"), ("euclidean", "path")])
@pytest.mark.parametrize("case", list(RECHECK) + ["ties"])
def test_fp64_recheck_classes(case, distance, norm):
    """Every FP64 pair value, in both orientations, within 1e-12 of the
    oracle's (relative where it exceeds 1: raw costs), and every cell exact."""
    if case == "ties":
        # frames of two codes at right angles: distances 0 and 1/2 (or sqrt 2), so
        # paths of equal cost and different length abound and the predecessor
        # order of each orientation decides
        w = workloads.batched_c4(n_groups=4, size_lo=10, size_hi=10, len_lo=1, len_hi=40, dim=2,
                                 dtype=torch.float32, seed=5)
        code = torch.from_numpy(np.random.default_rng(5).integers(0, 2, w.n_frames))
        w.features = torch.nn.functional.one_hot(code, 2).float()
    else:
        w = workloads.batched_c4(centroid_std=0.1, seed=81, **RECHECK[case])
    print(f"[case] recheck {case} {distance} {norm} items={w.n_items} dim={w.dim}", flush=True)
    t, res = gpu_score(w, norm=norm, distance=distance, margin=1e4, keep_pairs=True)
    orc = oracle.score(w.features_f32_host(), w.offsets, w.attrs, w.on, w.by, w.across, "dtw", norm,
                       distance=distance)
    xs, ys, want = all_oracle_pairs(orc)
    _, fl, f64 = res.pairs(xs, ys)
    assert ((fl & 2) != 0).all()
    assert (np.abs(f64 - want) <= 1e-12 * np.maximum(want, 1.0)).all()
    assert np.array_equal(res.half_units, orc.half_units)


# Pooled mode, every pair marked.  Groups of n items at dim D with n >= D take the
# tiles of the pair matrices (the FP64 means fit the list's memory), with n < D the
# list; 16 x 16 tiles, 64 x 128 blocks of them, a remainder of features.
@pytest.mark.parametrize("distance", ["angular", "euclidean"])
@pytest.mark.parametrize("n,dim,dtype", [(15, 8, torch.float32), (17, 16, torch.bfloat16), (70, 33, torch.float32),
                                         (140, 50, torch.float32), (20, 64, torch.bfloat16),
                                         (9, 130, torch.float32)])
def test_fp64_recheck_pooled(n, dim, dtype, distance):
    w = workloads.batched_c4(n_groups=3, size_lo=n, size_hi=n, len_lo=1, len_hi=9, dim=dim, dtype=dtype,
                             centroid_std=0.1, seed=n)
    # the second half of each label's items repeats the first: exact ties
    feats, off = w.features.clone(), w.offsets
    for k in range(0, w.n_items - 1, 5):
        m = min(off[k + 1] - off[k], off[k + 2] - off[k + 1])
        if off[k + 1] - off[k] == off[k + 2] - off[k + 1]:
            feats[off[k + 1]:off[k + 1] + m] = feats[off[k]:off[k] + m]
    w.features = feats
    print(f"[case] pooled recheck n={n} dim={dim} {distance}", flush=True)
    t, res = gpu_score(w, mode="pooled", distance=distance, margin=1e4, keep_pairs=True)
    orc = oracle.score(w.features_f32_host(), w.offsets, w.attrs, w.on, w.by, w.across, "pooled", "path",
                       distance=distance)
    xs, ys, want = all_oracle_pairs(orc)
    _, fl, f64 = res.pairs(xs, ys)
    assert ((fl & 2) != 0).all()
    assert (np.abs(f64 - want) <= 1e-12 * np.maximum(want, 1.0)).all()
    assert np.array_equal(res.half_units, orc.half_units)


# Rows of large cells, sorted in LDS: |B| at the two capacities and past the
# larger one (counted by brute force), values that crowd one bucket (repeated
# items), a margin that sends some rows or all to the FP64 recount.
@pytest.mark.parametrize("margin", [-1.0, 0.02, 1e4])
@pytest.mark.parametrize("nb,na,repeat", [(255, 64, 1), (1024, 20, 1), (1025, 20, 40), (600, 40, 60), (4096, 12, 1),
                                          (4097, 12, 1)])
def test_sorted_rows(nb, na, repeat, margin):
    rng = np.random.default_rng(nb)
    n = na + nb
    label = np.r_[np.zeros(na, np.int32), np.ones(nb, np.int32)]
    x = rng.standard_normal((n, 3)).astype(np.float32)
    x[:na] += 0.5
    if repeat > 1:  # runs of `repeat` equal items
        x = x[np.arange(n) // repeat * repeat]
    attrs = np.stack([label, np.zeros(n, np.int32)], 1)
    w = workloads.Workload("sorted", torch.from_numpy(x), np.arange(n + 1, dtype=np.int64), attrs, ["l", "g"], 0, [1],
                           [])
    print(f"[case] sorted rows nb={nb} na={na} repeat={repeat} margin={margin}", flush=True)
    t, res = gpu_score(w, mode="pooled", margin=margin)
    # the definition in FP64, row by row (one-frame items; only rows of class 0 and 1 as X)
    u = x.astype(np.float64)
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    uniq, inv = np.unique(x, axis=0, return_inverse=True)   # equal items share one distance
    v = uniq.astype(np.float64)
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    d = np.arccos(np.clip(v @ v.T, -1, 1))
    np.fill_diagonal(d, 0.0)
    d = d[np.ix_(inv.ravel(), inv.ravel())]
    want = []
    for A, B in ((np.arange(na), np.arange(na, n)), (np.arange(na, n), np.arange(na))):
        s = 0
        for i in A:
            a = np.sort(d[i, A[A != i]])
            b = np.sort(d[i, B])
            s += int((2 * len(b) - np.searchsorted(b, a, "left") - np.searchsorted(b, a, "right")).sum())
        want.append(s)
    assert res.half_units.tolist() == want


# The plain FP32 form's fused kernel against its strip form (which a task takes
# once any item has more than 64 frames): every pair value bit for bit.  Lengths
# to the row block's 64 frames, groups over several column blocks, dims off and on
# the staging chunk, frames of two codes (ties between paths of different length),
# infinities and NaN in the features (Euclidean: the order of comparisons shows).
@pytest.mark.parametrize("norm", ["path", "none"])
@pytest.mark.parametrize("case,distance", [("ragged", "angular"), ("ragged", "euclidean"), ("one-frame", "angular"),
                                           ("codes", "angular"), ("codes", "euclidean"), ("odd", "euclidean"),
                                           ("units", "units")])
def test_plain_fused_equals_strips(case, distance, norm):
    import paper_2505_02692_amd as fx
    from test_gpu_parity import ctx
    len_hi = {"one-frame": 1, "units": 40}.get(case, 64)
    w = workloads.batched_c4(n_groups=9, size_lo=15, size_hi=40, len_lo=1, len_hi=len_hi, dim=70 if case == "ragged" else 8,
                             centroid_std=0.3, dtype=torch.float32, seed=17)
    rng = np.random.default_rng(3)
    feats = w.features.clone()
    if case == "codes":
        feats = torch.nn.functional.one_hot(torch.from_numpy(rng.integers(0, 2, w.n_frames)), 8).float()
    if case == "odd":
        for v in (np.nan, np.inf, -np.inf, 3e38):
            for f in rng.integers(0, w.n_frames, 12):
                feats[f, int(rng.integers(0, 8))] = v
    if case == "units":
        feats = torch.from_numpy(rng.integers(0, 3, w.n_frames).astype(np.int32))
    # the same items and a group of their own for two long ones
    extra = torch.ones((66 + 3, 8 if case != "ragged" else 70)) if case != "units" else torch.ones(69, dtype=torch.int32)
    attrs = np.concatenate([w.attrs, [[0, 9999], [0, 9999], [1, 9999]]]).astype(np.int32)
    off = np.concatenate([w.offsets, w.offsets[-1] + np.array([1, 67, 69])]).astype(np.int64)
    kw = dict(precision="fp32", distance=distance, norm=norm, keep_pairs=True)
    print(f"[case] plain fused {case} {distance} {norm}", flush=True)
    short = fx.Task(fx.Dataset(ctx(), feats.cuda().contiguous(), w.offsets, w.attrs), 0, [1]).score(**kw)
    both = fx.Task(fx.Dataset(ctx(), torch.cat([feats, extra.to(feats.dtype)]).cuda().contiguous(), off, attrs), 0,
                   [1]).score(**kw)
    xs, ys = [], []
    for g in np.unique(w.attrs[:, 1]):
        items = np.flatnonzero(w.attrs[:, 1] == g)
        if len(np.unique(w.attrs[items, 0])) == 2 and len(items) > 2:
            i, j = np.meshgrid(items, items, indexing="ij")
            xs.append(i.ravel())
            ys.append(j.ravel())
    xs, ys = np.concatenate(xs), np.concatenate(ys)
    a, b = short.pairs(xs, ys)[0], both.pairs(xs, ys)[0]
    assert len(xs) > 1000
    assert np.array_equal(a, b, equal_nan=True)
    if case == "odd":
        assert np.isnan(a).any() and np.isinf(a).any()
    else:
        assert np.isfinite(a).all()


# The BF16 form's work units where their edges meet: blocks of one-frame items
# (64 and 128 items), items that fill a row block, items that leave a block's last
# frame over, pairs that end in the first or last of four steps.  Frames of 70
# normal features: the BF16 cosine is off by at most 2^-8, an angle by that over
# its sine (> 0.8), so a distance by less than 0.002 and a path's cost by that a
# step; and a value depends on neither the column block's width nor the grid.
@pytest.mark.parametrize("norm", ["path", "none"])
@pytest.mark.parametrize("lens", [[1], [64], [63, 1], [1, 62, 2, 3], [31, 33, 32], [5, 6, 7, 8, 9]],
                         ids=lambda v: "-".join(map(str, v)))
def test_fused_unit_edges(lens, norm):
    import paper_2505_02692_amd as fx
    from test_gpu_parity import ctx
    rng = np.random.default_rng(11)
    n_of = [3, 65, 150] if lens == [1] else [3, 29, 41]
    length = np.concatenate([np.resize(lens, n) for n in n_of])
    off = np.concatenate([[0], np.cumsum(length)]).astype(np.int64)
    attrs = np.concatenate([np.stack([rng.permutation(np.arange(n) % 2), np.full(n, g)], 1)
                            for g, n in enumerate(n_of)]).astype(np.int32)
    feats = torch.from_numpy(rng.standard_normal((int(off[-1]), 70), dtype=np.float32))
    print(f"[case] unit edges {lens} {norm}", flush=True)
    ds = fx.Dataset(ctx(), feats.cuda().contiguous(), off, attrs)
    res = [fx.Task(ds, 0, [1]).score(norm=norm, keep_pairs=True, fused_cols=c, fused_blocks_per_cu=b)
           for c, b in ((128, 4), (256, 2), (128, 1))]
    orc = oracle.score(feats.numpy(), off, attrs, 0, [1], [], "dtw", norm)
    xs, ys, want = all_oracle_pairs(orc)
    got = [r.pairs(xs, ys) for r in res]
    for r, (a, fl, _) in zip(res, got):
        assert np.array_equal(r.half_units, orc.half_units)
        assert np.array_equal(a, got[0][0]) and np.array_equal(fl & 1, got[0][1] & 1)
    sure = (got[0][1] & 1) == 0
    steps = length[xs] + length[ys] - 1
    tol = 0.002 * (steps if norm == "none" else 1)
    assert (np.abs(got[0][0] - want) <= tol)[sure].all()


# Tasks whose items are taken in the packing order (an item meets 12,000 frames or
# more of its group; group sizes from one row block to several column blocks, one
# group of two items) against the same scores in task order: the streaming kernel
# for the BF16 form, FP64 oracle for the counts, and the score from the scratch
# memory, where the order lies in the recheck list.  Pair values: as above.
@pytest.mark.parametrize("kind", ["bf16", "euclidean", "fp32", "units"])
@pytest.mark.parametrize("norm", ["path", "none"])
def test_packing_order(kind, norm):
    import paper_2505_02692_amd as fx
    from test_gpu_parity import ctx
    rng = np.random.default_rng(23)
    n_of = [2, 9, 40, 77, 150]
    length = rng.integers(1, 65, sum(n_of))
    off = np.concatenate([[0], np.cumsum(length)]).astype(np.int64)
    attrs = np.concatenate([np.stack([rng.permutation(np.arange(n) % 3), np.full(n, g)], 1)
                            for g, n in enumerate(n_of)]).astype(np.int32)
    meet = sum(length[attrs[:, 1] == g].sum() ** 2 for g in range(1, len(n_of))) / sum(n_of[1:])
    assert meet > 12000
    if kind == "units":
        feats = torch.from_numpy(rng.integers(0, 5, int(off[-1])).astype(np.int32))
        ref = torch.nn.functional.one_hot(feats.long(), 5).numpy().astype(np.float32)
    else:
        feats = torch.from_numpy(rng.standard_normal((int(off[-1]), 40), dtype=np.float32))
        ref = feats.numpy()
    opts = dict(norm=norm, precision="fp32" if kind == "fp32" else "bf16",
                distance={"bf16": "angular", "fp32": "angular"}.get(kind, kind))
    print(f"[case] packing order {kind} {norm}", flush=True)
    ds = fx.Dataset(ctx(), feats.cuda().contiguous(), off, attrs)
    t = fx.Task(ds, 0, [1])
    res = t.score(keep_pairs=True, **opts)
    scratch, _ = fx.fabx_score_noalloc(t.h, fx.make_opts(**opts), len(t))
    assert np.array_equal(scratch, res.half_units)
    if kind == "bf16":
        assert np.array_equal(t.score(fused_cols=512, **opts).half_units, res.half_units)
        assert np.array_equal(fx.fabx_score_noalloc(t.h, fx.make_opts(fused_cols=512, **opts), len(t))[0],
                              res.half_units)
        assert np.array_equal(t.score(fused_cols=256, **opts).half_units, res.half_units)
        sub = fx.Task(ds, 0, [1], [], fx.Subsampler(seed=3, max_a=30, max_b=30, max_x=30))
        assert np.array_equal(sub.score(fused_cols=512, **opts).half_units, sub.score(**opts).half_units)
    if kind in ("bf16", "euclidean"):
        orc = oracle.score(ref, off, attrs, 0, [1], [], "dtw", norm, distance=opts["distance"])
        assert np.array_equal(res.half_units, orc.half_units)
        if kind == "bf16":
            xs, ys, want = all_oracle_pairs(orc)
            got, fl, _ = res.pairs(xs, ys)
            tol = 0.002 * (length[xs] + length[ys] - 1 if norm == "none" else 1)
            assert (np.abs(got - want) <= tol)[(fl & 1) == 0].all()
    else:
        # a long item in a group of its own turns the task to the strip form in task order
        extra = torch.ones((66 + 3,) + feats.shape[1:], dtype=feats.dtype)
        off2 = np.concatenate([off, off[-1] + np.array([1, 67, 69])]).astype(np.int64)
        attrs2 = np.concatenate([attrs, [[0, 9999], [0, 9999], [1, 9999]]]).astype(np.int32)
        t2 = fx.Task(fx.Dataset(ctx(), torch.cat([feats, extra]).cuda().contiguous(), off2, attrs2), 0, [1])
        strips = t2.score(keep_pairs=True, **opts)
        xs, ys = np.nonzero((attrs[:, None, 1] == attrs[None, :, 1]) & (attrs[:, None, 1] > 0))
        assert np.array_equal(res.pairs(xs, ys)[0], strips.pairs(xs, ys)[0])
        assert np.array_equal(res.half_units, strips.half_units[:len(res.half_units)])


# Collapse of many cells with a sparse key space (buckets of the key's top bits)
# and of few (one sort), bit for bit the level-by-level definition: rows of equal
# kept keys averaged, summed in row order, in key order.
@pytest.mark.parametrize("labels,sorted_by", [(100, "buckets"), (12, "one sort")])
def test_collapse_sparse_keys(labels, sorted_by):
    import paper_2505_02692_amd as fx
    from test_gpu_parity import ctx
    rng = np.random.default_rng(31)
    attrs = np.array([(lab, c, sp) for lab in range(labels) for c in range(3)
                      for sp in rng.choice(60, 6, replace=False)], np.int32)
    n = len(attrs)
    feats = torch.from_numpy(rng.standard_normal((n, 8), dtype=np.float32)).cuda()
    print(f"[case] collapse sparse {sorted_by} items={n}", flush=True)
    t = fx.Task(fx.Dataset(ctx(), feats, np.arange(n + 1), attrs), 0, [1], [2])
    res = t.score(mode="pooled")
    keys, attr_of = t.keys, np.array([0, 0, 1, 2, 2])
    score = res.half_units / (2.0 * res.n_triplets)
    assert (len(score) >= 1 << 15) == (sorted_by == "buckets")
    for levels in ([[1], [2]], [[1]], [[1, 2]]):
        rows, cols = score, keys
        attr = attr_of
        for lv in levels:
            keep = ~np.isin(attr, lv)
            cols, attr = cols[:, keep], attr[keep]
            uniq, first, inv = np.unique(cols, axis=0, return_index=True, return_inverse=True)
            total = np.zeros(len(uniq))
            np.add.at(total, inv.ravel(), rows)  # one by one, in row order
            rows, cols = total / np.bincount(inv.ravel()), uniq
        assert res.collapse(levels) == 1.0 - np.cumsum(rows)[-1] / len(rows)


# Rows of large cells with more infinities than a bucket takes (frames whose FP32
# length overflows, in the Euclidean BF16 form): the sort's padding must not come
# before the row's own infinities, whose places it would stand for.
@pytest.mark.parametrize("na,nb", [(40, 300), (12, 1025)])
def test_sorted_rows_with_infinities(na, nb):
    rng = np.random.default_rng(na)
    n = na + nb
    x = rng.standard_normal((n, 8)).astype(np.float32)
    x[::2] *= 1e25
    attrs = np.stack([np.r_[np.zeros(na, np.int32), np.ones(nb, np.int32)], np.zeros(n, np.int32)], 1)
    w = workloads.Workload("infinities", torch.from_numpy(x), np.arange(n + 1, dtype=np.int64), attrs, ["l", "g"], 0,
                           [1], [])
    print(f"[case] sorted rows with infinities na={na} nb={nb}", flush=True)
    t, res = gpu_score(w, mode="pooled", distance="euclidean", keep_pairs=True)
    orc = oracle.score(x, w.offsets, attrs, 0, [1], [], "pooled", "path", distance="euclidean")
    xs, ys, _ = all_oracle_pairs(orc)
    f32, fl, _ = res.pairs(xs, ys)
    assert np.isinf(f32).sum() > 1000 and ((fl & 2) != 0).all()  # the margin is infinite too
    assert np.array_equal(res.half_units, orc.half_units)


# Rows of large cells with NaN distances (features with NaN or infinities): a
# comparison with a NaN is neither less nor equal, so it adds nothing, whatever its
# place in the sorted row.  One NaN (the insertion sort of a bucket) and more than a
# bucket takes, in the plain form's values and in the FP64 ones of the recheck.
@pytest.mark.parametrize("n_odd", [1, 60])
@pytest.mark.parametrize("precision,distance,value", [("fp32", "euclidean", np.nan), ("bf16", "angular", np.inf),
                                                      ("bf16", "euclidean", np.nan)])
@pytest.mark.parametrize("na,nb", [(40, 300), (12, 1025)])
def test_sorted_rows_with_nan(na, nb, precision, distance, value, n_odd):
    rng = np.random.default_rng(nb)
    n = na + nb
    x = rng.standard_normal((n, 8)).astype(np.float32)
    x[rng.choice(np.arange(na, n), n_odd, replace=False), 3] = value
    x[rng.choice(na, 3, replace=False), 5] = value
    attrs = np.stack([np.r_[np.zeros(na, np.int32), np.ones(nb, np.int32)], np.zeros(n, np.int32)], 1)
    w = workloads.Workload("nan", torch.from_numpy(x), np.arange(n + 1, dtype=np.int64), attrs, ["l", "g"], 0, [1], [])
    print(f"[case] sorted rows with NaN na={na} nb={nb} {precision} {distance} n_odd={n_odd}", flush=True)
    t, res = gpu_score(w, mode="pooled", precision=precision, distance=distance, margin=1e4, keep_pairs=True)
    xs, ys = (v.ravel() for v in np.meshgrid(np.arange(n), np.arange(n), indexing="ij"))
    f32, fl, f64 = res.pairs(xs, ys)
    if precision == "bf16":
        assert ((fl & 2) != 0)[xs != ys].all()
    d = (f32 if precision == "fp32" else f64).reshape(n, n)
    assert np.isnan(d[:na, na:]).any()
    want = []
    for A, B in ((np.arange(na), np.arange(na, n)), (np.arange(na, n), np.arange(na))):
        s = 0
        for i in A:
            a, b = d[i, A[A != i]][:, None], d[i, B][None]
            s += 2 * int((a < b).sum()) + int((a == b).sum())
        want.append(s)
    assert res.half_units.tolist() == want


# The FP64 recheck of features with infinities or NaN.  Euclidean distances of frames
# with equal infinities are NaN among infinite ones: there the order of comparisons
# shows in the costs, and each orientation has its own.
@pytest.mark.parametrize("norm", ["path", "none"])
@pytest.mark.parametrize("distance,value", [("angular", np.inf), ("euclidean", np.nan), ("euclidean", np.inf)])
@pytest.mark.parametrize("case", list(RECHECK))
def test_fp64_recheck_nan(case, distance, value, norm):
    w = workloads.batched_c4(centroid_std=0.1, seed=82, **dict(RECHECK[case], dtype=torch.float32))
    rng = np.random.default_rng(7)
    for k in range(0, w.n_items, 2):
        lo, hi = int(w.offsets[k]), int(w.offsets[k + 1])
        for f in rng.integers(lo, hi, 3):
            w.features[int(f), int(rng.integers(0, 2))] = value if k % 3 else -value
    print(f"[case] recheck with NaN {case} {distance} {value} {norm} items={w.n_items}", flush=True)
    t, res = gpu_score(w, norm=norm, distance=distance, margin=1e4, keep_pairs=True)
    orc = oracle.score(w.features_f32_host(), w.offsets, w.attrs, w.on, w.by, w.across, "dtw", norm, distance=distance)
    xs, ys, want = [], [], []
    for items, m in orc.groups.values():
        i, j = np.nonzero(~np.eye(len(items), dtype=bool))
        xs.append(items[i])
        ys.append(items[j])
        want.append(m[i, j])
    xs, ys, want = (np.concatenate(v) for v in (xs, ys, want))
    _, fl, f64 = res.pairs(xs, ys)
    # pairs with an item of more than 64 frames are in FP64 from the start, marked or not
    # (an unmarked one's value is returned rounded to FP32)
    length, marked = np.diff(w.offsets), (fl & 2) != 0
    known = marked | (np.maximum(length[xs], length[ys]) > 64)
    assert np.isnan(want[known]).any()
    if np.isinf(value) and distance == "euclidean":
        swapped = {(int(x), int(y)): v for x, y, v in zip(xs, ys, want)}
        assert any(np.isnan(v) != np.isnan(swapped[int(y), int(x)]) for x, y, v in zip(xs, ys, want))
        assert known.mean() > 0.9  # infinite values tie, and are not compared in FP64 for that alone
    else:
        assert known.all()
        assert np.array_equal(res.half_units, orc.half_units)
    assert np.array_equal(np.isnan(f64[known]), np.isnan(want[known]))
    assert np.array_equal(np.isinf(f64[known]), np.isinf(want[known]))
    ok = marked & np.isfinite(want)
    assert (np.abs(f64[ok] - want[ok]) <= 1e-12 * np.maximum(want[ok], 1.0)).all()


# Rows of large cells at the edges of the sort's sizes (64 places a wave, 256 to 4096
# a block), with many equal values and one far away: counts by the definition from
# the pair values they compare, and every near tie marked.
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("nb", [2, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 2048, 2049])
def test_sorted_row_sizes(nb, precision):
    rng = np.random.default_rng(nb)
    na = max(2, -(-8192 // nb))
    n = na + nb
    x = rng.integers(1, 9, (n, 3)).astype(np.float32)
    x[n - 1] = (-50, -49, -51)
    attrs = np.stack([np.r_[np.zeros(na, np.int32), np.ones(nb, np.int32)], np.zeros(n, np.int32)], 1)
    w = workloads.Workload("sizes", torch.from_numpy(x), np.arange(n + 1, dtype=np.int64), attrs, ["l", "g"], 0, [1], [])
    print(f"[case] sorted row sizes nb={nb} na={na} {precision}", flush=True)
    t, res = gpu_score(w, mode="pooled", precision=precision, keep_pairs=True, **({"margin": 1e-3} if precision == "bf16" else {}))
    xs, ys = (v.ravel() for v in np.meshgrid(np.arange(n), np.arange(n), indexing="ij"))
    f32, fl, f64 = (v.reshape(n, n) for v in res.pairs(xs, ys))
    marked = (fl & 2) != 0
    want = []
    for A, B in ((np.arange(na), np.arange(na, n)), (np.arange(na, n), np.arange(na))):
        s = 0
        for i in A:
            a, b = A[A != i][:, None], B[None]
            both = marked[i, a] & marked[i, b]
            s += 2 * int(np.where(both, f64[i, a] < f64[i, b], f32[i, a] < f32[i, b]).sum())
            s += int(np.where(both, f64[i, a] == f64[i, b], f32[i, a] == f32[i, b]).sum())
            if precision == "bf16":
                assert both[np.abs(f32[i, a] - f32[i, b]) <= 0.99e-3].all()
        want.append(s)
    assert res.half_units.tolist() == want


# The memory a server counts for a job: plain and unit scores of items of at most 64
# frames take no distance matrix, so they are admitted next to one another in a
# budget far below their squared frame count.
@pytest.mark.parametrize("kind", ["fp32", "units"])
def test_server_admits_plain_jobs_without_a_distance_buffer(kind):
    import paper_2505_02692_amd as fx
    from test_gpu_parity import ctx
    rng = np.random.default_rng(2)
    n, budget = 600, 64 << 20
    length = rng.integers(10, 31, n)
    off = np.concatenate([[0], np.cumsum(length)]).astype(np.int64)
    assert int(off[-1]) ** 2 * 4 > 8 * budget
    attrs = np.stack([np.arange(n) % 3, np.zeros(n)], 1).astype(np.int32)
    feats = (torch.from_numpy(rng.integers(0, 9, int(off[-1])).astype(np.int32)) if kind == "units" else
             torch.from_numpy(rng.standard_normal((int(off[-1]), 16), dtype=np.float32)))
    opts = dict(distance="units") if kind == "units" else dict(precision="fp32")
    print(f"[case] server budget {kind}", flush=True)
    ds = fx.Dataset(ctx(), feats.cuda().contiguous(), off, attrs)
    want = fx.Task(ds, 0, [1]).score(**opts).half_units
    srv = fx.Server(ctx(), hbm_budget_bytes=budget, n_streams=2)
    ids = [srv.submit(ds, 0, [1], **opts) for _ in range(3)]
    got = [srv.wait(i)[1] for i in ids]
    high = srv.stats["hbm_high_water"]
    srv.close()
    assert all(np.array_equal(g, want) for g in got) and 0 < high <= budget


# The packing order of a task's items (16 bytes each on the device) counts in a job's
# footprint: the same items in task order, which one group with an item of more than
# 64 frames makes them keep, count that much less but for the group itself.
def test_server_footprint_counts_the_packing_order():
    import re
    import paper_2505_02692_amd as fx
    from test_gpu_parity import ctx
    n = 10000
    off = np.arange(0, 6 * n + 1, 6, dtype=np.int64)
    attrs = np.stack([np.arange(n) % 2, np.arange(n) // 500], 1).astype(np.int32)
    off2 = np.concatenate([off, off[-1] + np.array([1, 2, 67])]).astype(np.int64)
    attrs2 = np.concatenate([attrs, [[0, 99], [1, 99], [0, 99]]]).astype(np.int32)
    srv = fx.Server(ctx(), hbm_budget_bytes=1, n_streams=1)
    footprint = []
    for o, a in ((off, attrs), (off2, attrs2)):
        ds = fx.Dataset(ctx(), torch.ones((int(o[-1]), 4), device="cuda"), o, a)
        with pytest.raises(fx.FabxError) as e:
            srv.submit(ds, 0, [1])
        footprint.append(int(re.search(r"footprint (\d+) bytes", str(e.value)).group(1)))
    srv.close()
    assert footprint[0] - footprint[1] >= 16 * n - 32768


# The rounding of the FP64 distances over many features: an angle or a length takes
# about ten roundings after its sums, whose own error, added up in blocks, is no
# more than theirs: 1.5 half units in the last place as a root mean square (one chain
# over 1024 features: 2.7 and more).
@pytest.mark.parametrize("distance", ["angular", "euclidean"])
@pytest.mark.parametrize("mode", ["dtw", "pooled"])
@pytest.mark.parametrize("dim", [64, 1024])
def test_fp64_recheck_rounding(dim, mode, distance):
    n, m = dim + 6 if mode == "pooled" else 60, 60
    w = workloads.batched_c4(n_groups=1, size_lo=n, size_hi=n, len_lo=1, len_hi=1, dim=dim, dtype=torch.float32,
                             centroid_std=0.1, seed=n)
    print(f"[case] rounding {mode} {distance} dim={dim}", flush=True)
    t, res = gpu_score(w, mode=mode, distance=distance, margin=1e4, keep_pairs=True)
    xs, ys = np.triu_indices(m, 1)
    _, fl, f64 = res.pairs(xs, ys)
    assert ((fl & 2) != 0).all()
    f = w.features[:m].numpy().astype(np.longdouble)
    if distance == "angular":
        u = f / np.sqrt((f * f).sum(1, keepdims=True))
        want = np.arccos((u[xs] * u[ys]).sum(1)) / (4 * np.arctan(np.longdouble(1)))
    else:
        want = np.sqrt(((f[xs] - f[ys]) ** 2).sum(1))
    assert np.sqrt((((f64 - want) / want) ** 2).mean()) <= 1.5 * 2.0 ** -53


# The FP64 distance of two frames is the same in the kernels of all length classes: one
# frame against k copies of another costs k times their distance, added one by one.
@pytest.mark.parametrize("distance", ["angular", "euclidean"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("dim", [47, 200, 1000])
def test_fp64_recheck_same_sums_in_all_classes(dim, dtype, distance):
    rng = np.random.default_rng(dim)
    copies, n = [1, 7, 20, 40, 64, 65, 130], 6
    f = torch.from_numpy(rng.standard_normal((2 * n, dim)).astype(np.float32)).to(dtype)
    feats, length, attrs = [], [], []
    for i in range(n):  # group i: the frame, the other's copies, and a second of the frame's label
        for label, frame, k in [(0, 2 * i, 1)] + [(1, 2 * i + 1, k) for k in copies] + [(0, 2 * i + 1, 2)]:
            feats.append(f[frame].repeat(k, 1))
            length.append(k)
            attrs.append((label, i))
    w = workloads.Workload("copies", torch.cat(feats), np.concatenate([[0], np.cumsum(length)]).astype(np.int64),
                           np.array(attrs, np.int32), ["l", "g"], 0, [1], [])
    print(f"[case] copies dim={dim} {dtype} {distance}", flush=True)
    t, res = gpu_score(w, norm="none", distance=distance, margin=1e4, keep_pairs=True)
    per = len(copies) + 2
    for i in range(n):
        ys = np.arange(i * per + 1, i * per + 1 + len(copies))
        _, fl, f64 = res.pairs(np.full(len(ys), i * per), ys)
        assert ((fl & 2) != 0).all()
        assert np.array_equal(f64, [np.cumsum(np.full(k, f64[0]))[-1] for k in copies])


# Cells whose |A| x |B| fits a wave's lanes, those just past it, and cells of more rows
# x than a unit takes: few units (split by x once more) and many, X = A without x itself and X of another speaker.  Points of a coarse
# lattice, so that many comparisons tie or are left to the recount.
@pytest.mark.parametrize("groups", [3, 300])
@pytest.mark.parametrize("across", [False, True])
@pytest.mark.parametrize("na,nb", [(2, 1), (2, 2), (9, 7), (8, 8), (13, 5), (64, 1), (65, 1), (3, 21), (3, 22),
                                   (90, 1), (17, 40), (40, 17), (33, 2), (128, 3)])
def test_triplet_units_by_grid(na, nb, across, groups):
    rng = np.random.default_rng(na * 100 + nb)
    label = np.tile(np.r_[np.zeros(na, np.int32), np.ones(nb, np.int32)], (1 + across) * groups)
    speaker = np.tile(np.repeat(np.arange(1 + across), na + nb), groups)
    group = np.repeat(np.arange(groups), (1 + across) * (na + nb))
    n = len(label)
    x = rng.integers(1, 7, (n, 3)).astype(np.float32)
    attrs = np.stack([label, group, speaker], 1).astype(np.int32)
    w = workloads.Workload("grid", torch.from_numpy(x), np.arange(n + 1, dtype=np.int64), attrs, ["l", "g", "s"], 0, [1],
                           [2] if across else [])
    print(f"[case] units by grid na={na} nb={nb} across={across} groups={groups}", flush=True)
    t, res = gpu_score(w, mode="pooled", margin=1e-3, keep_pairs=True)
    # the definition, from the pair values that the counts compare
    per = n // groups
    xs, ys = (v.ravel() for v in np.meshgrid(np.arange(n), np.arange(per), indexing="ij"))
    f32, fl, f64 = (v.reshape(groups, per, per) for v in res.pairs(xs, xs // per * per + ys))
    marked = (fl & 2) != 0
    want, n_near = [], 0
    for c in oracle.cells(attrs, 0, [1], w.across):
        g, s = c.A[0] // per, 0
        for i in c.X % per:
            a, b = (c.A[c.A != c.X[0] // per * per + i] if c.exclude_self else c.A)[:, None] % per, c.B[None] % per
            both = marked[g, i, a] & marked[g, i, b]
            near = np.abs(f32[g, i, a] - f32[g, i, b]) <= 0.99e-3
            assert both[near].all()
            n_near += int(near.sum())
            s += 2 * int(np.where(both, f64[g, i, a] < f64[g, i, b], f32[g, i, a] < f32[g, i, b]).sum())
            s += int(np.where(both, f64[g, i, a] == f64[g, i, b], f32[g, i, a] == f32[g, i, b]).sum())
        want.append(s)
    assert n_near > 0 or groups * na * nb < 20
    wrong = np.flatnonzero(res.half_units != want)
    assert len(wrong) == 0, f"{len(wrong)} of {len(want)} cells"


# More units than kManyUnits (524,288), which a wave takes many at a time: cells on
# both sides of the 24 comparisons that one lane does alone, X = A without x itself and
# X of another speaker, rows left to the recount.
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("across", [False, True])
def test_triplets_of_many_units(across, precision):
    rng = np.random.default_rng(9)
    # (items of label 0, of label 1, groups); comparisons a cell: 8, 24, 24, 27, 48, 288, 729 (or without x itself)
    shapes = [(2, 2, 200000), (2, 6, 20000), (6, 2, 20000), (3, 3, 30000), (2, 12, 3000), (12, 2, 3000), (9, 9, 1000)]
    if across:
        shapes = [(a, b, g // 2) for a, b, g in shapes]
    spk = 1 + across
    label = np.concatenate([np.tile(np.r_[np.zeros(a, np.int32), np.ones(b, np.int32)], spk * g) for a, b, g in shapes])
    speaker = np.concatenate([np.tile(np.repeat(np.arange(spk), a + b), g) for a, b, g in shapes])
    size = np.concatenate([np.full(g, spk * (a + b)) for a, b, g in shapes])
    n = len(label)
    attrs = np.stack([label, np.repeat(np.arange(len(size)), size), speaker], 1).astype(np.int32)
    x = rng.integers(1, 9, (n, 3)).astype(np.float32)
    w = workloads.Workload("many", torch.from_numpy(x), np.arange(n + 1, dtype=np.int64), attrs, ["l", "g", "s"], 0, [1],
                           [2] if across else [])
    print(f"[case] many units across={across} {precision} items={n}", flush=True)
    t, res = gpu_score(w, mode="pooled", precision=precision, keep_pairs=True,
                       **({"margin": 1e-3} if precision == "bf16" else {}))
    assert len(t) >= 16 * 32768
    keys, hu = t.keys, res.half_units
    first_item = first_cell = 0
    for a, b, g in shapes:
        per = a + b
        # a group's cells in key order: labels (0, 1) then (1, 0), then speakers
        local = []
        for on, A0, B0 in ((0, np.arange(a), a + np.arange(b)), (1, a + np.arange(b), np.arange(a))):
            for s in range(spk):
                local.append((on, s, A0 + s * per, B0 + s * per, A0 + (spk - 1 - s) * per))
        m = spk * per
        i, j = (v.ravel() for v in np.meshgrid(np.arange(m), np.arange(m), indexing="ij"))
        at = first_item + m * np.arange(g)[:, None]
        f32, fl, f64 = (v.reshape(g, m, m) for v in res.pairs((at + i).ravel(), (at + j).ravel()))
        marked = (fl & 2) != 0
        got, k = (v[first_cell:first_cell + g * len(local)].reshape(g, len(local), -1) for v in (hu, keys))
        for c, (on, s, A, B, X) in enumerate(local):
            assert (k[:, c, 0] == on).all() and (k[:, c, 1] == 1 - on).all()
            assert not across or (k[:, c, 3] == s).all()
            want = np.zeros(g, np.int64)
            for xx in X:
                for aa in A:
                    if aa == xx:
                        continue
                    for bb in B:
                        both = marked[:, xx, aa] & marked[:, xx, bb]
                        da, db = (np.where(both, f64[:, xx, v], f32[:, xx, v].astype(np.float64)) for v in (aa, bb))
                        want += 2 * (da < db) + (da == db)
                        if precision == "bf16":
                            assert both[np.abs(f32[:, xx, aa] - f32[:, xx, bb]) <= 0.99e-3].all()
            assert np.array_equal(got[:, c, 0], want)
        first_item += g * m
        first_cell += g * len(local)
    assert precision == "fp32" or res.stats["n_recount_rows"] > 10000


# The plain form's strips, which a task with an item of more than 64 frames takes: many
# batches through a small buffer, one item a strip (items of up to 90 frames in groups of
# about 700), equal the one batch of the full buffer bit for bit, and the oracle.
@pytest.mark.parametrize("norm", ["path", "none"])
@pytest.mark.parametrize("distance", ["angular", "euclidean", "units"])
def test_plain_strips_in_batches(monkeypatch, distance, norm):
    import paper_2505_02692_amd as fx
    from test_gpu_parity import ctx
    w = workloads.batched_c4(n_groups=6, size_lo=14, size_hi=16, len_lo=3, len_hi=90, dim=20, dtype=torch.float32,
                             centroid_std=0.3, seed=23)
    if distance == "units":
        w.features = torch.from_numpy(np.random.default_rng(4).integers(0, 4, w.n_frames).astype(np.int32))
    length = np.diff(w.offsets)
    assert length.max() > 64
    opts = dict(precision="fp32", distance=distance, norm=norm, keep_pairs=True)
    ds = fx.Dataset(ctx(), w.features.cuda().contiguous(), w.offsets, w.attrs)
    res = {}
    for cells in ("4096", "40000", None):
        print(f"[case] strips in batches {distance} {norm} cells={cells}", flush=True)
        monkeypatch.delenv("FABX_PLAIN_DMAT_CELLS", raising=False)
        if cells:
            monkeypatch.setenv("FABX_PLAIN_DMAT_CELLS", cells)
        res[cells] = fx.Task(ds, w.on, w.by).score(**opts)
    feats = w.features.reshape(-1, 1).float().numpy() if distance == "units" else w.features_f32_host()
    orc = oracle.score(feats, w.offsets, w.attrs, w.on, w.by, [], "dtw", norm, distance=distance)
    xs, ys, want = all_oracle_pairs(orc)
    whole = res[None]
    f32 = whole.pairs(xs, ys)[0]
    for cells in ("4096", "40000"):
        assert np.array_equal(res[cells].half_units, whole.half_units)
        assert np.array_equal(res[cells].pairs(xs, ys)[0], f32)
    # FP32 sums: 2e-6 a step of the path, as for the whole form
    steps = length[xs] + length[ys] - 1 if norm == "none" else 1
    assert (np.abs(f32 - want) <= 2e-6 * steps * np.maximum(1, w.features.abs().max().item())).all()
    if distance == "units":
        assert np.array_equal(whole.half_units, orc.half_units)


# The no-allocation score of discrete units where the fused kernel's tables (with the
# packing order's) no longer fit the scratch beside the task, but strips through a small
# distance buffer do: a number of groups between those and the first that is refused.
def test_noalloc_units_fall_back_to_strips():
    import paper_2505_02692_amd as fx
    from test_gpu_parity import ctx
    rng = np.random.default_rng(8)
    per, L, most = 4, 60, 220000
    codes = torch.from_numpy(rng.integers(0, 5, most * per * L).astype(np.int32)).cuda()
    off = np.arange(0, most * per * L + 1, L, dtype=np.int64)
    attrs = np.stack([np.arange(most * per) % 2, np.arange(most * per) // per], 1).astype(np.int32)
    opts = fx.make_opts(distance="units")

    def attempt(groups):
        n = groups * per
        t = fx.Task(fx.Dataset(ctx(), codes[:n * L], off[:n + 1], attrs[:n]), 0, [1])
        print(f"[case] noalloc units, {groups} groups", flush=True)
        try:
            return t, fx.fabx_score_noalloc(t.h, opts, len(t))
        except fx.FabxError as e:
            assert e.code == -2
            return None

    lo, hi = 120000, most   # taken, refused
    t, (got, st) = attempt(lo)
    assert st["computed_dtw_cells"] != lo * (per * L) ** 2  # the fused kernel
    assert attempt(hi) is None
    while hi - lo > 1 and st["computed_dtw_cells"] != lo * (per * L) ** 2:
        mid = (lo + hi) // 2
        res = attempt(mid)
        if res is None:
            hi = mid
        else:
            lo, (t, (got, st)) = mid, res
    assert st["computed_dtw_cells"] == lo * (per * L) ** 2  # strips
    assert np.array_equal(got, t.score(distance="units").half_units)


# A task that would have a packing order makes it, its row blocks and plans at the first
# score that reads them: every order of first uses gives the scores of a fresh task.
@pytest.mark.parametrize("sequence", ["pdsw", "sdpw", "ndps", "wdnp", "fpds", "psnfwd"])
def test_packing_order_made_on_first_use(sequence):
    import paper_2505_02692_amd as fx
    from test_gpu_parity import ctx
    rng = np.random.default_rng(5)
    n, per = 400, 100
    length = rng.integers(10, 17, n)
    off = np.concatenate([[0], np.cumsum(length)]).astype(np.int64)
    assert sum(int(off[k + per] - off[k]) ** 2 for k in range(0, n, per)) // n >= 12000
    attrs = np.stack([np.arange(n) % 3, np.arange(n) // per], 1).astype(np.int32)
    feats = torch.from_numpy(rng.standard_normal((int(off[-1]), 24), dtype=np.float32)).cuda()
    kinds = dict(p=dict(mode="pooled"), d=dict(), s=dict(fused_cols=512), w=dict(fused_cols=256),
                 f=dict(precision="fp32"), n=dict())
    ds = fx.Dataset(ctx(), feats, off, attrs)
    want = {k: fx.Task(ds, 0, [1]).score(**o).half_units for k, o in kinds.items()}
    t = fx.Task(ds, 0, [1])
    for k in sequence + sequence[::-1]:
        print(f"[case] order on first use {sequence} {k}", flush=True)
        got = (fx.fabx_score_noalloc(t.h, fx.make_opts(), len(t))[0] if k == "n" else t.score(**kinds[k]).half_units)
        assert np.array_equal(got, want[k])


# The no-allocation score takes the fewest triplet units where the task's own would not
# fit (three a cell here, 12 bytes each, against one): the largest task it takes is within
# a group of what the fewest need.
def test_noalloc_takes_the_fewest_units_at_its_limit():
    import re
    import paper_2505_02692_amd as fx
    from test_gpu_parity import ctx
    rng = np.random.default_rng(8)
    per, most = 36, 22000
    feats = torch.from_numpy(rng.standard_normal((most * per, 4), dtype=np.float32)).cuda()
    off = np.arange(most * per + 1, dtype=np.int64)
    attrs = np.stack([np.tile(np.r_[np.zeros(34, np.int32), 1, 1], most), np.arange(most * per) // per], 1).astype(np.int32)
    opts = fx.make_opts(mode="pooled", precision="fp32")

    def attempt(groups):
        n = groups * per
        t = fx.Task(fx.Dataset(ctx(), feats[:n], off[:n + 1], attrs[:n]), 0, [1])
        print(f"[case] noalloc fewest units, {groups} groups", flush=True)
        try:
            return t, fx.fabx_score_noalloc(t.h, opts, len(t))[0]
        except fx.FabxError as e:
            assert e.code == -2
            return int(re.search(r"needs (\d+) bytes", str(e)).group(1))

    lo, hi = 1000, most   # taken, refused
    small, _ = attempt(lo)
    need = attempt(hi)
    per_group = need / hi
    while hi - lo > 1:
        mid = (lo + hi) // 2
        res = attempt(mid)
        if isinstance(res, int):
            hi, need = mid, res
        else:
            lo, (t, got) = mid, res
    # refused by less than a group, of the bytes it takes with two units: frames, pair
    # matrix, items, cells, units, group tables, counts, tile prefix, row block
    assert abs(per_group - (36 * 64 * 4 + 36 * 36 * 4 + 36 * 24 + 2 * 32 + 2 * 12 + 5 * 8 + 2 * 8 + 8 + 16)) < 2
    assert need - (256 << 20) <= per_group + 4096
    assert np.array_equal(got, t.score(mode="pooled", precision="fp32").half_units)
    assert len(small) == 2000
