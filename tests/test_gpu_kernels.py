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
