// FP64 recomputation of the item-pair distances whose triplet comparisons
// were too close to call in BF16 / FP32, or whose DTW path length was not
// robust.  Works from the raw features (F32 or BF16 widened exactly):
//   unit vector  u times 1 / ||u||, ||u|| = sqrt of the sum of squares
//   cosine       sum of products of the unit vectors
//   angle        acos(cos) when |cos| < 1 - 2^-20, else from the half chord
//                ||u - v|| / 2 or ||u + v|| / 2, which stays accurate near 0 and pi
//   distance     angle / pi; DTW with the diagonal > left > up predecessor order
// or, for the Euclidean distance (euclid != 0), the square root of the sum of
// squared differences of the raw frames (or means).
// Contraction into FMA is disabled (the fused multiply-adds are written out).
//
// The cosines of a pair's frames are an FP64 matrix product and run on the
// matrix cores: v_mfma_f64_16x16x4, 16 x 16 frame pairs at a time, operands
// straight from the features into registers (no LDS staging).  Every sum goes
// through the same steps whatever the frames' places in the tiles and
// whichever item comes first (fused multiply-adds over the features in one fixed
// order, in blocks), so equal inputs still give equal distances, and the two
// orientations of a pair share one evaluation.  Only where Euclidean distances of
// frames with infinities are NaN does the order of comparisons show in the costs:
// such a pair's transposed problem is swept by itself, with its own comparisons.
// (An angular frame with an infinity is at NaN from every frame, and every path
// then meets that row or column, in either orientation.)
#include "device_common.h"
#include "kernels.h"

#pragma clang fp contract(off)

namespace fabx {
namespace kern {
namespace {

constexpr int kMaxL = 64;                    // items of at most this many frames: k_recheck_small, k_recheck_tiled
constexpr int kLongMax = FABX_MAX_ITEM_FRAMES;  // longer ones (up to this): k_long_dtw
constexpr double kPi = 3.14159265358979323846;

template <typename T>
__device__ __forceinline__ double ld(const T *p, int64_t i);
template <>
__device__ __forceinline__ double ld<double>(const double *p, int64_t i) { return p[i]; }
template <>
__device__ __forceinline__ double ld<float>(const float *p, int64_t i) { return double(p[i]); }
template <>
__device__ __forceinline__ double ld<uint16_t>(const uint16_t *p, int64_t i) {
    return double(__uint_as_float(uint32_t(p[i]) << 16));
}

// The per-lane loops over the features below are unrolled so that the loads
// of several features are in flight at once; each lane still adds its terms
// in feature order.

// Sum of a double over the wave (butterfly; every lane gets the sum).
__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, dev::kWave);
    return v;
}

// 1 / ||frame|| (the whole wave; every lane gets it).
template <typename T>
__device__ __forceinline__ double wave_inv_norm(const T *row, int dim, int lane) {
    double s = 0.0;
#pragma unroll 4
    for (int k = lane; k < dim; k += dev::kWave) {
        const double v = ld(row, k);
        s += v * v;
    }
    return 1.0 / sqrt(wave_sum_f64(s));
}

// Angle / pi of nearly parallel or opposite unit vectors u, v (|cos| within
// 2^-20 of 1, so the half chord h is below 1e-3) from sm = ||u - v||^2 and
// sp = ||u + v||^2: twice the arc sine of the half chord, whose series to h^7
// is exact to FP64 rounding there.
__device__ __forceinline__ double near_angle_over_pi(double sm, double sp) {
    const double h2 = 0.25 * fmin(sm, sp), h = sqrt(h2);
    const double a = 2.0 * h * (1.0 + h2 * (1.0 / 6.0 + h2 * (3.0 / 40.0 + h2 * (15.0 / 336.0)))) / kPi;
    return sm <= sp ? a : 1.0 - a;
}

// The same of frames f and g (the whole wave, its lanes splitting the
// dimension; every lane gets it).
template <typename T>
__device__ __forceinline__ double wave_near_distance(const T *f, const T *g, int dim, int lane) {
    const double su = wave_inv_norm(f, dim, lane), sv = wave_inv_norm(g, dim, lane);
    double sm = 0.0, sp = 0.0;
#pragma unroll 4
    for (int k = lane; k < dim; k += dev::kWave) {
        const double a = ld(f, k) * su, b = ld(g, k) * sv;
        sm += (a - b) * (a - b);
        sp += (a + b) * (a + b);
    }
    return near_angle_over_pi(wave_sum_f64(sm), wave_sum_f64(sp));
}

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) double lds_double;

// Value of lane - 1 over the whole wave, or within each row of 16 lanes; the
// first lane gets `edge`.
__device__ __forceinline__ int shr1(int edge, int v, std::false_type) {
    return __builtin_amdgcn_update_dpp(edge, v, 0x138, 0xf, 0xf, false);  // wave_shr:1
}
__device__ __forceinline__ int shr1(int edge, int v, std::true_type) {
    return __builtin_amdgcn_update_dpp(edge, v, 0x111, 0xf, 0xf, false);  // row_shr:1
}
// the cost above: +inf above the first row
template <typename Row16>
__device__ __forceinline__ double shr1_cost(double v, Row16 r) {
    const long long b = __builtin_bit_cast(long long, v);
    const uint32_t lo = uint32_t(shr1(0, int(b), r)), hi = uint32_t(shr1(0x7FF00000, int(b >> 32), r));
    return __builtin_bit_cast(double, (long long)((uint64_t(hi) << 32) | lo));
}

// One anti-diagonal sweep: lane i holds row i of a DTW and is on column t - i
// at step t.  The path lengths of both orientations go along, packed (low
// half: rows as given, diagonal before left before up on exact ties; high
// half: the transposed problem, whose left is this one's up).  The costs are
// the same in both.  Steps off a row's columns compute values that nothing
// reads: the first column of a row takes +inf to its left, and a row's last
// cell is read at its own step.  kFlip: the transposed problem alone, in the high
// half, with the costs its own comparisons choose (they differ where NaN occur).
template <bool kFlip>
struct Sweep {
    double c = 0.0, up_prev = 0.0;
    uint32_t len = 0, lup_prev = 0;
    // first: column 0; row0: no row above at all; up, lup: the cell above (+inf, 0 for row0)
    __device__ __forceinline__ void step(bool first, bool row0, double d, double up, uint32_t lup) {
        constexpr double inf = __builtin_huge_val();
        const double diag = first ? (row0 ? 0.0 : inf) : up_prev;  // virtual cell (-1, -1): cost 0, length 0
        const double left = first ? inf : c;
        const bool from_diag = diag <= left && diag <= up;
        const bool from_left = row0 || left <= up;  // before up, rows as given
        const bool from_up = (kFlip && first) || up <= left;  // before left, transposed
        const double best = from_diag ? diag : (kFlip ? !from_up : from_left) ? left : up;
        const uint32_t lo = from_diag ? lup_prev : from_left ? len : lup;
        const uint32_t hi = from_diag ? lup_prev : from_up ? lup : len;
        up_prev = up;
        lup_prev = lup;
        c = best + d;
        len = ((hi & 0xFFFF0000u) | (lo & 0xFFFFu)) + 0x00010001u;
    }
};

// A whole DTW of rows of at most 64 (Row16: 16) lanes, lane i (first lane of the
// wave, or of its 16) on row i: row = its distances, steps t = 0 .. steps - 1,
// fin = the step of the lane's result.  Distances are read four steps ahead;
// the reads may run 8 past the last column and i before the first (the rows
// lie one after another, so both stay in the tile or its pad of 8).
template <typename Row16, bool kFlip = false>
__device__ __forceinline__ void sweep_rows(const double *row, int i, int steps, int fin, double &cost,
                                           uint32_t &len) {
    Sweep<kFlip> w;
    const double *at = row - i;
    double da[4], db[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) da[k] = at[k];
    auto four = [&](const double (&d)[4], int t0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int t = t0 + k;
            const double up = shr1_cost(w.c, Row16{});
            const uint32_t lup = uint32_t(shr1(0, int(w.len), Row16{}));
            w.step(t == i, i == 0, d[k], up, lup);
            if (t == fin) {
                cost = w.c;
                len = w.len;
            }
        }
    };
    for (int t = 0; t < steps; t += 8) {
#pragma unroll
        for (int k = 0; k < 4; ++k) db[k] = at[min(t + 4 + k, steps + 3)];
        four(da, t);
#pragma unroll
        for (int k = 0; k < 4; ++k) da[k] = at[min(t + 8 + k, steps + 3)];
        four(db, t + 4);
    }
}

// Four features of a row as they are stored.  load4 takes them with one access
// of the element type's alignment (rows of any width and base: the hardware
// takes dword and byte aligned vector loads); load4_tail fills with zeros past
// dim.  widen: one of them, exactly.
template <typename T>
struct Four;
template <>
struct Four<float> {
    typedef float V __attribute__((ext_vector_type(4), aligned(4)));
};
template <>
struct Four<uint16_t> {
    typedef unsigned short V __attribute__((ext_vector_type(4), aligned(2)));
};
template <>
struct Four<double> {
    typedef double V __attribute__((ext_vector_type(4), aligned(8)));
};
template <typename T>
__device__ __forceinline__ typename Four<T>::V load4(const T *p) {
    return *reinterpret_cast<const typename Four<T>::V *>(p);
}
template <typename T>
__device__ __forceinline__ typename Four<T>::V load4_tail(const T *row, int k, int dim) {
    typename Four<T>::V v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = k + e < dim ? row[k + e] : T(0);
    return v;
}
__device__ __forceinline__ double widen(double d) { return d; }
__device__ __forceinline__ double widen(float f) { return double(f); }
__device__ __forceinline__ double widen(unsigned short h) { return double(dev::bf16_to_f32(h)); }

// Sum over the four lanes that share lane % 16 (each holds the features
// 16 c + 4 (lane / 16) + 0..3 of its frame); every lane gets it.
__device__ __forceinline__ double sum_quarters(double v) {
    v += __shfl_xor(v, 16, dev::kWave);
    v += __shfl_xor(v, 32, dev::kWave);
    return v;
}

__device__ __forceinline__ double ror1(double v) {
    const long long b = __builtin_bit_cast(long long, v);
    const uint32_t lo = uint32_t(__builtin_amdgcn_update_dpp(0, int(b), 0x121, 0xf, 0xf, true));
    const uint32_t hi = uint32_t(__builtin_amdgcn_update_dpp(0, int(b >> 32), 0x121, 0xf, 0xf, true));
    return __builtin_bit_cast(double, (long long)((uint64_t(hi) << 32) | lo));
}

// Distances of kT tiles of 16 x 16 frame pairs by one wave.  Tile u: rows are
// the frames pa(u)(0..nr-1), columns pb(u)(0..nc-1); lane l loads row and column
// frame l % 16 (clamped to the last one) and the features 4 (l / 16) + 0..3 of
// each 16.  at(u, i, j) is where element (i, j) goes in LDS (also those of
// clamped rows and columns).
//  angular: cos from the MFMA accumulators (register r of lane l is row
//    l / 16 + 4 r, column l % 16) times the inverse norms, whose sums of squares
//    come from the same loads; an element with |cos| within 2^-20 of 1 is
//    redone afterwards by the whole wave with the half-chord sums.
//  Euclidean: the differences cannot go through a product without cancelling,
//    so each lane keeps its row frame against all 16 column frames, which it
//    gets by rotating them through the 16 lanes (DPP), and sums the squares of
//    its quarter of the features.  Returns whether this lane met a NaN distance.
//    (only where want(u, i, j))
// The sums are made in blocks of features that are then added up (the products in
// the elements' own places in LDS, at a turn of the load pipeline: a test per 16
// features for a block by width cost long items 5%), which keeps their rounding to
// that of a sum split over 64 lanes: at 1024 features one chain is off by 3.1e-16
// (relative, root mean square over frame pairs), the blocks by 0.9e-16, for 3% of a
// pass over 365,261 pairs of 5-25 frames, 768 features.  Blocks are the same in every
// kernel, and with them the distance of two frames.
struct All {
    __device__ bool operator()(int, int, int) const { return true; }
};
template <typename T, bool kEuclid, int kT, int kStages = sizeof(T) == 4 ? 2 : 4, typename Ptr, typename At,
          typename Want = All>
__device__ __forceinline__ bool tile_distances(int n_tiles, Ptr &&ptr, int dim, At &&at, Want &&want = All{}) {
    const int lane = threadIdx.x % dev::kWave, i16 = lane % 16, q = lane / 16;
    const T *pa[kT], *pb[kT];
    int nr[kT], nc[kT];
#pragma unroll
    for (int u = 0; u < kT; ++u) {
        pa[u] = pb[u] = nullptr;
        nr[u] = nc[u] = 0;
        if (u < n_tiles) {
            const T *a0, *b0;
            ptr(u, a0, nr[u], b0, nc[u]);
            pa[u] = a0 + int64_t(min(i16, nr[u] - 1)) * dim;
            pb[u] = b0 + int64_t(min(i16, nc[u] - 1)) * dim;
        }
    }
    bool odd = false;
    if constexpr (kEuclid) {
        for (int u = 0; u < n_tiles; ++u) {
            const T *a_row = pa[0], *b_row = pb[0];
#pragma unroll
            for (int k = 1; k < kT; ++k)
                if (k == u) { a_row = pa[k]; b_row = pb[k]; }
            double acc[16], sum[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = sum[r] = 0.0;
            for (int k0 = 0; k0 < dim; k0 += 16) {
                if (k0 > 0 && k0 % 32 == 0)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        sum[r] += acc[r];
                        acc[r] = 0.0;
                    }
                const bool whole = k0 + 16 <= dim;
                const typename Four<T>::V a = whole ? load4(a_row + k0 + 4 * q) : load4_tail(a_row, k0 + 4 * q, dim);
                const typename Four<T>::V b = whole ? load4(b_row + k0 + 4 * q) : load4_tail(b_row, k0 + 4 * q, dim);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double x = widen(a[e]);
                    double y = widen(b[e]);
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const double d = x - y;
                        acc[r] = __builtin_fma(d, d, acc[r]);
                        y = ror1(y);
                    }
                }
            }
            int j = i16;  // the column frame of rotation r, moved along with the values
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const double s = sum_quarters(sum[r] + acc[r]);
                odd = odd || s != s;
                if (q == r / 4) *at(u, i16, j) = sqrt(s);
                j = __builtin_amdgcn_update_dpp(0, j, 0x121, 0xf, 0xf, true);
            }
        }
    } else {
        constexpr int kBlock = 64;  // a multiple of every kernel's turn
        f64x4 acc[kT];
        double sa[kT], sb[kT], na[kT], nb[kT];  // a block's norm sums, and those of the blocks before
#pragma unroll
        for (int u = 0; u < kT; ++u) {
            acc[u] = f64x4{0.0, 0.0, 0.0, 0.0};
            sa[u] = sb[u] = na[u] = nb[u] = 0.0;
        }
        // the end of a block: its products are added up in the elements' places
        auto flush = [&](bool first) {
#pragma unroll
            for (int u = 0; u < kT; ++u)
                if (u < n_tiles) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        double *d = at(u, q + 4 * r, i16);
                        if (first) *d = acc[u][r];
                        else __builtin_amdgcn_ds_atomic_fadd_f64((lds_double *)d, acc[u][r]);
                    }
                    acc[u] = f64x4{0.0, 0.0, 0.0, 0.0};
                    na[u] += sa[u];
                    nb[u] += sb[u];
                    sa[u] = sb[u] = 0.0;
                }
        };
        // kStages register buffers of 16 features each, kStages - 1 of them in
        // flight while the products take one.  BF16 frames hold four in few registers;
        // for FP32 two are as fast as three, which no longer fit beside the sums.
        typename Four<T>::V a[kStages][kT], b[kStages][kT];
        auto load = [&](int st, int k0) {
#pragma unroll
            for (int u = 0; u < kT; ++u)
                if (u < n_tiles) {
                    a[st][u] = load4(pa[u] + k0 + 4 * q);
                    b[st][u] = load4(pb[u] + k0 + 4 * q);
                }
        };
        auto products = [&](int st) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int u = 0; u < kT; ++u)
                    if (u < n_tiles) {
                        const double x = widen(a[st][u][e]), y = widen(b[st][u][e]);
                        acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, acc[u], 0, 0, 0);
                        sa[u] = __builtin_fma(x, x, sa[u]);
                        sb[u] = __builtin_fma(y, y, sb[u]);
                    }
        };
        const int full = dim & ~15;
#pragma unroll
        for (int st = 0; st < kStages - 1; ++st)
            if (16 * st < full) load(st, 16 * st);
        for (int k0 = 0; k0 < full; k0 += 16 * kStages) {
            if (k0 > 0 && k0 % kBlock == 0) flush(k0 == kBlock);
#pragma unroll
            for (int st = 0; st < kStages; ++st) {
                const int k = k0 + 16 * st;
                if (k >= full) break;
                const int ahead = k + 16 * (kStages - 1);
                if (ahead < full) load((st + kStages - 1) % kStages, ahead);
                products(st);
            }
        }
        if (full < dim) {
#pragma unroll
            for (int u = 0; u < kT; ++u)
                if (u < n_tiles) {
                    a[0][u] = load4_tail(pa[u], full + 4 * q, dim);
                    b[0][u] = load4_tail(pb[u], full + 4 * q, dim);
                }
            products(0);
        }
        bool near = false;
#pragma unroll
        for (int u = 0; u < kT; ++u) {
            if (u >= n_tiles) continue;
            const double ssa = sum_quarters(na[u] + sa[u]), ssb = sum_quarters(nb[u] + sb[u]);
            const double su = 1.0 / sqrt(ssa), sv = 1.0 / sqrt(ssb);
            // (not unrolled: one copy of acos keeps the registers few)
#pragma unroll 1
            for (int r = 0; r < 4; ++r) {
                const int i = q + 4 * r;
                double dot = r == 0 ? acc[u][0] : r == 1 ? acc[u][1] : r == 2 ? acc[u][2] : acc[u][3];
                if (full > kBlock) dot += *at(u, i, i16);
                // 1 / (||u|| ||v||), with one step towards the square root's reciprocal, which
                // takes away most of the norms' own roundings
                const double s0 = __shfl(su, i, dev::kWave) * sv, pp = __shfl(ssa, i, dev::kWave) * ssb;
                const double c = dot * __builtin_fma(0.5 * s0, __builtin_fma(-(pp * s0), s0, 1.0), s0);
                const bool is_near = !(fabs(c) < 1.0 - 0x1p-20);
                near = near || (is_near && want(u, i, i16));
                *at(u, i, i16) = is_near ? -1.0 : acos(c) / kPi;
            }
        }
        // the elements left at -1 (distances are >= 0), by the whole wave
        if (__any(near))
#pragma unroll 1
            for (int u = 0; u < n_tiles; ++u) {
                const T *a, *b;
                int n_r, n_c;
                ptr(u, a, n_r, b, n_c);
#pragma unroll 1
                for (int e = 0; e < n_r * n_c; ++e) {
                    const int i = e / n_c, j = e % n_c;
                    double *d = at(u, i, j);
                    if (!(*d < 0.0) || !want(u, i, j)) continue;  // wave-uniform
                    const double v = wave_near_distance(a + int64_t(i) * dim, b + int64_t(j) * dim, dim, lane);
                    if (lane == 0) *d = v;
                }
            }
    }
    return odd;
}

// A listed pair: task items x (low word) and y (high word) of one group.
struct Pair {
    int64_t x, y;
};
__device__ __forceinline__ Pair pair_of(int64_t entry) {
    return {int64_t(uint32_t(entry)), int64_t(uint64_t(entry) >> 32)};
}
struct PairSlots {
    int64_t xy, yx;
};
__device__ __forceinline__ PairSlots slots_of(const Pair &pr, const int32_t *__restrict__ item_group,
                                              const int64_t *__restrict__ g_item0,
                                              const int64_t *__restrict__ g_n,
                                              const int64_t *__restrict__ g_pair_base) {
    const int64_t g = item_group[pr.x], n = g_n[g], i0 = g_item0[g], base = g_pair_base[g];
    return {base + (pr.x - i0) * n + (pr.y - i0), base + (pr.y - i0) * n + (pr.x - i0)};
}

// Costs of both orientations and their packed path lengths, and the pair's values.
struct Costs {
    double xy, yx;
    uint32_t len;
    __device__ __forceinline__ double value_xy(int norm) const {
        return norm == FABX_NORM_PATH ? xy / double(len & 0xFFFFu) : xy;
    }
    __device__ __forceinline__ double value_yx(int norm) const {
        return norm == FABX_NORM_PATH ? yx / double(len >> 16) : yx;
    }
};
__device__ __forceinline__ void store_pair(const Pair &pr, const Costs &c, int norm,
                                           const int32_t *__restrict__ item_group,
                                           const int64_t *__restrict__ g_item0, const int64_t *__restrict__ g_n,
                                           const int64_t *__restrict__ g_pair_base, double *__restrict__ p64) {
    const PairSlots s = slots_of(pr, item_group, g_item0, g_n, g_pair_base);
    p64[s.xy] = c.value_xy(norm);
    p64[s.yx] = c.value_yx(norm);
}

// Costs of a pair by sweep_rows; odd: its tile holds a NaN (uniform over the wave).
template <typename Row16>
__device__ __forceinline__ Costs sweep_pair(const double *row, int i, int steps, int fin, bool odd) {
    Costs c{0.0, 0.0, 0};
    sweep_rows<Row16>(row, i, steps, fin, c.xy, c.len);
    c.yx = c.xy;
    if (odd) {
        uint32_t len = 0;
        sweep_rows<Row16, true>(row, i, steps, fin, c.yx, len);
        c.len = (c.len & 0xFFFFu) | (len & 0xFFFF0000u);
    }
    return c;
}

// Tiles t0, t0 + step, ... (row-major) of a pair's frame distances into dm, two
// at a time; whether this lane met a NaN.
template <typename T, bool kEuclid>
__device__ __forceinline__ bool pair_tiles(const T *__restrict__ feat, int dim, const Pair &pr, int N, int M,
                                           const int64_t *__restrict__ item_src, int t0, int step, double *dm,
                                           int ld_dm) {
    const T *fx = feat + item_src[pr.x] * int64_t(dim);
    const T *fy = feat + item_src[pr.y] * int64_t(dim);
    const int tm = (M + 15) / 16, n_tiles = (N + 15) / 16 * tm;
    bool odd = false;
#pragma unroll 1
    for (int t = t0; t < n_tiles; t += 2 * step) {
        const int ti[2] = {t / tm, (t + step) / tm}, tj[2] = {t % tm, (t + step) % tm};
        odd |= tile_distances<T, kEuclid, 2>(
            t + step < n_tiles ? 2 : 1,
            [&](int u, const T *&a, int &nr, const T *&b, int &nc) {
                a = fx + int64_t(16 * ti[u]) * dim;
                b = fy + int64_t(16 * tj[u]) * dim;
                nr = min(16, N - 16 * ti[u]);
                nc = min(16, M - 16 * tj[u]);
            },
            dim, [&](int u, int r, int c) { return dm + (16 * ti[u] + r) * ld_dm + 16 * tj[u] + c; });
    }
    return odd;
}

// Pairs of items of at most 16 frames: one tile each.  A wave takes kP pairs
// at a time: their products on the matrix cores two by two (independent
// chains), their distances into LDS, then their DTWs side by side, 16 lanes each.
// Bound by the FP64 matrix rate (a tile is a 16 x 16 x dim product: lengths of
// about 10 frames use 40% of it) and the loads from L2.  Lists too short to
// give every SIMD a wave of four pairs take one pair a wave (kP = 1), which
// ends sooner.  The XCDs take contiguous parts of the list (its pairs are
// grouped by row item, so a part's frames stay in that XCD's L2).  365,261
// marked pairs of the 100,000-item task at dim 768 (lengths 5-25): 22.1 ms with
// a block per pair and a wave per frame pair, 2.7 ms here.
constexpr int kTileLd = 17;
template <typename T, bool kEuclid, int kP>
__device__ __forceinline__ void small_pairs(const T *__restrict__ feat, int dim, int64_t e0, int64_t total,
                                            double *dm, const int64_t *__restrict__ g_item0,
                                            const int64_t *__restrict__ g_n,
                                            const int64_t *__restrict__ g_pair_base,
                                            const int64_t *__restrict__ item_src,
                                            const int32_t *__restrict__ item_len,
                                            const int32_t *__restrict__ item_group,
                                            const int64_t *__restrict__ list, int norm,
                                            double *__restrict__ p64) {
    const int lane = threadIdx.x % dev::kWave, i = lane % 16, q = lane / 16;
    const int n_pairs = int(min<int64_t>(kP, total - e0));
    // (the previous DTW's reads of dm are over: same wave, LDS in order)
    bool odd = false;
#pragma unroll 1
    for (int h = 0; h < n_pairs; h += 2)
        odd |= tile_distances<T, kEuclid, kP < 2 ? 1 : 2>(
            min(2, n_pairs - h),
            [&](int u, const T *&a, int &nr, const T *&b, int &nc) {
                const Pair pr = pair_of(list[e0 + h + u]);
                a = feat + item_src[pr.x] * int64_t(dim);
                b = feat + item_src[pr.y] * int64_t(dim);
                nr = item_len[pr.x];
                nc = item_len[pr.y];
            },
            dim, [&](int u, int r, int c) { return dm + ((h + u) * 16 + r) * kTileLd + c; });
    __builtin_amdgcn_wave_barrier();
    const int qp = min(q, n_pairs - 1);
    const Pair pr = pair_of(list[e0 + qp]);
    const int N = item_len[pr.x], M = item_len[pr.y];
    int steps = N + M - 1;
#pragma unroll
    for (int o = 32; o >= 16; o >>= 1) steps = max(steps, __shfl_xor(steps, o, dev::kWave));
    const Costs c = sweep_pair<std::true_type>(dm + (qp * 16 + i) * kTileLd, i, __builtin_amdgcn_readfirstlane(steps),
                                               N + M - 2, kEuclid && __any(odd));
    if (q == qp && i == N - 1) store_pair(pr, c, norm, item_group, g_item0, g_n, g_pair_base, p64);
    __builtin_amdgcn_wave_barrier();
}

template <typename T, bool kEuclid>
__global__ __launch_bounds__(256, 3) void k_recheck_small(const T *__restrict__ feat, int dim,
                                                          const int64_t *__restrict__ g_item0,
                                                          const int64_t *__restrict__ g_n,
                                                          const int64_t *__restrict__ g_pair_base,
                                                          const int64_t *__restrict__ item_src,
                                                          const int32_t *__restrict__ item_len,
                                                          const int32_t *__restrict__ item_group,
                                                          const int64_t *__restrict__ list,
                                                          const unsigned int *__restrict__ count,
                                                          int64_t max_count, int norm, double *__restrict__ p64) {
    constexpr int kP = 4;
    __shared__ double dm_s[4 * kP * 16 * kTileLd + 8];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / dev::kWave);
    const int64_t total = min(int64_t(*count), max_count);
    const int64_t waves = int64_t(gridDim.x / 8) * 4;  // per XCD; gridDim.x is a multiple of 8
    const int64_t first = int64_t(blockIdx.x / 8) * 4 + w;
    auto go = [&](auto p_tag) {
        constexpr int p = decltype(p_tag)::value;
        const int64_t part = ((total + 7) / 8 + p - 1) / p * p;  // pairs per XCD
        const int64_t lo = int64_t(blockIdx.x % 8) * part, hi = min(total, lo + part);
        for (int64_t e = lo + first * p; e < hi; e += waves * p)
            small_pairs<T, kEuclid, p>(feat, dim, e, hi, dm_s + w * (kP * 16 * kTileLd), g_item0, g_n, g_pair_base, item_src,
                                       item_len, item_group, list, norm, p64);
    };
    if (total >= 8 * waves * kP)
        go(std::integral_constant<int, kP>{});
    else
        go(std::integral_constant<int, 1>{});
}

// Pairs with an item of 17 to 32 frames: a wave per pair, its up to four tiles
// two at a time, then its DTW; no barriers, so the waves of a SIMD overlap one's
// products with another's sweep.  A list too short to fill the chip with waves is
// left to k_recheck_tiled, whose four waves a pair end sooner (2,664 marked pairs
// of the same task: 68 us with a wave a pair, 32 us with a block).  The 17-25
// frame pairs of that task's 365,261: 4.6 ms from LDS-staged register tiles,
// 2.2 ms with a block per pair, 1.4 ms here.
constexpr int kMidL = 32, kMidMin = 2048;
template <typename T, bool kEuclid>
__global__ __launch_bounds__(256, 3) void k_recheck_mid(const T *__restrict__ feat, int dim,
                                                        const int64_t *__restrict__ g_item0,
                                                        const int64_t *__restrict__ g_n,
                                                        const int64_t *__restrict__ g_pair_base,
                                                        const int64_t *__restrict__ item_src,
                                                        const int32_t *__restrict__ item_len,
                                                        const int32_t *__restrict__ item_group,
                                                        const int64_t *__restrict__ list,
                                                        const unsigned int *__restrict__ count,
                                                        int64_t max_count, int norm, double *__restrict__ p64) {
    constexpr int kLd = kMidL + 1;
    __shared__ double dm_s[4 * kMidL * kLd + 8 + kMidL];  // pad: idle lanes read up to 32 rows further
    const int lane = threadIdx.x % dev::kWave;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / dev::kWave);
    double *dm = dm_s + w * (kMidL * kLd);
    const int64_t total = min(int64_t(*count), max_count);
    if (total < kMidMin) return;
    const int64_t part = (total + 7) / 8, lo = int64_t(blockIdx.x % 8) * part, hi = min(total, lo + part);
    for (int64_t e = lo + int64_t(blockIdx.x / 8) * 4 + w; e < hi; e += int64_t(gridDim.x / 8) * 4) {
        const Pair pr = pair_of(list[e]);
        const int N = item_len[pr.x], M = item_len[pr.y];
        const bool odd = pair_tiles<T, kEuclid>(feat, dim, pr, N, M, item_src, 0, 1, dm, kLd);
        __builtin_amdgcn_wave_barrier();
        const Costs c = sweep_pair<std::false_type>(dm + min(lane, kMidL - 1) * kLd, lane, N + M - 1, N + M - 2,
                                                    kEuclid && __any(odd));
        if (lane == N - 1) store_pair(pr, c, norm, item_group, g_item0, g_n, g_pair_base, p64);
        __builtin_amdgcn_wave_barrier();
    }
}

// Pairs with an item of 33 to 64 frames (and a short list of the class before):
// a 256-thread block per pair, its four waves sharing the tiles; wave 0 then
// runs the DTW.  10,687 pairs of 1-60 frames at dim 512: 5.7 -> 0.73 ms (from a
// serial sum per frame pair over LDS-staged features).
template <typename T, bool kEuclid>
__global__ __launch_bounds__(256, 3) void k_recheck_tiled(const T *__restrict__ feat, int dim,
                                                          const int64_t *__restrict__ g_item0,
                                                          const int64_t *__restrict__ g_n,
                                                          const int64_t *__restrict__ g_pair_base,
                                                          const int64_t *__restrict__ item_src,
                                                          const int32_t *__restrict__ item_len,
                                                          const int32_t *__restrict__ item_group,
                                                          PairLists lists, int norm, double *__restrict__ p64) {
    constexpr int kLd = kMaxL + 1;
    __shared__ double dm[kMaxL * kLd + 8 + kMaxL];
    __shared__ int odd_s;  // the pair has a NaN distance
    if constexpr (kEuclid) {
        if (threadIdx.x == 0) odd_s = 0;
        __syncthreads();
    }
    const int lane = threadIdx.x % dev::kWave;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / dev::kWave);
    const int64_t n_mid = *lists.n_mid < kMidMin ? int64_t(*lists.n_mid) : 0;
    const int64_t total = min(int64_t(*lists.n_large), lists.cap) + n_mid;
    const int64_t part = (total + 7) / 8, lo = int64_t(blockIdx.x % 8) * part, hi = min(total, lo + part);
    for (int64_t e = lo + blockIdx.x / 8; e < hi; e += gridDim.x / 8) {
        // the large class fills its list from the end
        const Pair pr = pair_of(e < n_mid ? lists.mid[e] : lists.small_large[lists.cap - 1 - (e - n_mid)]);
        const int N = item_len[pr.x], M = item_len[pr.y];
        if (pair_tiles<T, kEuclid>(feat, dim, pr, N, M, item_src, w, 4, dm, kLd) && kEuclid) odd_s = 1;
        __syncthreads();
        if (w == 0) {
            const bool odd = kEuclid && __builtin_amdgcn_readfirstlane(odd_s) != 0;
            const Costs c = sweep_pair<std::false_type>(dm + lane * kLd, lane, N + M - 1, N + M - 2, odd);
            if (lane == N - 1) store_pair(pr, c, norm, item_group, g_item0, g_n, g_pair_base, p64);
            if (odd && lane == 0) odd_s = 0;
        }
        __syncthreads();
    }
}

// Pairs in which an item has more than kMaxL frames, each unordered pair once:
// the same arithmetic, tiled.  Rows go in chunks of 64 (lane = row), each chunk
// sweeping all M columns along anti-diagonals; a chunk hands its last row's
// costs and path lengths to the next one through LDS (`rowc`, `rowl`).  Waves
// 0..3 make the frame distances of a chunk 32 columns at a time (16 x 16 tiles,
// two per wave) into a ring of four 32-column tiles while wave 4 runs the DTW on
// the tile before: at step s lane i reads column s - i, so the steps of tile k
// (s in [32k, 32k + 32)) read tiles k - 2 .. k only, and tile k + 1 goes where
// tile k - 3 was.  Rows are the item that needs fewer chunk steps.  Bound by the
// sweep's chain of dependent FP64 steps (two blocks fit a CU by their LDS).
// 682 items of 10-200 frames in 60 groups, dim 256, 9.3e7 frame pairs: 92 ms
// (each orientation by itself, a wave per frame pair), 4.2 ms here.
// The value of pair (x, y) goes to p64, p32 and flags (0: robust, unmarked) of
// both its slots.
template <typename T, bool kEuclid>
__global__ __launch_bounds__(320, 3) void k_long_dtw(const T *__restrict__ feat, int dim,
                                                  const int64_t *__restrict__ g_item0,
                                                  const int64_t *__restrict__ g_n,
                                                  const int64_t *__restrict__ g_pair_base,
                                                  const int64_t *__restrict__ item_src,
                                                  const int32_t *__restrict__ item_len,
                                                  const int32_t *__restrict__ item_group,
                                                  const int64_t *__restrict__ list, int64_t n_list, int norm,
                                                  double *__restrict__ p64, float *__restrict__ p32,
                                                  uint8_t *__restrict__ flags) {
    constexpr int kTc = 32, kRing = 4, kLd = kRing * kTc + 1;
    __shared__ double dm[dev::kWave * kLd];        // [row of chunk][ring column]
    __shared__ double rowc[kLongMax];              // previous chunk's last row: costs
    __shared__ uint32_t rowl[kLongMax];            // and path lengths
    __shared__ int odd_s;                          // the pair has a NaN distance
    if constexpr (kEuclid) {
        if (threadIdx.x == 0) odd_s = 0;
        __syncthreads();
    }
    const int lane = threadIdx.x % dev::kWave;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / dev::kWave);
    for (int64_t e = blockIdx.x; e < n_list; e += gridDim.x) {
        Pair pr = pair_of(list[e]);
        int N = item_len[pr.x], M = item_len[pr.y];
        if ((N + 63) / 64 * (M + 63) > (M + 63) / 64 * (N + 63)) {
            const Pair sw = {pr.y, pr.x};
            pr = sw;
            const int n = N;
            N = M;
            M = n;
        }
        const T *fx = feat + item_src[pr.x] * int64_t(dim);
        const T *fy = feat + item_src[pr.y] * int64_t(dim);
        const int n_tiles = (M + kTc - 1) / kTc;
        auto sweep = [&](auto &s) {
            for (int r0 = 0; r0 < N; r0 += dev::kWave) {
                const int nr = min(dev::kWave, N - r0);
                s = {};
                int t = 0;
                const int steps = M + nr - 1;
                // tile k is made in phase k and swept in phase k + 1
                for (int k = 0; k <= n_tiles; ++k) {
                    if (w < 4) {
                        const int r = 16 * w, c0 = k * kTc;
                        if (k < n_tiles && r < nr) {
                            const int nc = min(kTc, M - c0);
                            double *out = dm + r * kLd + (k % kRing) * kTc;
                            const bool odd = tile_distances<T, kEuclid, 2, 2>(
                                nc > 16 ? 2 : 1,
                                [&](int u, const T *&a, int &na, const T *&b, int &nb) {
                                    a = fx + int64_t(r0 + r) * dim;
                                    b = fy + int64_t(c0 + 16 * u) * dim;
                                    na = min(16, nr - r);
                                    nb = min(16, nc - 16 * u);
                                },
                                dim,
                                [&](int u, int i, int j) { return out + i * kLd + 16 * u + j; });
                            if (kEuclid && odd) odd_s = 1;
                        }
                    } else if (k > 0) {
                        const int i = lane, t_end = k == n_tiles ? steps : k * kTc;
                        // four steps' distances (and the row above the chunk, lane 0's) at a time
                        auto four = [&](const double (&d)[4], const double (&ru)[4], const uint32_t (&rl)[4], int n) {
    #pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                if (q >= n) break;
                                const int j = t - i;
                                double up = shr1_cost(s.c, std::false_type{});  // lane i - 1's cost, step t - 1
                                uint32_t lup = uint32_t(shr1(0, int(s.len), std::false_type{}));
                                if (r0 > 0 && i == 0) {
                                    up = ru[q];
                                    lup = rl[q];
                                }
                                s.step(j == 0, r0 == 0 && i == 0, d[q], up, lup);
                                if (i == nr - 1 && j >= 0 && j < M) {  // this chunk's last row, for the next chunk
                                    rowc[j] = s.c;
                                    rowl[j] = s.len;
                                }
                                ++t;
                            }
                        };
                        auto fetch = [&](double (&d)[4], double (&ru)[4], uint32_t (&rl)[4], int t0) {
    #pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                d[q] = dm[i * kLd + ((t0 + q - i) & (kRing * kTc - 1))];
                                const int j = min(t0 + q, kLongMax - 1);
                                ru[q] = r0 > 0 ? rowc[j] : 0.0;
                                rl[q] = r0 > 0 ? rowl[j] : 0;
                            }
                        };
                        double d0[4], d1[4], u0[4], u1[4];
                        uint32_t l0[4], l1[4];
                        fetch(d0, u0, l0, t);
                        while (t < t_end) {
                            fetch(d1, u1, l1, t + 4);
                            four(d0, u0, l0, t_end - t);
                            if (t >= t_end) break;
                            fetch(d0, u0, l0, t + 4);
                            four(d1, u1, l1, t_end - t);
                        }
                    }
                    __syncthreads();
                }
            }
        };
        // lane (N - 1) % 64 of wave 4 ends on cell (N - 1, M - 1)
        Sweep<false> s;
        sweep(s);
        Costs c{s.c, s.c, s.len};
        if constexpr (kEuclid) {
            const bool odd = odd_s != 0;  // uniform: written before the sweep's last barrier
            __syncthreads();              // and not again before every wave has read it
            if (odd) {
                Sweep<true> t;
                sweep(t);
                c = {s.c, t.c, (s.len & 0xFFFFu) | (t.len & 0xFFFF0000u)};
                if (threadIdx.x == 0) odd_s = 0;
                __syncthreads();
            }
        }
        if (w == 4 && lane == (N - 1) % dev::kWave) {
            const PairSlots sl = slots_of(pr, item_group, g_item0, g_n, g_pair_base);
            const double vxy = c.value_xy(norm), vyx = c.value_yx(norm);
            p64[sl.xy] = vxy;
            p64[sl.yx] = vyx;
            p32[sl.xy] = float(vxy);
            p32[sl.yx] = float(vyx);
            flags[sl.xy] = flags[sl.yx] = 0;
        }
    }
}

// Pooled mode.  With few marked pairs each is done by itself from the raw frames
// (k_recheck_pooled).  From n_items / 2 marked slots on, where that would read
// the features more often than once, every item's FP64 mean is made once
// (k_mean64) and the marked pairs are taken as 16 x 16 tiles of the groups' pair
// matrices (k_pooled_tiles); the means go where the pair list was.  The host
// leaves out the second way when the means do not fit there.
__device__ __forceinline__ bool by_tiles(unsigned int n_marked, int64_t n_items, bool fits) {
    return fits && 2 * int64_t(n_marked) >= n_items;
}

// The FP64 mean of frames f[0..N) at features k.. of this thread (sequential
// sums, then one division); n_k: valid features of the four.
template <typename T>
__device__ __forceinline__ void mean4(const T *f, int N, int dim, int k, double (&m)[4]) {
    for (int e = 0; e < 4; ++e) m[e] = 0.0;
    const bool whole = k + 4 <= dim;
#pragma unroll 4
    for (int t = 0; t < N; ++t) {
        const T *row = f + int64_t(t) * dim;
        const typename Four<T>::V v = whole ? load4(row + k) : load4_tail(row, k, dim);
#pragma unroll
        for (int e = 0; e < 4; ++e) m[e] += widen(v[e]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) m[e] /= double(N);
}

// HBM-bound: one read of the features, 8 bytes a feature and item written.
template <typename T>
__global__ __launch_bounds__(256) void k_mean64(const T *__restrict__ feat, int dim,
                                                const int64_t *__restrict__ item_src,
                                                const int32_t *__restrict__ item_len, int64_t n_items,
                                                const unsigned int *__restrict__ n_marked,
                                                double *__restrict__ means) {
    if (!by_tiles(*n_marked, n_items, true)) return;
    const int lane = threadIdx.x % dev::kWave;
    for (int64_t x = int64_t(blockIdx.x) * 4 + threadIdx.x / dev::kWave; x < n_items; x += int64_t(gridDim.x) * 4) {
        const T *f = feat + item_src[x] * int64_t(dim);
        const int N = item_len[x];
        for (int k = 4 * lane; k < dim; k += 4 * dev::kWave) {
            double m[4];
            mean4(f, N, dim, k, m);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (k + e < dim) means[x * int64_t(dim) + k + e] = m[e];
        }
    }
}

// Blocks take 64 x 128 tiles of the groups' pair matrices (tile_prefix), waves 16
// rows of them, two 16 x 16 tiles of unordered pairs x < y with a marked slot at a
// time.  Bound by the FP64 matrix rate and the means' loads.  9.7e6 marked pairs
// of 87,489 items at dim 512 (lengths 1-60): 519 ms pair by pair, 2.2 ms here
// after 0.63 ms for the means.
template <bool kEuclid>
__global__ __launch_bounds__(256, 2) void k_pooled_tiles(const double *__restrict__ means, int dim,
                                                         const int64_t *__restrict__ g_item0,
                                                         const int64_t *__restrict__ g_n,
                                                         const int64_t *__restrict__ g_pair_base,
                                                         const int64_t *__restrict__ tile_prefix, int64_t n_groups,
                                                         int64_t n_tiles, int64_t n_items,
                                                         const unsigned int *__restrict__ n_marked,
                                                         const uint8_t *__restrict__ flags,
                                                         double *__restrict__ p64) {
    if (!by_tiles(*n_marked, n_items, true)) return;
    __shared__ double dm_s[4][2 * 16 * kTileLd];
    const int lane = threadIdx.x % dev::kWave, i16 = lane % 16, q = lane / 16;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / dev::kWave);
    double *dm = dm_s[w];
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int64_t g = dev::find_segment_wave(tile_prefix, n_groups, tile);
        const int64_t n = g_n[g], local = tile - tile_prefix[g], ntc = (n + 127) / 128;
        const int64_t x0 = local / ntc * 64 + 16 * w, c0 = local % ntc * 128;
        if (x0 >= n) continue;
        const double *rows = means + g_item0[g] * int64_t(dim);
        const uint8_t *fl = flags + g_pair_base[g];
        double *out = p64 + g_pair_base[g];
#pragma unroll 1
        for (int64_t y0 = c0; y0 < min(c0 + 128, n); y0 += 32) {
            if (y0 + 31 <= x0) continue;  // below the diagonal
            uint32_t mxy = 0, myx = 0;    // bit 4 u + r: this lane's element of tile u, register r is marked
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int64_t x = x0 + q + 4 * r, y = y0 + 16 * u + i16;
                    if (x < y && y < n) {
                        if (fl[x * n + y] & 2) mxy |= 1u << (4 * u + r);
                        if (fl[y * n + x] & 2) myx |= 1u << (4 * u + r);
                    }
                }
            const uint32_t m = mxy | myx;
            if (__ballot(m != 0) == 0) continue;
            tile_distances<double, kEuclid, 2, 2>(
                y0 + 16 < n ? 2 : 1,
                [&](int u, const double *&a, int &nr, const double *&b, int &nc) {
                    a = rows + x0 * dim;
                    b = rows + (y0 + 16 * u) * dim;
                    nr = int(min<int64_t>(16, n - x0));
                    nc = int(min<int64_t>(16, n - (y0 + 16 * u)));
                },
                dim, [&](int u, int r, int c) { return dm + (16 * u + r) * kTileLd + c; },
                [&](int u, int r, int c) { return x0 + r < y0 + 16 * u + c; });
            __builtin_amdgcn_wave_barrier();
            for (uint32_t b = m; b; b &= b - 1) {
                const int k = __builtin_ctz(b), u = k / 4, i = q + 4 * (k % 4);
                const int64_t x = x0 + i, y = y0 + 16 * u + i16;
                const double d = dm[(16 * u + i) * kTileLd + i16];
                if ((mxy >> k) & 1u) out[x * n + y] = d;
                if ((myx >> k) & 1u) out[y * n + x] = d;
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// One block per listed pair: the two items' mean frames (threads over the
// features), then wave 0 takes their norms and cosine and, near +-1, the
// half-chord sums, its lanes splitting the dimension.
template <typename T>
__global__ __launch_bounds__(256) void k_recheck_pooled(const T *__restrict__ feat, int dim,
                                                        const int64_t *__restrict__ g_item0,
                                                        const int64_t *__restrict__ g_n,
                                                        const int64_t *__restrict__ g_pair_base,
                                                        const int64_t *__restrict__ item_src,
                                                        const int32_t *__restrict__ item_len,
                                                        const int32_t *__restrict__ item_group,
                                                        const int64_t *__restrict__ list, int64_t cap,
                                                        const unsigned int *__restrict__ count, int64_t n_items,
                                                        const unsigned int *__restrict__ n_marked, int tiles_fit,
                                                        int euclid, double *__restrict__ p64) {
    if (by_tiles(*n_marked, n_items, tiles_fit != 0)) return;
    __shared__ double mx[2048];
    __shared__ double my[2048];
    const int lane = threadIdx.x % dev::kWave;
    const int64_t total = min(int64_t(*count), cap);
    for (int64_t e = blockIdx.x; e < total; e += gridDim.x) {
        const Pair pr = pair_of(list[e]);
        const int N = item_len[pr.x], M = item_len[pr.y];
        const T *fx = feat + item_src[pr.x] * int64_t(dim);
        const T *fy = feat + item_src[pr.y] * int64_t(dim);
        const int n4 = (dim + 3) / 4;
        for (int t = threadIdx.x; t < 2 * n4; t += blockDim.x) {
            const bool second = t >= n4;
            const int k = 4 * (second ? t - n4 : t);
            double m[4];
            mean4(second ? fy : fx, second ? M : N, dim, k, m);
#pragma unroll
            for (int f = 0; f < 4; ++f)
                if (k + f < dim) (second ? my : mx)[k + f] = m[f];
        }
        __syncthreads();
        if (threadIdx.x < dev::kWave) {
            double d;
            if (euclid) {
                double sd = 0.0;
                for (int k = lane; k < dim; k += dev::kWave) sd += (mx[k] - my[k]) * (mx[k] - my[k]);
                d = sqrt(wave_sum_f64(sd));
            } else {
                double sx = 0.0, sy = 0.0;
                for (int k = lane; k < dim; k += dev::kWave) {
                    sx += mx[k] * mx[k];
                    sy += my[k] * my[k];
                }
                const double ix = 1.0 / sqrt(wave_sum_f64(sx)), iy = 1.0 / sqrt(wave_sum_f64(sy));
                double c = 0.0;
                for (int k = lane; k < dim; k += dev::kWave) c += (mx[k] * ix) * (my[k] * iy);
                c = wave_sum_f64(c);
                if (fabs(c) < 1.0 - 0x1p-20) {
                    d = acos(c) / kPi;
                } else {
                    double sm = 0.0, sp = 0.0;
                    for (int k = lane; k < dim; k += dev::kWave) {
                        const double a = mx[k] * ix, b = my[k] * iy;
                        sm += (a - b) * (a - b);
                        sp += (a + b) * (a + b);
                    }
                    d = near_angle_over_pi(wave_sum_f64(sm), wave_sum_f64(sp));
                }
            }
            if (lane == 0) {
                const PairSlots s = slots_of(pr, item_group, g_item0, g_n, g_pair_base);
                p64[s.xy] = d;
                p64[s.yx] = d;
            }
        }
        __syncthreads();
    }
}

}  // namespace

// Calls go(typed features, euclid tag) for the dataset's type and distance.
template <typename Go>
static void typed(const void *features, int dtype, int euclid, Go &&go) {
    if (dtype == FABX_DTYPE_F32) {
        const float *f = static_cast<const float *>(features);
        euclid ? go(f, std::true_type{}) : go(f, std::false_type{});
    } else {
        const uint16_t *f = static_cast<const uint16_t *>(features);
        euclid ? go(f, std::true_type{}) : go(f, std::false_type{});
    }
}

void long_dtw(hipStream_t s, const void *features, int dtype, int dim, const GroupTables &g,
              const ItemTables &it, const int32_t *item_group, const int64_t *list, int64_t n_list, int norm,
              int euclid, double *p64, float *p32, uint8_t *flags) {
    if (n_list <= 0) return;
    const unsigned blocks = unsigned(std::min<int64_t>(n_list, 4096));
    typed(features, dtype, euclid, [&](auto *f, auto eu) {
        using T = std::remove_const_t<std::remove_pointer_t<decltype(f)>>;
        hipLaunchKernelGGL((k_long_dtw<T, decltype(eu)::value>), dim3(blocks), dim3(320), 0, s, f, dim,
                           g.item0, g.n_items, g.pair_base, it.src, it.len,
                           item_group, list, n_list, norm, p64, p32, flags);
    });
    FABX_HIP(hipGetLastError());
}

void recheck_dtw(hipStream_t s, const void *features, int dtype, int dim, const GroupTables &g,
                 const ItemTables &it, const int32_t *item_group, const PairLists &lists, int n_cu, int max_len,
                 int norm, int euclid, double *p64) {
    const int64_t cap = lists.cap;
    if (cap <= 0) return;
    // three blocks of four waves per CU (their registers), or fewer when the list cannot fill them
    const int64_t per_xcd = std::max(1, 3 * n_cu / 8);
    const unsigned small = 8u * unsigned(std::max<int64_t>(1, std::min<int64_t>(per_xcd, (cap + 31) / 32)));
    const unsigned mid = small;
    const unsigned tiled = 8u * unsigned(std::max<int64_t>(1, std::min<int64_t>(per_xcd, (cap + 7) / 8)));
    typed(features, dtype, euclid, [&](auto *f, auto eu) {
        using T = std::remove_const_t<std::remove_pointer_t<decltype(f)>>;
        hipLaunchKernelGGL((k_recheck_small<T, decltype(eu)::value>), dim3(small), dim3(256), 0, s, f, dim, g.item0,
                           g.n_items, g.pair_base, it.src, it.len, item_group, lists.small_large, lists.n_small, cap,
                           norm, p64);
        if (max_len > 16 && cap >= kMidMin)
            hipLaunchKernelGGL((k_recheck_mid<T, decltype(eu)::value>), dim3(mid), dim3(256), 0, s, f, dim, g.item0,
                               g.n_items, g.pair_base, it.src, it.len, item_group, lists.mid, lists.n_mid, cap, norm,
                               p64);
        if (max_len > 16)
            hipLaunchKernelGGL((k_recheck_tiled<T, decltype(eu)::value>), dim3(tiled), dim3(256), 0, s, f, dim,
                               g.item0, g.n_items, g.pair_base, it.src, it.len, item_group, lists, norm, p64);
    });
    FABX_HIP(hipGetLastError());
}

void recheck_pooled(hipStream_t s, const void *features, int dtype, int dim, const GroupTables &g,
                    const ItemTables &it, const int32_t *item_group, const PairLists &lists, double *means,
                    const int64_t *tile_prefix, int64_t n_tiles, const uint8_t *flags, int euclid, double *p64) {
    if (lists.cap <= 0) return;
    if (dim > 2048) fail(FABX_EINVAL, "pooled recheck supports dim <= 2048");
    const unsigned blocks = unsigned(std::min<int64_t>(lists.cap, 4096));
    typed(features, dtype, euclid, [&](auto *f, auto) {
        using T = std::remove_const_t<std::remove_pointer_t<decltype(f)>>;
        hipLaunchKernelGGL(k_recheck_pooled<T>, dim3(blocks), dim3(256), 0, s, f, dim, g.item0, g.n_items,
                           g.pair_base, it.src, it.len, item_group, lists.small_large, lists.cap, lists.n_small,
                           it.n_items, lists.n_marked, means ? 1 : 0, euclid, p64);
        if (means)
            hipLaunchKernelGGL(k_mean64<T>, dim3(grid_for(it.n_items, 4)), dim3(256), 0, s, f, dim, it.src, it.len,
                               it.n_items, lists.n_marked, means);
    });
    if (means)
        hipLaunchKernelGGL(euclid ? k_pooled_tiles<true> : k_pooled_tiles<false>, dim3(grid_for(n_tiles, 1)),
                           dim3(256), 0, s, means, dim, g.item0, g.n_items, g.pair_base, tile_prefix, g.n_groups,
                           n_tiles, it.n_items, lists.n_marked, flags, p64);
    FABX_HIP(hipGetLastError());
}

}  // namespace kern
}  // namespace fabx
