// Plain FP32 form (and discrete units), DTW mode, items of at most 64 frames:
// frame distances and DTW in one kernel, each unordered item pair once.  Every
// value equals bit for bit what the strip form (k_plain.hip: distance matrix in
// HBM, one wave per ordered pair), which longer items still take, gives it:
//
//  - the Gram products run on v_mfma_f32_32x32x2_f32, whose accumulation is
//    the same chain of fused multiply-adds over the features in order as the
//    strip form's vector code (measured: 0 of 1024 sums of 768 terms differ);
//    the Euclidean sums stay on the vector ALUs in the same order;
//  - frame distances and DTW costs do not depend on a pair's orientation, only
//    the predecessor chosen among equal ones does: the path lengths of both
//    orientations go along (low half: (x, y), diagonal before left before up;
//    high half: (y, x), whose left is this one's up), and (y, x) gets its own
//    quotient;
//  - a unit with a distance that is not finite (features with infinities or
//    NaN), where the order of comparisons shows in the costs as well, sweeps
//    each orientation by itself with the strip form's comparisons.
//
// Work units, blocks and the DTW's lane layout are those of the BF16 form
// (k_fused.hip): a row block of at most 64 frames against a column block of at
// most 128, lane = frame row, each of four waves streaming its share of the
// column items past all rows.
#include "device_common.h"
#include "fused_unit.h"
#include "kernels.h"

namespace fabx {
namespace kern {
namespace {

using dev::kInf;
using dev::kWave;

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kRows = 64, kCols = kFusedColFrames;
constexpr int kAngular = 0, kEuclid = 1, kUnits = 2;
constexpr int kDStride = kCols + 2;                           // LDS distance tile stride
constexpr int kTileFloats = kRows * kDStride + kWave + 4;     // with the sweep's tail guard
constexpr int kFlagLen = kWave + kCols + kWave + 8;           // column flags between zero guards
// angular staging: K chunks of 32 features; each 8 of a row lie as k 0 2 4 6, 1 3 5 7,
// so that a lane (half-wave h takes features of parity h) reads four steps' operands
// at once; rows of 36 floats keep those reads off each other's banks
constexpr int kKc = 32, kStageLd = kKc + 4;
// Euclidean staging: K chunks of 16 features, feature-major
constexpr int kKe = 16, kRowLd = kRows + 4, kColLd = kCols + 4;

__device__ __forceinline__ float shr1(float v) {  // lane - 1's value (lane 0 reads 0)
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ uint32_t shr1(uint32_t v) {
    return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x138, 0xf, 0xf, true));
}

// 64 x 128 frame distances (theta / pi) of packed unit rows r0.. and c0.. into
// dt.  Rows past nr and nc repeat the last.
__device__ __forceinline__ void angular_tile(float *smem, const float *__restrict__ xn, int dim_pad, int64_t r0,
                                             int nr, int64_t c0, int nc, int c_lo, float *dt) {
    const int lane = threadIdx.x % kWave, w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    constexpr int kPer = (kRows + kCols) * (kKc / 8) / 256;  // 8-feature pieces per thread
    f32x4 lo[kPer], hi[kPer];
    auto load = [&](int k0) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int p = threadIdx.x + 256 * i, r = p / (kKc / 8), q = p % (kKc / 8);
            const int64_t row = r < kRows ? r0 + min(r, nr - 1) : c0 + min(r - kRows, nc - 1);
            const f32x4 *s = reinterpret_cast<const f32x4 *>(xn + row * dim_pad + k0 + 8 * q);
            lo[i] = s[0];
            hi[i] = s[1];
        }
    };
    f32x16 acc[2];
#pragma unroll
    for (int i = 0; i < 16; ++i) { acc[0][i] = 0.0f; acc[1][i] = 0.0f; }
    const int col0 = 32 * w, half = lane / 32;
    const bool mine = col0 < nc && col0 + 32 > c_lo, low = nr > 32;
    load(0);
    // (a loop for each of the two cases: a branch per product puts every read from LDS,
    // and its wait, right before its product; 60k items of 9 frames, 768 features, with
    // the DTW: 1.45 -> 1.25 ms)
    auto products = [&](auto low_tag) {
        constexpr bool kLow = decltype(low_tag)::value;
        for (int k0 = 0; k0 < dim_pad; k0 += kKc) {
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                const int p = threadIdx.x + 256 * i;
                f32x4 *d = reinterpret_cast<f32x4 *>(smem + p / (kKc / 8) * kStageLd + p % (kKc / 8) * 8);
                d[0] = f32x4{lo[i][0], lo[i][2], hi[i][0], hi[i][2]};
                d[1] = f32x4{lo[i][1], lo[i][3], hi[i][1], hi[i][3]};
            }
            __syncthreads();
            if (k0 + kKc < dim_pad) load(k0 + kKc);
            if (mine)
#pragma unroll
                for (int j = 0; j < kKc / 8; ++j) {
                    const float *at = smem + (lane % 32) * kStageLd + 8 * j + 4 * half;
                    const f32x4 a0 = *reinterpret_cast<const f32x4 *>(at);
                    const f32x4 b = *reinterpret_cast<const f32x4 *>(at + (kRows + col0) * kStageLd);
                    f32x4 a1;
                    if (kLow) a1 = *reinterpret_cast<const f32x4 *>(at + 32 * kStageLd);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0[e], b[e], acc[0], 0, 0, 0);
                        if (kLow) acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[e], b[e], acc[1], 0, 0, 0);
                    }
                }
            __syncthreads();
        }
    };
    if (low) products(std::true_type{});
    else products(std::false_type{});
    if (!mine) return;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (h == 1 && !low) break;
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
            if (32 * h + 8 * g4 >= nr) break;
#pragma unroll
            for (int i = 4 * g4; i < 4 * g4 + 4; ++i) {
                const int r = 32 * h + 8 * g4 + 4 * half + i % 4;
                const float cs = fminf(fmaxf(acc[h][i], -1.0f), 1.0f);
                // (the clamp drops a NaN sum, as the strip form's does: always finite)
                dt[r * kDStride + col0 + lane % 32] = acosf(cs) * dev::kInvPi;
            }
        }
    }
}

// The same of raw rows' Euclidean distances: 4 x 8 elements a thread; odd collects
// the largest bit pattern.
__device__ __forceinline__ void euclid_tile(float *smem, const float *__restrict__ xn, int dim_pad, int64_t r0,
                                            int nr, int64_t c0, int nc, float *dt, uint32_t &odd) {
    const int ty = threadIdx.x / 16, tx = threadIdx.x % 16;
    float *As = smem, *Bs = smem + kKe * kRowLd;
    constexpr int kPer = (kRows + kCols) * (kKe / 4) / 256;
    float acc[4][8] = {};
    f32x4 v[kPer];
    auto load = [&](int k0) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int p = threadIdx.x + 256 * i, r = p / (kKe / 4), q = p % (kKe / 4);
            const int64_t row = r < kRows ? r0 + min(r, nr - 1) : c0 + min(r - kRows, nc - 1);
            v[i] = *reinterpret_cast<const f32x4 *>(xn + row * dim_pad + k0 + 4 * q);
        }
    };
    load(0);
    for (int k0 = 0; k0 < dim_pad; k0 += kKe) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int p = threadIdx.x + 256 * i, r = p / (kKe / 4), q = p % (kKe / 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (r < kRows) As[(4 * q + e) * kRowLd + r] = v[i][e];
                else Bs[(4 * q + e) * kColLd + r - kRows] = v[i][e];
            }
        }
        __syncthreads();
        if (k0 + kKe < dim_pad) load(k0 + kKe);
#pragma unroll
        for (int k = 0; k < kKe; ++k) {
            const f32x4 av = *reinterpret_cast<const f32x4 *>(As + k * kRowLd + 4 * ty);
            const f32x4 b0 = *reinterpret_cast<const f32x4 *>(Bs + k * kColLd + 8 * tx);
            const f32x4 b1 = *reinterpret_cast<const f32x4 *>(Bs + k * kColLd + 8 * tx + 4);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float d = av[i] - (j < 4 ? b0[j % 4] : b1[j % 4]);
                    acc[i][j] = fmaf(d, d, acc[i][j]);
                }
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float d = __builtin_sqrtf(acc[i][j]);
            if (4 * ty + i < nr && 8 * tx + j < nc) odd = max(odd, __float_as_uint(d) & 0x7FFFFFFFu);
            dt[(4 * ty + i) * kDStride + 8 * tx + j] = d;
        }
}

template <int kKind, bool kPath>
__global__ __launch_bounds__(256, 4) void k_plain_fused(const void *__restrict__ packed, int dim_pad,
                                                        const int64_t *__restrict__ g_item0,
                                                        const int64_t *__restrict__ g_n,
                                                        const int64_t *__restrict__ g_pair_base,
                                                        const int32_t *__restrict__ item_len,
                                                        const int64_t *__restrict__ item_dst,
                                                        const int32_t *__restrict__ order, FusedPlan plan,
                                                        int64_t grid_q, float *__restrict__ p32) {
    constexpr int kStage = kKind == kAngular ? (kRows + kCols) * kStageLd
                           : kKind == kEuclid ? kKe * (kRowLd + kColLd)
                                              : kRows + kCols;
    __shared__ __attribute__((aligned(16))) float smem[kStage > kTileFloats ? kStage : kTileFloats];
    __shared__ uint32_t colflag[4][kFlagLen];
    __shared__ uint32_t odd_s;
    __shared__ unit::Items<kCols> items_s;  // where the unit's items begin and end
    float *dt = smem;
    const int lane = threadIdx.x % kWave, w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    colflag[w][lane] = 0;  // the guard before every span
    // XCD x takes the contiguous unit range [x * grid_q, (x + 1) * grid_q), as the BF16 kernel
    const int64_t xcd = blockIdx.x % 8, n_m = gridDim.x / 8;
    for (int64_t j = blockIdx.x / 8; j < grid_q; j += n_m) {
        const int64_t u = xcd * grid_q + j;
        if (u >= plan.n_units) break;  // uniform; later units are larger
        const int64_t bi = dev::find_segment_wave(plan.unit_prefix, plan.n_bands, u);
        const int rb0 = plan.band_rb[bi], band_rows = plan.band_rb[bi + 1] - rb0;
        const int64_t local = u - plan.unit_prefix[bi];
        const int64_t rbi = rb0 + local % band_rows;
        const int c_local = plan.rb_cstart[rb0] + int(local / band_rows);
        if (c_local < plan.rb_cstart[rbi]) continue;  // uniform: wholly below the group's diagonal
        const int64_t g = plan.rb[4 * rbi];
        const int cbi = plan.g_cb0[g] + c_local;
        const int r_item0 = plan.rb[4 * rbi + 1], r_nitems = plan.rb[4 * rbi + 2], r_frames = plan.rb[4 * rbi + 3];
        const int c_item0 = plan.cb[4 * cbi + 1], c_nitems = plan.cb[4 * cbi + 2], c_frames = plan.cb[4 * cbi + 3];
        const int64_t r0 = item_dst[r_item0], c0 = item_dst[c_item0];
        const int64_t pbase = g_pair_base[g], gn = g_n[g], gitem0 = g_item0[g];
        // columns before the row block's first item belong to other units
        const int c_skip = int(min(max(r0 - c0, int64_t(0)), int64_t(c_frames)));
        unit::find_items<kCols>(items_s, item_len, r_item0, r_nitems, c_item0, c_nitems);
        if (threadIdx.x == 0) odd_s = 0;

        [[maybe_unused]] uint32_t odd = 0;  // the largest distance's bits
        if constexpr (kKind == kAngular) {
            angular_tile(smem, static_cast<const float *>(packed), dim_pad, r0, r_frames, c0, c_frames, c_skip,
                         dt);
        } else if constexpr (kKind == kEuclid) {
            euclid_tile(smem, static_cast<const float *>(packed), dim_pad, r0, r_frames, c0, c_frames, dt, odd);
        } else {
            const int32_t *codes = static_cast<const int32_t *>(packed);
            int rc[kRows / 4], cc[2];  // rows w, w + 4, ...; columns lane, lane + 64
#pragma unroll
            for (int i = 0; i < 2; ++i) cc[i] = codes[c0 + min(lane + 64 * i, c_frames - 1)];
#pragma unroll
            for (int i = 0; i < kRows / 4; ++i) rc[i] = codes[r0 + min(w + 4 * i, r_frames - 1)];
#pragma unroll
            for (int i = 0; i < kRows / 4; ++i)
#pragma unroll
                for (int c = 0; c < 2; ++c) dt[(w + 4 * i) * kDStride + lane + 64 * c] = rc[i] != cc[c] ? 1.0f : 0.0f;
        }
        if (kKind == kEuclid && __ballot(odd >= 0x7F800000u) != 0 && lane == 0) atomicOr(&odd_s, 1u);

        if constexpr (kKind == kUnits) __syncthreads();  // the masks (the other forms' tiles have barriers)
        // the row item of lane `lane`, this wave's columns and their flags between
        // zero guards
        const unit::Row row = unit::row_of(items_s, lane, r_frames);
        const int ir = row.ir;
        const int max_n = __builtin_amdgcn_readfirstlane(int(items_s.longest));
        const unit::Cols<kCols> cols(items_s);
        const unit::Span span = unit::span_of<kCols>(cols, w, c_skip, c_frames);
        const int s_begin = span.begin, s_end = span.end;
        if (s_end > s_begin) {
            const int n = s_end - s_begin;
            for (int c = lane; c < n; c += kWave) colflag[w][kWave + c] = cols.flag(s_begin + c, c_frames);
            for (int c = n + lane; c < n + kWave + 8; c += kWave) colflag[w][kWave + c] = 0;
        }
        __syncthreads();
        const int S = s_end - s_begin;
        // kBoth: one sweep for both orientations; kXY, kYX: one orientation with the
        // strip form's comparisons
        constexpr int kBoth = 0, kXY = 1, kYX = 2;
        const bool odd_unit = kKind == kEuclid && odd_s != 0;  // uniform
        // A pair's end: its cost replaces the distance there in the tile, its path
        // lengths the distance above (both already read; in an item of one row the only
        // path has the column item's length, and the cost overwrites the lengths).
        auto sweep = [&](auto mode_tag) {
            constexpr int mode = decltype(mode_tag)::value;
            const bool top = ir == 0;
            const float diag_first = top ? 0.0f : kInf;  // virtual cell (-1, -1)
            const float top_pen = top ? kInf : 0.0f;
            uint32_t not_top = top ? 0u : ~0u;
            asm("" : "+v"(not_top));  // (a mask, not a selection: one instruction with the shift)
            float *cost_at = dt + lane * kDStride + s_begin - ir;
            uint32_t *len_at = reinterpret_cast<uint32_t *>(cost_at - (top ? 0 : kDStride));
            const float *dcol = cost_at;
            const uint32_t *fcol = &colflag[w][kWave - ir];
            const uint32_t out_min = row.last ? 0x80000000u : 0xFFFFFFFFu;
            const int steps = S + max_n - 1;
            float c = kInf, up_prev = kInf;
            uint32_t L = 0, lup_prev = 0;
            auto step = [&](const uint32_t cf, const float dv) {
                const bool first = uint8_t(cf) != 0;
                // a first row has no row above.  kBoth: the lane above may hold a NaN then
                // (it is outside its columns), so up is only asked whether it is less, and
                // fminf drops it
                float up = shr1(c);
                if (mode == kBoth) up += top_pen;
                else up = top ? kInf : up;
                const float diag = first ? diag_first : up_prev, left = first ? kInf : c;
                const bool le = !(up < left), ge = up <= left;
                const bool from_diag = diag <= left && (mode == kBoth ? !(up < diag) : diag <= up);
                up_prev = up;
                if (kPath) {
                    const uint32_t lup = shr1(L) & not_top;
                    uint32_t sel;
                    if (mode == kBoth) {
                        const uint32_t lo = le ? L : lup, hi = ge ? lup : L;
                        sel = (hi & 0xFFFF0000u) | (lo & 0xFFFFu);
                    } else {
                        sel = (mode == kXY ? left <= up : !ge) ? L : lup;
                    }
                    L = (from_diag ? lup_prev : sel) + 0x00010001u;
                    lup_prev = lup;
                }
                float best;
                if (mode == kBoth) best = fminf(fminf(diag, left), up);
                else best = from_diag ? diag : (mode == kXY ? left <= up : !ge) ? left : up;
                c = dv + best;
            };
            // four steps at a time from one of two register buffers while the other
            // takes the next four
            auto load4 = [&](uint32_t (&f)[4], float (&d)[4], int t0) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    f[k] = fcol[t0 + k];
                    d[k] = dcol[t0 + k];
                }
            };
            auto run_n = [&](const uint32_t (&f)[4], const float (&d)[4], int t0, auto n_tag) {
                constexpr int N = decltype(n_tag)::value;
                float cs[N];
                uint32_t ls[N], top_f = f[0];
#pragma unroll
                for (int k = 0; k < N; ++k) {
                    top_f = max(top_f, f[k]);
                    step(f[k], d[k]);
                    cs[k] = c;
                    ls[k] = L;
                }
                if (top_f >= out_min) {
#pragma unroll
                    for (int k = 0; k < N; ++k)
                        if (f[k] >= out_min) {
                            if (kPath) len_at[t0 + k] = ls[k];
                            cost_at[t0 + k] = cs[k];
                        }
                }
            };
            uint32_t fa[4], fb[4];
            float da[4], db[4];
            load4(fa, da, 0);
            auto rest = [&](const uint32_t (&f)[4], const float (&d)[4], int t0, int n) {  // uniform n
                if (n >= 4) run_n(f, d, t0, std::integral_constant<int, 4>{});
                else if (n == 3) run_n(f, d, t0, std::integral_constant<int, 3>{});
                else if (n == 2) run_n(f, d, t0, std::integral_constant<int, 2>{});
                else run_n(f, d, t0, std::integral_constant<int, 1>{});
            };
            int t = 0;
            for (; t + 8 <= steps; t += 8) {
                load4(fb, db, t + 4);
                run_n(fa, da, t, std::integral_constant<int, 4>{});
                load4(fa, da, t + 8);
                run_n(fb, db, t + 4, std::integral_constant<int, 4>{});
            }
            if (t < steps) {
                load4(fb, db, t + 4);
                rest(fa, da, t, steps - t);
                if (t + 4 < steps) rest(fb, db, t + 4, steps - t - 4);
            }
        };
        // the pairs of the wave's columns, a lane each: mode kBoth both slots, kXY / kYX
        // its own
        auto write = [&](auto mode_tag) {
            constexpr int mode = decltype(mode_tag)::value;
            __builtin_amdgcn_wave_barrier();
            unit::for_pairs<kCols>(cols, span, r_nitems, r_item0, c_item0, gitem0, order,
                                   [&](int i, int j, int64_t px, int64_t py, bool same) {
                const int r = items_s.row_last[i], col = items_s.col_last[j];
                const float cost = dt[r * kDStride + col];
                uint32_t len = 0;
                if (kPath) {
                    const int first_r = i > 0 ? items_s.row_last[i - 1] + 1 : 0;
                    const int first_c = j > 0 ? items_s.col_last[j - 1] + 1 : 0;
                    len = r == first_r ? uint32_t(col - first_c + 1) * 0x00010001u
                                       : __float_as_uint(dt[(r - 1) * kDStride + col]);
                }
                auto quotient = [&](uint32_t n) {
                    if (!kPath) return cost;
                    // integer costs: the double quotient rounded once (equal fractions give
                    // equal values)
                    if (kKind == kUnits) return float(double(cost) / double(n));
                    return cost / float(n);
                };
                if (mode != kYX) p32[pbase + px * gn + py] = quotient(len & 0xFFFFu);
                if (mode != kXY && !same) p32[pbase + py * gn + px] = quotient(len >> 16);
            });
        };
        auto sweep_and_write = [&](auto mode_tag) {
            if (S <= 0) return;
            sweep(mode_tag);
            write(mode_tag);
        };
        if (!odd_unit) {
            sweep_and_write(std::integral_constant<int, kBoth>{});
        } else if constexpr (kKind == kEuclid) {
            // each orientation by itself; the tile again for the second, since the ends of
            // pairs overwrote distances
            sweep_and_write(std::integral_constant<int, kXY>{});
            __syncthreads();
            euclid_tile(smem, static_cast<const float *>(packed), dim_pad, r0, r_frames, c0, c_frames, dt, odd);
            __syncthreads();
            sweep_and_write(std::integral_constant<int, kYX>{});
        }
        __syncthreads();  // the next unit overwrites the tile and the flags
    }
}

}  // namespace

void plain_fused(hipStream_t s, const void *packed, int dim_pad, const GroupTables &g, const ItemTables &it,
                 const FusedPlan &plan, int distance, int norm, float *p32) {
    if (plan.n_units <= 0) return;
    if (plan.cols != kCols) fail(FABX_EINVAL, "the plain fused kernel takes column blocks of 128 frames");
    if (distance != FABX_DISTANCE_UNITS && dim_pad % kKc) fail(FABX_EINVAL, "padded dim must be a multiple of 32");
    const int64_t q = (plan.n_units + 7) / 8;
    const dim3 grid(unsigned(8 * std::min<int64_t>(q, dev::kMaxBlocks / 8))), block(256);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, 0, s, packed, dim_pad, g.item0, g.n_items, g.pair_base, it.len, it.dst,
                           it.order, plan, q, p32);
    };
    const bool path = norm == FABX_NORM_PATH;
    if (distance == FABX_DISTANCE_UNITS)
        path ? go(k_plain_fused<kUnits, true>) : go(k_plain_fused<kUnits, false>);
    else if (distance == FABX_DISTANCE_EUCLIDEAN)
        path ? go(k_plain_fused<kEuclid, true>) : go(k_plain_fused<kEuclid, false>);
    else
        path ? go(k_plain_fused<kAngular, true>) : go(k_plain_fused<kAngular, false>);
    FABX_HIP(hipGetLastError());
}

}  // namespace kern
}  // namespace fabx
