// Triplet comparison and per-cell reduction (cell discriminability formula of
// the Background section), in integer half units: each triple adds
// 2 [d(x,a) < d(x,b)] + [d(x,a) == d(x,b)].
//
// Work unit = (cell, range of x).  Both distances come from the row of x in the
// group's pair matrix (a few hundred bytes, in L1/L2).  A row with a near tie or
// a non-robust pair is left to the FP64 recount; the other rows' counts stay in
// the lanes, are reduced once per unit and added with one 64-bit atomic, so the
// result does not depend on scheduling.
#include "device_common.h"
#include "kernels.h"

namespace fabx {
namespace kern {
namespace {

using dev::kWave;

constexpr uint8_t kNonRobust = 1;
constexpr uint8_t kMarked = 2;

// A unit by a wave.  |A| x |B| of at most a wave's lanes: as many whole rows x as
// fit, a lane each comparison.  Otherwise the larger of A and B lies in the lanes (as
// many rows side by side as fit), and the other one's values pass by, one per step,
// so a row's values and flags are read once and a step is a lane shuffle and three
// comparisons; a row whose grid was walked in passes of 64 read four values per
// comparison and waited for them.  (Passing values for small rows too made 131,671
// cells of well separated labels take 113 us instead of 86; with the grid 82.)
//  kMany = false: a wave takes one unit at a time (at most 16 passes over rows, see
//    unit_rows()); below 4096 units each is split by x into four, where a few large
//    ones would otherwise end last (957 uneven cells 26 -> 13 us, 3635 31 -> 15; 760
//    even ones 12 -> 14, 4000 even ones 11 -> 18).  At most 12,288 blocks: a block
//    costs its tables' latency and an atomic for its recount rows (131,671 cells 96, 87
//    and 88 us with 8192, 12,288 and 16,384 blocks; 60,000 cells of 2 x 2 items 25, 28
//    and 30; 40,000 such cells with 18,475 recount rows 93, 106 and 106).
//  kMany = true, from kManyUnits units on (tasks across speakers have millions of
//    cells of a few triples, and a wave per unit spent its time on the unit's tables
//    and its reduction): a wave takes `chunk` consecutive units, one per lane; those
//    of at most kLaneWork comparisons are done by their lane alone, the others by
//    the wave one after another.  (1.77e6 cells across speakers 0.52 -> 0.15 ms, 863,150
//    such cells 0.25 -> 0.07; but 960,000 cells of 27 comparisons, just past kLaneWork,
//    0.32 -> 0.35, and 131,671 cells of uneven sizes 0.09 -> 0.18 with 4 units a wave,
//    0.59 with 16, whose larger units queue in a few waves.)
// Rows for the recount are collected in LDS and leave 128 at a time, or with one
// atomic of the block at its end: one atomic per row on the common counter was
// most of the time where many rows go there.
// Bound by the latency of the chain unit, cell, row values.  100,000 items with
// 126,303 rows for the recount: 1.27 -> 0.14 ms (0.086 -> 0.082 without such rows).
constexpr int kLaneWork = 24, kRowBuf = 128;
constexpr int64_t kManyUnits = 16 * 32768;

template <bool kMany>
__global__ __launch_bounds__(256) void k_triplets(const CellDev *__restrict__ cells,
                                                  const int32_t *__restrict__ units, int64_t n_units, int chunk,
                                                  int log_parts, const int64_t *__restrict__ g_pair_base,
                                                  const int64_t *__restrict__ g_n,
                                                  const float *__restrict__ p32,
                                                  unsigned long long *__restrict__ W,
                                                  uint8_t *flags, float margin,
                                                  int32_t *__restrict__ recount,
                                                  unsigned int *__restrict__ recount_n,
                                                  int64_t recount_cap,
                                                  const unsigned int *__restrict__ scale) {
    __shared__ int2 rowbuf_s[4][kRowBuf];
    const int lane = threadIdx.x % kWave;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (scale) margin *= __uint_as_float(*scale);  // margin in units of the largest frame length
    int2 *rowbuf = rowbuf_s[wv];
    int n_rows = 0;  // wave-uniform
    auto write_rows = [&](unsigned int at) {
        for (int i = lane; i < n_rows; i += kWave) {
            const int64_t k = int64_t(at) + i;
            if (k < recount_cap) {
                recount[2 * k] = rowbuf[i].x;
                recount[2 * k + 1] = rowbuf[i].y;
            }
        }
    };
    auto flush = [&] {
        unsigned int at = 0;
        if (lane == 0) at = atomicAdd(recount_n, unsigned(n_rows));
        write_rows(__shfl(at, 0, kWave));
        __builtin_amdgcn_wave_barrier();
        n_rows = 0;
    };
    // the block's last rows, with one atomic (every wave comes here)
    auto flush_block = [&] {
        __shared__ unsigned int n_s[4], at_s;
        if (!flags) return;
        if (lane == 0) n_s[wv] = unsigned(n_rows);
        __syncthreads();
        const unsigned int total = n_s[0] + n_s[1] + n_s[2] + n_s[3];
        if (total == 0) return;
        if (threadIdx.x == 0) at_s = atomicAdd(recount_n, total);
        __syncthreads();
        unsigned int at = at_s;
        for (int k = 0; k < wv; ++k) at += n_s[k];
        write_rows(at);
    };
    // row (cell, x) of each lane with p set (all lanes call)
    auto push = [&](bool p, int cell, int xi) {
        const unsigned long long m = __ballot(p);
        if (!m) return;
        const int c = __popcll(m);
        if (n_rows + c > kRowBuf) flush();
        if (p) rowbuf[n_rows + __popcll(m & ((1ull << lane) - 1ull))] = make_int2(cell, xi);
        __builtin_amdgcn_wave_barrier();
        n_rows += c;
    };
    // a unit of few comparisons a row: as many whole rows as fit, a lane each comparison
    auto unit_by_grid = [&](const int cell, const int xb, const int xe, const int a0, const int na, const int b0,
                            const int nb, const int x0, const int excl, const int64_t base, const int64_t n) {
        const int per = na * nb;
        const float inv = __builtin_amdgcn_rcpf(float(per));  // (exact as below)
        const int rows = int((kWave + 0.5f) * inv), r = int((float(lane) + 0.5f) * inv), k = lane - r * per;
        const int a = int((float(k) + 0.5f) * __builtin_amdgcn_rcpf(float(nb))), al = a0 + a, bl = b0 + k - a * nb;
        unsigned int acc = 0;
        for (int xs = xb; xs < xe; xs += rows) {
            const int xi = xs + r, xl = x0 + xi;
            const bool on = r < rows && xi < xe;
            const int64_t row = base + int64_t(xl) * n;
            unsigned int add = 0;
            bool near = false;
            if (on && !(excl && al == xl)) {
                const float da = p32[row + al], db = p32[row + bl];
                add = (da < db ? 1u : 0u) + (da <= db ? 1u : 0u);
                if (flags) {
                    const uint8_t fa = flags[row + al], fb = flags[row + bl];
                    near = fabsf(da - db) <= margin || ((fa | fb) & kNonRobust) != 0;
                    if (near) {
                        if (!(fa & kMarked)) flags[row + al] = fa | kMarked;
                        if (!(fb & kMarked)) flags[row + bl] = fb | kMarked;
                    }
                }
            }
            const unsigned long long dirty = __ballot(near);
            if (dirty) {  // uniform
                const unsigned long long seg = per == kWave ? ~0ull : ((1ull << per) - 1ull) << (r * per);
                const bool row_dirty = r < rows && (dirty & seg) != 0;
                push(on && row_dirty && k == 0, cell, xi);
                if (row_dirty) add = 0;
            }
            acc += add;
        }
        const unsigned int total = dev::wave_scan_u32(acc);
        if (lane == kWave - 1 && total) atomicAdd(&W[cell], (unsigned long long)total);
    };
    auto unit_by_wave = [&](const int cell, const int xb, const int xe, const int a0, const int na, const int b0,
                            const int nb, const int x0, const int excl, const int64_t base, const int64_t n) {
        // lane side: the larger set; the other passes by
        const bool lanes_b = nb >= na;
        const int l0 = lanes_b ? b0 : a0, nl = lanes_b ? nb : na;
        const int s0 = lanes_b ? a0 : b0, ns = lanes_b ? na : nb;
        const int width = min(nl, kWave);
        // lane / width and 64 / width by the reciprocal (exact: the halves keep the
        // quotients at least 1 / 128 away from a whole number)
        const float inv = __builtin_amdgcn_rcpf(float(width));
        const int rows = int((kWave + 0.5f) * inv), r = int((float(lane) + 0.5f) * inv), k = lane - r * width;
        auto seg = [&] {  // the lanes of this lane's row
            return r < rows ? (width == kWave ? ~0ull : ((1ull << width) - 1ull) << (r * width)) : 0ull;
        };
        unsigned long long acc = 0;
        for (int xs = xb; xs < xe; xs += rows) {
            const int xi = xs + r, xl = x0 + xi;
            const bool on = r < rows && xi < xe;
            const int64_t row = base + int64_t(xl) * n;
            // a value of one side and its flags; x itself and places past the set
            // are NaN (no comparison with them counts or is near)
            auto value = [&](int at, bool in, uint8_t &f) {
                f = flags && in ? flags[row + at] : uint8_t(0);
                return in ? p32[row + at] : __builtin_nanf("");
            };
            unsigned long long dirty = 0;  // lanes that met a near tie
            unsigned long long cnt = 0;
            for (int lc = 0; lc < nl; lc += kWave) {
                const int l_at = l0 + lc + k;
                const bool l_in = on && lc + k < nl && !(excl && !lanes_b && l_at == xl);
                uint8_t lf;
                const float lv = value(l_at, l_in, lf);
                const unsigned long long act = __ballot(l_in);
                unsigned long long near = 0;
                unsigned int below = 0;  // sum of [d_xa < d_xb] + [d_xa <= d_xb]
                for (int sc = 0; sc < ns; sc += width) {
                    const int s_at = s0 + sc + k;
                    const bool s_in = on && sc + k < ns && !(excl && lanes_b && s_at == xl);
                    uint8_t sf;
                    const float sv = value(s_at, s_in, sf);
                    const bool fragile = __ballot((lf | sf) & kNonRobust) != 0;  // rare, uniform
                    bool s_near = false;
                    const int steps = min(width, ns - sc);
                    // four passing values at a time, so that their shuffles overlap
                    // (past the last step they are NaN)
                    for (int i = 0; i < steps; i += 4) {
                        float o[4];
                        unsigned long long m[4] = {0, 0, 0, 0};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float v = __shfl(sv, r * width + i + e, kWave);
                            o[e] = i + e < steps ? v : __builtin_nanf("");
                        }
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float da = lanes_b ? o[e] : lv, db = lanes_b ? lv : o[e];
                            below += (da < db ? 1u : 0u) + (da <= db ? 1u : 0u);
                            if (flags) m[e] = __ballot(fabsf(o[e] - lv) <= margin);
                        }
                        if (fragile)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const int f = lf | __shfl(int(sf), r * width + i + e, kWave);
                                m[e] |= __ballot(i + e < steps && (f & kNonRobust) != 0);
                            }
                        if ((m[0] | m[1] | m[2] | m[3]) & act)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                near |= m[e] & act;
                                if (k == i + e && (m[e] & act & seg())) s_near = true;
                            }
                    }
                    if (s_near && s_in && !(sf & kMarked)) flags[row + s_at] = sf | kMarked;
                }
                if (l_in) cnt += below;
                if (near) {  // uniform
                    if (((near >> lane) & 1ull) && !(lf & kMarked)) flags[row + l_at] = lf | kMarked;
                    dirty |= near;
                }
            }
            if (dirty) {  // uniform
                const bool row_dirty = (dirty & seg()) != 0;
                push(on && row_dirty && k == 0, cell, xi);
                if (row_dirty) cnt = 0;
            }
            acc += cnt;
        }
        // (a unit has at most 8192 comparisons or one x)
        if (int64_t(na) * nb <= (int64_t(1) << 24)) {
            const unsigned int total = dev::wave_scan_u32(unsigned(acc));
            if (lane == kWave - 1 && total) atomicAdd(&W[cell], (unsigned long long)total);
        } else {
            const unsigned long long total = dev::wave_sum_u64(acc);
            if (lane == 0 && total) atomicAdd(&W[cell], total);
        }
    };
    const int64_t n_work = n_units << log_parts;
    const int64_t wave = int64_t(blockIdx.x) * 4 + wv, waves = int64_t(gridDim.x) * 4;
    if constexpr (!kMany) {
        // the tables of the next units are read ahead, one level (unit, cell, group)
        // per unit done: read in turn they cost a unit four trips to memory
        struct Unit {
            int cell, xb, xe;
        };
        auto unit_at = [&](int64_t u) {
            u = min(u, n_work - 1);
            const int32_t *un = units + 3 * (u >> log_parts);
            const int per = (un[2] - un[1] + (1 << log_parts) - 1) >> log_parts;
            const int xb = un[1] + int(u & ((1 << log_parts) - 1)) * per;
            return Unit{un[0], xb, min(xb + per, un[2])};
        };
        Unit u1 = unit_at(wave), u2 = unit_at(wave + waves), u3;
        CellDev c1 = cells[u1.cell], c2;
        int64_t base1 = g_pair_base[c1.group], n1 = g_n[c1.group], base2, n2;
        c2 = cells[u2.cell];
        for (int64_t u = wave; u < n_work; u += waves) {
            base2 = g_pair_base[c2.group];
            n2 = g_n[c2.group];
            u3 = unit_at(u + 2 * waves);
            if (c1.na > 0 && c1.nb > 0 && u1.xb < u1.xe) {  // uniform
                if (int64_t(c1.na) * c1.nb <= kWave)
                    unit_by_grid(u1.cell, u1.xb, u1.xe, c1.a0, c1.na, c1.b0, c1.nb, c1.x0, c1.exclude_self, base1, n1);
                else
                    unit_by_wave(u1.cell, u1.xb, u1.xe, c1.a0, c1.na, c1.b0, c1.nb, c1.x0, c1.exclude_self, base1, n1);
            }
            u1 = u2;
            c1 = c2;
            base1 = base2;
            n1 = n2;
            u2 = u3;
            c2 = cells[u3.cell];
        }
        flush_block();
        return;
    }
    auto bcast = [](int v, int src) { return __builtin_amdgcn_readlane(v, src); };
    auto bcast64 = [&](int64_t v, int src) {
        return int64_t(uint32_t(bcast(int(v), src))) | (int64_t(bcast(int(v >> 32), src)) << 32);
    };
    // the loop bounds are uniform across the wave
    for (int64_t u0 = wave * chunk; u0 < n_units; u0 += waves * chunk) {
        const bool has = lane < chunk && u0 + lane < n_units;
        int cell = 0, xb = 0, xe = 0;
        CellDev c{};
        int64_t base = 0, n = 0;
        if (has) {
            const int32_t *u = units + 3 * (u0 + lane);
            cell = u[0];
            xb = u[1];
            xe = u[2];
            c = cells[cell];
            base = g_pair_base[c.group];
            n = g_n[c.group];
        }
        const int64_t comparisons = has && c.na > 0 && c.nb > 0 ? int64_t(xe - xb) * c.na * c.nb : 0;
        const int mine = comparisons <= kLaneWork ? int(comparisons) : 0;

        // units of a few comparisons, each by its lane
        if (__ballot(mine > 0)) {
            unsigned int acc = 0, cnt = 0;
            int a = 0, b = 0, x = xb, dirty = 0;
            for (int t = 0; __ballot(t < mine); ++t) {
                bool end = false;
                if (t < mine) {
                    const int xl = c.x0 + x, al = c.a0 + a, bl = c.b0 + b;
                    if (!(c.exclude_self && al == xl)) {
                        const int64_t row = base + int64_t(xl) * n;
                        const float da = p32[row + al], db = p32[row + bl];
                        if (flags) {
                            const uint8_t fa = flags[row + al], fb = flags[row + bl];
                            if (fabsf(da - db) <= margin || ((fa | fb) & kNonRobust)) {
                                dirty = 1;
                                if (!(fa & kMarked)) flags[row + al] = fa | kMarked;
                                if (!(fb & kMarked)) flags[row + bl] = fb | kMarked;
                            }
                        }
                        cnt += da < db ? 2u : (da == db ? 1u : 0u);
                    }
                    if (++b == c.nb) {
                        b = 0;
                        if (++a == c.na) {
                            a = 0;
                            end = true;
                        }
                    }
                }
                if (flags) push(end && dirty, cell, x);
                if (end) {
                    if (!dirty) acc += cnt;
                    cnt = 0;
                    dirty = 0;
                    ++x;
                }
            }
            if (acc) atomicAdd(&W[cell], (unsigned long long)acc);
        }

        // the others, by the wave
        for (unsigned long long todo = __ballot(comparisons > kLaneWork); todo; todo &= todo - 1) {
            const int src = __builtin_ctzll(todo);
            unit_by_wave(bcast(cell, src), bcast(xb, src), bcast(xe, src), bcast(c.a0, src), bcast(c.na, src),
                         bcast(c.b0, src), bcast(c.nb, src), bcast(c.x0, src), bcast(c.exclude_self, src),
                         bcast64(base, src), bcast64(n, src));
        }
    }
    flush_block();
}

// Count of sorted values v[0..n) below `key` (strict: v < key) or at most `key`.
template <typename V>
__device__ __forceinline__ int count_below(const V *v, int n, V key, bool inclusive) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        const bool left = inclusive ? v[mid] <= key : v[mid] < key;
        if (left) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Exclusive prefix sums over the 256 threads of one count each; total: their
// sum.  scratch [4] is free again after the next barrier.
__device__ __forceinline__ uint32_t block_prefix(uint32_t v, uint32_t *scratch, uint32_t &total) {
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    uint32_t incl = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t u = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += u;
    }
    if (lane == kWave - 1) scratch[w] = incl;
    __syncthreads();
    uint32_t before = 0;
    total = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (k < w) before += scratch[k];
        total += scratch[k];
    }
    return before + incl - v;
}

// v of lane ^ kD.
template <int kD>
__device__ __forceinline__ uint32_t xor_lane(uint32_t v) {
    const int i = int(v);
    if constexpr (kD == 1) return uint32_t(__builtin_amdgcn_update_dpp(0, i, 0xB1, 0xf, 0xf, true));  // quad 1 0 3 2
    if constexpr (kD == 2) return uint32_t(__builtin_amdgcn_update_dpp(0, i, 0x4E, 0xf, 0xf, true));  // quad 2 3 0 1
    if constexpr (kD == 4) {  // half rows mirrored, then the quads
        const int m = __builtin_amdgcn_update_dpp(0, i, 0x141, 0xf, 0xf, true);
        return uint32_t(__builtin_amdgcn_update_dpp(0, m, 0x1B, 0xf, 0xf, true));
    }
    if constexpr (kD == 8) return uint32_t(__builtin_amdgcn_update_dpp(0, i, 0x128, 0xf, 0xf, true));  // row_ror:8
    if constexpr (kD == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return threadIdx.x & 16 ? r[0] : r[1];
    }
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return threadIdx.x & 32 ? r[0] : r[1];
}

// The n <= 256 kPer values src[0..n) sorted into sv, with their positions in si, by
// a 256-thread block; returns how many are numbers (any NaN lie last: a comparison
// with one is never true, so the counts leave them out).  A bitonic sort of kPer
// consecutive places a thread, in registers: an exchange of places lies within a
// thread, a wave (lane exchanges), or, three times in all, between waves through sv
// and si.  Keys are the values' bits in an unsigned order, NaN above the numbers and
// the padding above both.  Where a merge descends the keys are inverted, so that the
// lower place always takes the lower key.  Its time does not depend on the values
// (buckets of equal width left rows of tied or far-flung values to a sort through
// LDS, and cost such tasks 30%).  Bound by the vector ALUs.  The sorted counting of
// 16,000 rows of 2000 values: 1.37 ms with a bitonic sort through LDS, 0.59 here;
// 40,000 rows of 500: 0.71 and 0.36.
template <int kPer>
__device__ __forceinline__ int sort_places(const float *__restrict__ src, int n, float *sv, uint16_t *si) {
    constexpr int kLogPer = kPer == 1 ? 0 : kPer == 2 ? 1 : kPer == 4 ? 2 : kPer == 8 ? 3 : 4;
    // merges needed (with one place a thread the values start in the first n places)
    const int merges = kPer > 1 || n < 2 ? kLogPer + 8 : 32 - __builtin_clz(unsigned(n - 1));
    const int tid = threadIdx.x;
    uint32_t key[kPer], id[kPer];
#pragma unroll
    for (int m = 0; m < kPer; ++m) {
        id[m] = uint32_t(tid + 256 * m);
        key[m] = ~0u;
        if (int(id[m]) < n) {
            const float v = src[id[m]];
            const uint32_t b = __float_as_uint(v);
            key[m] = v == v ? b ^ (uint32_t(int(b) >> 31) | 0x80000000u) : ~1u;
        }
    }
    // the lower of this place's and the other's key, or the higher where `upper`
    auto keep = [](uint32_t &k, uint32_t &i, uint32_t ok, uint32_t oi, bool upper) {
        const bool take = upper ? k < ok : ok < k;
        k = take ? ok : k;
        i = take ? oi : i;
    };
    auto lanes = [&](auto d_tag) {
        constexpr int d = decltype(d_tag)::value;
        const bool upper = (tid & d) != 0;
#pragma unroll
        for (int m = 0; m < kPer; ++m) keep(key[m], id[m], xor_lane<d>(key[m]), xor_lane<d>(id[m]), upper);
    };
    uint32_t *xk = reinterpret_cast<uint32_t *>(sv);
    auto waves = [&](int d) {
#pragma unroll
        for (int m = 0; m < kPer; ++m) {
            xk[256 * m + tid] = key[m];
            si[256 * m + tid] = uint16_t(id[m]);
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < kPer; ++m)
            keep(key[m], id[m], xk[256 * m + (tid ^ d)], si[256 * m + (tid ^ d)], (tid & d) != 0);
        __syncthreads();
    };
    // merges of 2^p places
#pragma unroll 1
    for (int p = 1; p <= merges; ++p) {
#pragma unroll
        for (int m = 0; m < kPer; ++m) {  // (the last merge ascends where the values are)
            const uint32_t at = uint32_t(tid * kPer + m);
            key[m] ^= 0u - (((at >> p) ^ (p > 1 ? at >> (p - 1) : 0u)) & 1u);
        }
        if (p > kLogPer + 7) waves(128);
        if (p > kLogPer + 6) waves(64);
        if (p > kLogPer + 5) lanes(std::integral_constant<int, 32>{});
        if (p > kLogPer + 4) lanes(std::integral_constant<int, 16>{});
        if (p > kLogPer + 3) lanes(std::integral_constant<int, 8>{});
        if (p > kLogPer + 2) lanes(std::integral_constant<int, 4>{});
        if (p > kLogPer + 1) lanes(std::integral_constant<int, 2>{});
        if (p > kLogPer) lanes(std::integral_constant<int, 1>{});
#pragma unroll
        for (int d = kPer / 2; d > 0; d /= 2)
            if ((1 << p) > d)
#pragma unroll
                for (int m = 0; m < kPer; ++m)
                    if ((m & d) == 0 && key[m + d] < key[m]) {
                        const uint32_t k = key[m], i = id[m];
                        key[m] = key[m + d];
                        id[m] = id[m + d];
                        key[m + d] = k;
                        id[m + d] = i;
                    }
    }
#pragma unroll
    for (int m = 0; m < kPer; ++m) {
        const uint32_t b = key[m] ^ (uint32_t(~int(key[m]) >> 31) | 0x80000000u);
        sv[tid * kPer + m] = key[m] >= ~1u ? __builtin_nanf("") : __uint_as_float(b);
        si[tid * kPer + m] = uint16_t(id[m]);
    }
    __syncthreads();
    return sv[n - 1] == sv[n - 1] ? n : count_below(sv, n, __builtin_inff(), true);
}
// As few places a thread as hold the row (n <= kCap).
template <int kCap>
__device__ __forceinline__ int sort_row(const float *__restrict__ src, int n, float *sv, uint16_t *si) {
    if (n <= 256) return sort_places<1>(src, n, sv, si);
    if (n <= 512) return sort_places<2>(src, n, sv, si);
    if (kCap <= 1024 || n <= 1024) return sort_places<4>(src, n, sv, si);
    if constexpr (kCap > 1024) {
        if (n <= 2048) return sort_places<8>(src, n, sv, si);
        return sort_places<16>(src, n, sv, si);
    }
}

// Large cells, one block per unit (cell, one x): the row's distances to B are
// sorted in LDS, with their B positions, then each a adds
// 2|B| - #(d_xb < d_xa) - #(d_xb <= d_xa), which equals the sum over b of
// 2[d_xa < d_xb] + [d_xa == d_xb].  Near ties and non-robust pairs are found as
// in k_triplets (the b within margin of d_xa form one sorted range) and make
// the row go to the FP64 recount with the involved pairs marked.  kCap: room for
// the task's largest |B|, 1024 (more blocks per CU) or kSortedMaxB.
template <int kCap>
__global__ __launch_bounds__(256) void k_triplets_sorted(const CellDev *__restrict__ cells,
                                                         const int32_t *__restrict__ units, int64_t n_units,
                                                         const int64_t *__restrict__ g_pair_base,
                                                         const int64_t *__restrict__ g_n,
                                                         const float *__restrict__ p32,
                                                         unsigned long long *__restrict__ W,
                                                         uint8_t *flags, float margin,
                                                         int32_t *__restrict__ recount,
                                                         unsigned int *__restrict__ recount_n,
                                                         int64_t recount_cap,
                                                         const unsigned int *__restrict__ scale) {
    if (scale) margin *= __uint_as_float(*scale);  // margin in units of the largest frame length
    __shared__ float sv[kCap];
    __shared__ uint16_t si[kCap];
    __shared__ unsigned long long red[4];
    __shared__ int bad[4];
    const int tid = threadIdx.x, lane = tid % kWave, w = tid / kWave;
    for (int64_t unit = blockIdx.x; unit < n_units; unit += gridDim.x) {
        const int32_t cell_id = units[3 * unit];
        const int32_t xi = units[3 * unit + 1];
        const CellDev c = cells[cell_id];
        const int64_t base = g_pair_base[c.group];
        const int64_t n = g_n[c.group];
        const int nb = c.nb;
        const int xl = c.x0 + xi;
        const float *row = p32 + base + int64_t(xl) * n;
        uint8_t *frow = flags ? flags + base + int64_t(xl) * n : nullptr;
        const int nv = sort_row<kCap>(row + c.b0, nb, sv, si);
        // count, near ties, non-robust pairs
        unsigned long long cnt = 0;
        int dirty = 0, all_b = 0, all_a = 0;
        for (int a = tid; a < c.na; a += 256) {
            const int al = c.a0 + a;
            if (c.exclude_self && al == xl) continue;
            const float da = row[al];
            const int lb = count_below(sv, nv, da, false), ub = count_below(sv, nv, da, true);
            if (da == da) cnt += unsigned(2 * nv - lb - ub);
            if (frow) {
                const uint8_t fa = frow[al];
                if (fa & kNonRobust) {
                    dirty = all_b = 1;
                    frow[al] = fa | kMarked;
                }
                const int lo = count_below(sv, nv, da - margin, false);
                const int hi = count_below(sv, nv, da + margin, true);
                if (lo < hi) {
                    dirty = 1;
                    frow[al] = frow[al] | kMarked;
                    for (int k = lo; k < hi; ++k) {
                        const int bl = c.b0 + si[k];
                        frow[bl] = frow[bl] | kMarked;
                    }
                }
            }
        }
        if (frow)
            for (int b = tid; b < nb; b += 256)
                if (frow[c.b0 + b] & kNonRobust) {
                    dirty = all_a = 1;
                    frow[c.b0 + b] = frow[c.b0 + b] | kMarked;
                }
        const unsigned long long wsum = dev::wave_sum_u64(cnt);
        const int wflags = (dev::wave_any(dirty) ? 1 : 0) | (dev::wave_any(all_b) ? 2 : 0) |
                           (dev::wave_any(all_a) ? 4 : 0);
        if (lane == 0) {
            red[w] = wsum;
            bad[w] = wflags;
        }
        __syncthreads();
        const unsigned long long total = red[0] + red[1] + red[2] + red[3];
        const int f = bad[0] | bad[1] | bad[2] | bad[3];
        if (f & 2)  // a non-robust (x, a): every comparison it takes part in is a near tie
            for (int b = tid; b < nb; b += 256) frow[c.b0 + b] = frow[c.b0 + b] | kMarked;
        if (f & 4)  // a non-robust (x, b)
            for (int a = tid; a < c.na; a += 256) {
                const int al = c.a0 + a;
                if (!(c.exclude_self && al == xl)) frow[al] = frow[al] | kMarked;
            }
        if (tid == 0) {
            if (f & 1) {
                const unsigned int k = atomicAdd(recount_n, 1u);
                if (int64_t(k) < recount_cap) {
                    recount[2 * int64_t(k)] = cell_id;
                    recount[2 * int64_t(k) + 1] = xi;
                }
            } else if (total) {
                atomicAdd(&W[cell_id], total);
            }
        }
        __syncthreads();  // the next unit reuses the sort buffers and reductions
    }
}

// Zeroes the per-cell counts W [n_cells] and the score's kCounterBytes counter bytes
// that follow them, except the error item (the word at byte 8), which starts
// at all ones.
__global__ __launch_bounds__(256) void k_init(unsigned long long *__restrict__ W, int64_t n_cells) {
    const int64_t n = n_cells + kCounterBytes / 8;
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
        W[i] = i == n_cells + 1 ? ~0ull : 0ull;
}

// The marked pairs as (x, y) task items (x the low word), one entry where both
// orientations are marked, in the classes of PairLists (the small ones from
// small_large's start, the large ones from its end: together at most the
// unordered pairs, so they never meet).  In DTW mode pairs with an item of more
// than 64 frames hold their FP64 value already and are only counted; the slots
// (x, x), which nothing compares, are not looked at.  Every pair the triplet
// kernels mark belongs to a row they also send to the recount, so with no such
// row there is nothing to collect.  One pass over the flags, 16 slots
// per lane (HBM-bound when few are marked), and one atomic per class and wave of
// 1024 slots.
__global__ __launch_bounds__(256) void k_collect_pairs(const uint8_t *__restrict__ flags, int64_t n_slots,
                                                       const int64_t *__restrict__ g_item0,
                                                       const int64_t *__restrict__ g_n,
                                                       const int64_t *__restrict__ g_pair_base, int64_t n_groups,
                                                       const int32_t *__restrict__ item_len, PairLists lists,
                                                       const unsigned int *__restrict__ recount_n, int pooled) {
    if (*recount_n == 0) return;
    const int lane = threadIdx.x % kWave;
    const int64_t n16 = (n_slots + 15) / 16;
    for (int64_t c = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; c - lane < n16;
         c += int64_t(gridDim.x) * blockDim.x) {
        const int64_t s0 = 16 * c;
        uint32_t mask = 0;  // bit k: slot s0 + k is marked
        if (s0 + 16 <= n_slots) {
            const uint4 f = *reinterpret_cast<const uint4 *>(flags + s0);
            // the mark bits of four bytes, gathered into four bits
            auto bits = [](uint32_t v) { return (((v >> 1) & 0x01010101u) * 0x01020408u) >> 24; };
            mask = bits(f.x) | (bits(f.y) << 4) | (bits(f.z) << 8) | (bits(f.w) << 12);
        } else {
            for (int64_t k = s0; k < n_slots; ++k) mask |= uint32_t((flags[k] & kMarked) != 0) << (k - s0);
        }
        if (__ballot(mask != 0) == 0) continue;
        // visits the marked slots in order: fn(bit, x, y, group's first item, its items, its first slot)
        const int64_t g_first = mask ? dev::find_segment(g_pair_base, n_groups, s0 + __builtin_ctz(mask)) : 0;
        auto visit = [&](uint32_t bits, auto &&fn) {
            int64_t g = g_first, base = 0, n = 0, i0 = 0, end = 0;
            for (; bits; bits &= bits - 1) {
                const int k = __builtin_ctz(bits);
                const int64_t slot = s0 + k;
                if (n == 0 || slot >= end) {
                    while (slot >= g_pair_base[g + 1]) ++g;
                    base = g_pair_base[g];
                    end = g_pair_base[g + 1];
                    n = g_n[g];
                    i0 = g_item0[g];
                }
                const int64_t local = slot - base;
                int64_t x, y;
                if (end - base <= int64_t(0xFFFFFFFF)) {
                    x = uint32_t(local) / uint32_t(n);
                    y = uint32_t(local) - uint32_t(x) * uint32_t(n);
                } else {
                    x = local / n;
                    y = local - x * n;
                }
                fn(k, x, y, i0, n, base);
            }
        };
        uint32_t small = 0, mid = 0, large = 0, diag = 0;
        visit(mask, [&](int k, int64_t x, int64_t y, int64_t i0, int64_t n, int64_t base) {
            if (x == y) {
                diag |= 1u << k;
                return;
            }
            if (x > y && (flags[base + y * n + x] & kMarked)) return;  // listed as (y, x)
            const int L = pooled ? 0 : max(item_len[i0 + x], item_len[i0 + y]);
            if (L <= 16) small |= 1u << k;
            else if (L <= 32) mid |= 1u << k;
            else if (L <= 64) large |= 1u << k;
        });
        // counts of the wave before this lane (a wave holds 1024 slots), and its totals
        const uint32_t mine = uint32_t(__popc(small)) | (uint32_t(__popc(large)) << 16);
        const uint32_t mine2 = uint32_t(__popc(mid)) | (uint32_t(__popc(mask & ~diag)) << 16);
        uint32_t incl = mine, incl2 = mine2;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const uint32_t v = __shfl_up(incl, o, kWave), v2 = __shfl_up(incl2, o, kWave);
            if (lane >= o) {
                incl += v;
                incl2 += v2;
            }
        }
        uint32_t bs = 0, bm = 0, bl = 0;
        if (lane == kWave - 1) {
            if (incl2 >> 16) atomicAdd(lists.n_marked, incl2 >> 16);
            if (incl & 0xFFFFu) bs = atomicAdd(lists.n_small, incl & 0xFFFFu);
            if (incl2 & 0xFFFFu) bm = atomicAdd(lists.n_mid, incl2 & 0xFFFFu);
            if (incl >> 16) bl = atomicAdd(lists.n_large, incl >> 16);
        }
        const uint32_t excl = incl - mine, excl2 = incl2 - mine2;
        int64_t at_s = int64_t(uint32_t(__shfl(bs, kWave - 1, kWave))) + (excl & 0xFFFFu);
        int64_t at_m = int64_t(uint32_t(__shfl(bm, kWave - 1, kWave))) + (excl2 & 0xFFFFu);
        int64_t at_l = int64_t(uint32_t(__shfl(bl, kWave - 1, kWave))) + (excl >> 16);
        visit(small | mid | large, [&](int k, int64_t x, int64_t y, int64_t i0, int64_t, int64_t) {
            const int64_t e = (i0 + x) | ((i0 + y) << 32);
            if ((mid >> k) & 1u) {
                if (at_m < lists.cap) lists.mid[at_m] = e;
                ++at_m;
            } else {
                const int64_t at = (small >> k) & 1u ? at_s++ : lists.cap - 1 - at_l++;
                if (at >= 0 && at < lists.cap) lists.small_large[at] = e;
            }
        });
    }
}

// One wave per row (cell, x); skip_sorted: rows of sorted_cell() cells are left
// to k_recount_sorted.
__global__ __launch_bounds__(256) void k_recount(const CellDev *__restrict__ cells,
                                                 const int32_t *__restrict__ rows,
                                                 const unsigned int *__restrict__ n_rows,
                                                 int64_t max_rows, int skip_sorted,
                                                 const int64_t *__restrict__ g_pair_base,
                                                 const int64_t *__restrict__ g_n,
                                                 const float *__restrict__ p32,
                                                 const double *__restrict__ p64,
                                                 const uint8_t *__restrict__ flags,
                                                 unsigned long long *__restrict__ W) {
    const int lane = threadIdx.x % kWave;
    const int64_t total = min(int64_t(*n_rows), max_rows);
    const int64_t n_waves = int64_t(gridDim.x) * 4;
    for (int64_t r = int64_t(blockIdx.x) * 4 + threadIdx.x / kWave; r < total; r += n_waves) {
        const int32_t cell_id = rows[2 * r], xi = rows[2 * r + 1];
        const CellDev c = cells[cell_id];
        if (skip_sorted && sorted_cell(c.na, c.nb)) continue;  // wave-uniform
        const int64_t base = g_pair_base[c.group];
        const int64_t n = g_n[c.group];
        const int xl = c.x0 + xi;
        const int64_t roff = base + int64_t(xl) * n;
        const int nb = c.nb;
        const int step_a = kWave / nb, step_b = kWave % nb;
        int a = lane / nb, b = lane % nb;
        unsigned int cnt = 0;
        while (a < c.na) {
            const int al = c.a0 + a, bl = c.b0 + b;
            if (!(c.exclude_self && al == xl)) {
                // FP64 when both pairs were recomputed; otherwise this comparison was
                // already decided far from a tie in FP32 (gap > margin >= 2 x error)
                const bool both = (flags[roff + al] & kMarked) && (flags[roff + bl] & kMarked);
                const double da = both ? p64[roff + al] : double(p32[roff + al]);
                const double db = both ? p64[roff + bl] : double(p32[roff + bl]);
                cnt += da < db ? 2u : (da == db ? 1u : 0u);
            }
            a += step_a;
            b += step_b;
            if (b >= nb) { b -= nb; ++a; }
        }
        const unsigned long long row_total = dev::wave_sum_u64(cnt);
        if (lane == 0 && row_total) atomicAdd(&W[cell_id], row_total);
    }
}

// Rows of large cells, a block each, by the same rule: the FP32 counts of all
// (a, b) from the row's sorted B distances, with the pairs of two recomputed
// distances taken out (prefix counts of the recomputed b in sorted order) and
// counted again from their sorted FP64 values.  Those start in FP32 order, which
// is theirs but for neighbours within the FP32 error, so odd-even exchanges until
// nothing moves sort them in a few rounds.  63,037 rows of up to 1000 x 1000
// comparisons: 42.9 ms with a wave a row over all of them, 1.4 ms here; 550 such
// rows (one wave each left most of the chip idle): 4.4 ms, 0.03 here.
template <int kCap>
__global__ __launch_bounds__(256) void k_recount_sorted(const CellDev *__restrict__ cells,
                                                        const int32_t *__restrict__ rows,
                                                        const unsigned int *__restrict__ n_rows, int64_t max_rows,
                                                        const int64_t *__restrict__ g_pair_base,
                                                        const int64_t *__restrict__ g_n,
                                                        const float *__restrict__ p32,
                                                        const double *__restrict__ p64,
                                                        const uint8_t *__restrict__ flags,
                                                        unsigned long long *__restrict__ W) {
    constexpr int kPer = kCap / 256;
    __shared__ float sv[kCap];
    __shared__ uint16_t si[kCap];
    __shared__ uint32_t marked[kCap + 1], scratch[4];  // marked[k]: recomputed b among the row's first k numbers
    __shared__ double sd[kCap];
    const int tid = threadIdx.x, lane = tid % kWave;
    const int64_t total = min(int64_t(*n_rows), max_rows);
    for (int64_t r = blockIdx.x; r < total; r += gridDim.x) {
        const int32_t cell_id = rows[2 * r], xi = rows[2 * r + 1];
        const CellDev c = cells[cell_id];
        if (!sorted_cell(c.na, c.nb)) continue;  // block-uniform
        const int xl = c.x0 + xi, nb = c.nb;
        const int64_t roff = g_pair_base[c.group] + int64_t(xl) * g_n[c.group];
        const float *row = p32 + roff;
        const double *row64 = p64 + roff;
        const uint8_t *frow = flags + roff;
        const int nv = sort_row<kCap>(row + c.b0, nb, sv, si);
        uint32_t bits = 0, bits64 = 0, n_both;  // bits64: those whose FP64 distance is a number
        double v64[kPer];
#pragma unroll
        for (int m = 0; m < kPer; ++m) {
            const int k = kPer * tid + m;
            if (k < nb && (frow[c.b0 + si[k]] & kMarked)) {
                if (k < nv) bits |= 1u << m;
                v64[m] = row64[c.b0 + si[k]];
                if (v64[m] == v64[m]) bits64 |= 1u << m;
            }
        }
        const uint32_t before = block_prefix(uint32_t(__popc(bits)) | (uint32_t(__popc(bits64)) << 16), scratch, n_both);
        uint32_t at = before & 0xFFFFu, at64 = before >> 16;
#pragma unroll
        for (int m = 0; m < kPer; ++m) {
            marked[kPer * tid + m] = at;
            at += (bits >> m) & 1u;
            if ((bits64 >> m) & 1u) sd[at64++] = v64[m];
        }
        const int nm32 = int(n_both & 0xFFFFu), nm = int(n_both >> 16);
        if (tid == 255) marked[kCap] = uint32_t(nm32);
        __syncthreads();
        for (int moved = 1; moved;) {
            int swapped = 0;
            for (int odd = 0; odd < 2; ++odd) {
                for (int i = 2 * tid + odd; i + 1 < nm; i += 512) {
                    const double u = sd[i], v = sd[i + 1];
                    if (u > v) {
                        sd[i] = v;
                        sd[i + 1] = u;
                        swapped = 1;
                    }
                }
                if (odd == 0) __syncthreads();
            }
            moved = __syncthreads_or(swapped);
        }
        unsigned long long cnt = 0;
        for (int a = tid; a < c.na; a += 256) {
            const int al = c.a0 + a;
            if (c.exclude_self && al == xl) continue;
            const float da = row[al];
            const int lb = count_below(sv, nv, da, false), ub = count_below(sv, nv, da, true);
            int half = da == da ? 2 * nv - lb - ub : 0;
            if (frow[al] & kMarked) {
                const double da64 = row64[al];
                if (da == da) half -= 2 * nm32 - int(marked[lb]) - int(marked[ub]);
                if (da64 == da64)
                    half += 2 * nm - count_below(sd, nm, da64, false) - count_below(sd, nm, da64, true);
            }
            cnt += unsigned(half);
        }
        const unsigned long long wsum = dev::wave_sum_u64(cnt);
        if (lane == 0 && wsum) atomicAdd(&W[cell_id], wsum);
        __syncthreads();  // the next row reuses the buffers
    }
}

}  // namespace

void triplets(hipStream_t s, const CellDev *cells, const int32_t *units, int64_t n_units,
              const GroupTables &g, const float *p32, unsigned long long *W, uint8_t *flags,
              float margin, int32_t *recount, unsigned int *recount_n, int64_t recount_cap,
              const unsigned int *scale) {
    if (n_units <= 0) return;
    if (n_units >= kManyUnits) {
        const int chunk = int(std::min<int64_t>(kWave, n_units / 32768));
        hipLaunchKernelGGL(k_triplets<true>, dim3(grid_for(n_units, 4 * chunk)), dim3(256), 0, s, cells, units, n_units,
                           chunk, 0, g.pair_base, g.n_items, p32, W, flags, margin, recount, recount_n, recount_cap,
                           scale);
    } else {
        // a wave's units lie far apart, so that neighbouring large ones spread out
        const int log_parts = n_units < 4096 ? 2 : 0;
        hipLaunchKernelGGL(k_triplets<false>, dim3(grid_for(n_units << log_parts, 4, 12288)), dim3(256), 0, s, cells, units,
                           n_units, 1, log_parts, g.pair_base, g.n_items, p32, W, flags, margin, recount, recount_n,
                           recount_cap, scale);
    }
    FABX_HIP(hipGetLastError());
}

void triplets_sorted(hipStream_t s, const CellDev *cells, const int32_t *units, int64_t n_units, int max_b,
                     const GroupTables &g, const float *p32, unsigned long long *W, uint8_t *flags,
                     float margin, int32_t *recount, unsigned int *recount_n, int64_t recount_cap,
                     const unsigned int *scale) {
    if (n_units <= 0) return;
    if (max_b > kSortedMaxB) fail(FABX_EINVAL, "a sorted cell's B is larger than the sort takes");
    hipLaunchKernelGGL(max_b <= 1024 ? k_triplets_sorted<1024> : k_triplets_sorted<kSortedMaxB>,
                       dim3(grid_for(n_units, 1)), dim3(256), 0, s, cells, units, n_units,
                       g.pair_base, g.n_items, p32, W, flags, margin, recount, recount_n, recount_cap, scale);
    FABX_HIP(hipGetLastError());
}

void init_score(hipStream_t s, unsigned long long *W, int64_t n_cells) {
    const int64_t blocks = std::min<int64_t>((n_cells + kCounterBytes / 8 + 255) / 256, 4096);
    hipLaunchKernelGGL(k_init, dim3(unsigned(blocks)), dim3(256), 0, s, W, n_cells);
    FABX_HIP(hipGetLastError());
}

void collect_pairs(hipStream_t s, const uint8_t *flags, int64_t n_slots, const GroupTables &g, const ItemTables &it,
                   const PairLists &lists, const unsigned int *recount_n, bool pooled) {
    if (n_slots <= 0) return;
    const int64_t blocks = std::min<int64_t>((n_slots + 4095) / 4096, 4096);
    hipLaunchKernelGGL(k_collect_pairs, dim3(unsigned(blocks)), dim3(256), 0, s, flags, n_slots, g.item0, g.n_items,
                       g.pair_base, g.n_groups, it.len, lists, recount_n, pooled ? 1 : 0);
    FABX_HIP(hipGetLastError());
}

void recount(hipStream_t s, const CellDev *cells, const int32_t *rows, const unsigned int *n_rows,
             int64_t max_rows, int max_b, const GroupTables &g, const float *p32, const double *p64,
             const uint8_t *flags, unsigned long long *W) {
    if (max_rows <= 0) return;
    if (max_b > kSortedMaxB) fail(FABX_EINVAL, "a sorted cell's B is larger than the sort takes");
    const int64_t blocks = std::min<int64_t>((max_rows + 3) / 4, 2048);
    hipLaunchKernelGGL(k_recount, dim3(unsigned(blocks)), dim3(256), 0, s, cells, rows, n_rows,
                       max_rows, max_b > 0 ? 1 : 0, g.pair_base, g.n_items, p32, p64, flags, W);
    if (max_b > 0)
        hipLaunchKernelGGL(max_b <= 1024 ? k_recount_sorted<1024> : k_recount_sorted<kSortedMaxB>,
                           dim3(unsigned(std::min<int64_t>(max_rows, 2048))), dim3(256), 0, s, cells, rows, n_rows,
                           max_rows, g.pair_base, g.n_items, p32, p64, flags, W);
    FABX_HIP(hipGetLastError());
}

}  // namespace kern
}  // namespace fabx
