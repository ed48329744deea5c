// Device helpers shared by the fused DTW kernels: where the items of a work
// unit's row block (at most 64 frames) and column block (kC frames) begin, as bit
// masks over their frames, and what a lane and a wave take from them.
//
// The masks are made from the item lengths by two waves (kC / 64 column items or
// one row item per lane, one prefix sum, one LDS OR per item) while the first
// frames are on their way; a walk over the items by every wave cost a dependent
// load and a dozen instructions per item, four times per unit.  It shows where
// units are few and small (distance stage, with the branch-free steps of the
// kernels): 400 items 21 -> 17 us, discrete units 156 -> 126 us.
#pragma once

#include "device_common.h"

namespace fabx {
namespace kern {
namespace unit {

using dev::kWave;

// In LDS: where items begin (rows, columns), the row block's longest item, and
// each item's last frame.
template <int kC>
struct Items {
    uint32_t row_first[2], col_first[kC / 32];
    uint32_t longest;
    uint8_t row_last[64], col_last[kC];
};

// Waves 0 (rows) and 1 (columns) fill `m`; readable after the next barrier.
template <int kC>
__device__ __forceinline__ void find_items(Items<kC> &m, const int32_t *__restrict__ item_len, int r_item0,
                                           int r_nitems, int c_item0, int c_nitems) {
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    if (w == 0) {
        if (lane < 2) m.row_first[lane] = 0;
        const int L = lane < r_nitems ? item_len[r_item0 + lane] : 0;
        const int incl = int(dev::wave_scan_u32(unsigned(L)));
        const int at = incl - L;
        if (L > 0) {
            atomicOr(&m.row_first[at / 32], 1u << (at % 32));
            m.row_last[lane] = uint8_t(incl - 1);
        }
        const unsigned longest = dev::wave_max_u32(unsigned(L));
        if (lane == kWave - 1) m.longest = longest;
    } else if (w == 1) {
        constexpr int kPer = kC / kWave;  // items per lane
        if (lane < kC / 32) m.col_first[lane] = 0;
        int L[kPer], sum = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int i = kPer * lane + k;
            L[k] = i < c_nitems ? item_len[c_item0 + i] : 0;
            sum += L[k];
        }
        int at = int(dev::wave_scan_u32(unsigned(sum))) - sum;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            if (L[k] > 0) {
                atomicOr(&m.col_first[at / 32], 1u << (at % 32));
                m.col_last[kPer * lane + k] = uint8_t(at + L[k] - 1);
            }
            at += L[k];
        }
    }
}

// Frame r of the row block (lane r): its index in its item, whether it is the
// item's last.
struct Row {
    int ir;
    bool last;
};
template <int kC>
__device__ __forceinline__ Row row_of(const Items<kC> &m, int r, int frames) {
    const uint64_t first = uint64_t(m.row_first[0]) | (uint64_t(m.row_first[1]) << 32);
    const uint64_t upto = first & (~0ull >> (63 - r));  // bit 0 is always set
    Row o;
    o.ir = r - (63 - __builtin_clzll(upto));
    o.last = r == frames - 1 || (r < 63 && ((first >> (r + 1)) & 1u));
    if (r >= frames) o = Row{0, false};
    return o;
}

// The column block's mask in scalar registers.
template <int kC>
struct Cols {
    uint64_t f[kC / 64];
    __device__ __forceinline__ explicit Cols(const Items<kC> &m) {
#pragma unroll
        for (int k = 0; k < kC / 64; ++k)
            f[k] = uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(m.col_first[2 * k])))) |
                   (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(m.col_first[2 * k + 1])))) << 32);
    }
    // First item start at or after column p (uniform), or `none`.
    __device__ __forceinline__ int next_first(int p, int none) const {
        int at = none;
#pragma unroll
        for (int k = kC / 64 - 1; k >= 0; --k) {
            const int q = p - 64 * k;
            const uint64_t v = q <= 0 ? f[k] : q < 64 ? f[k] & (~0ull << q) : 0;
            if (v) at = 64 * k + __builtin_ctzll(v);
        }
        return at;
    }
    // Item starts before column p (uniform).
    __device__ __forceinline__ int items_before(int p) const {
        int n = 0;
#pragma unroll
        for (int k = 0; k < kC / 64; ++k) {
            const int q = p - 64 * k;
            n += q >= 64 ? __builtin_popcountll(f[k]) : q > 0 ? __builtin_popcountll(f[k] & ~(~0ull << q)) : 0;
        }
        return n;
    }
    // Column c starts an item (c < kC).
    __device__ __forceinline__ uint32_t starts(int c) const {
        uint64_t v = f[0];
#pragma unroll
        for (int k = 1; k < kC / 64; ++k)
            if (c >= 64 * k) v = f[k];
        return uint32_t(v >> (c % 64)) & 1u;
    }
    // The kernels' flag word of column c of `frames`: byte 0 = 1 at an item's first
    // column, bit 31 = its last column.
    __device__ __forceinline__ uint32_t flag(int c, int frames) const {
        return starts(c) | (c == frames - 1 ? 0x80000000u : starts(c + 1) << 31);
    }
};

// The columns [begin, end) of wave w: the items whose first frame falls in its
// quarter of the needed columns (from `skip` on, where an item starts).
struct Span {
    int begin, end;
};
template <int kC>
__device__ __forceinline__ Span span_of(const Cols<kC> &cols, int w, int skip, int frames) {
    const int kept = frames - skip;
    const int lo = skip + (w * kept + 3) / 4, hi = skip + ((w + 1) * kept + 3) / 4;
    return {cols.next_first(lo, frames), cols.next_first(hi, frames)};
}

// The pairs (row item i, column item j) of the wave's span that the unit writes,
// in turn over its lanes: those whose row item comes no later in the packing order.
// fn(i, j, x, y, same) with the items' places x, y in their group, whose first
// task item is item0; r_item0, c_item0: the blocks' first positions; order: the
// task item at each position (null: the position).
template <int kC, typename Fn>
__device__ __forceinline__ void for_pairs(const Cols<kC> &cols, const Span &span, int r_nitems, int r_item0,
                                          int c_item0, int64_t item0, const int32_t *__restrict__ order, Fn &&fn) {
    const int j0 = cols.items_before(span.begin), nj = cols.items_before(span.end) - j0;
    // (exact: at most 64 x 256 pairs, and the half keeps the quotient 1 / 512 away
    // from a whole number)
    const float inv = __builtin_amdgcn_rcpf(float(nj));
    for (int k = threadIdx.x % kWave; k < r_nitems * nj; k += kWave) {
        const int i = int((float(k) + 0.5f) * inv), j = j0 + k - i * nj;
        const int pr = r_item0 + i, pc = c_item0 + j;
        if (pr <= pc) fn(i, j, (order ? order[pr] : pr) - item0, (order ? order[pc] : pc) - item0, pr == pc);
    }
}

}  // namespace unit
}  // namespace kern
}  // namespace fabx
