// Diagonal storage of the batch's bands (gfx950, wave64).
//
// A symmetric band whose entries lie on at most kBdsMax distances |i - j| <= 31
// keeps, in its slices' SELL-64 places (columns stay, for the 2BFS), the main
// diagonal and the upper ones instead of whole rows: place t of a slice holds
// a_ii (t = 0) or a_{i, i + d_t} of its 64 rows, NaN where the pattern has no
// entry (stored values are finite).  The lower entry a_{i, i - d} is the upper
// one of row i - d, in the same slice or the one before.
//
// A product then reads nh + 1 values a row, straight through, where SELL-64
// reads 2 nh + 1 values and as many 32-bit columns; every address follows from
// the row, so the loads do not wait for columns; and the vector's elements of a
// slice are formed once (with a halo of 31 on both sides, in LDS) instead of
// once per entry.  Each lane adds its row's entries from the lowest diagonal to
// the highest in one fma chain from 0, absent ones skipped: SELL-64's bits.
//
// What bounds it: the chain work list, state, slice offset, matrix, then the
// plane reads.  96 mixed systems of up to 100,000 rows, whose bands (half-width
// 8) run on when the others are done: 36.6 us a product over the run before,
// 21.1 now; the batch 139 -> 104 ms.  Looking every entry's mirror image up at
// admission takes 0.2 ms of that.

#pragma once

#include "batch_step.hpp"

namespace mpcg {
namespace batch {

constexpr int kBdsHalo = kBandMaxBw;
constexpr int kBdsLds = 64 + 2 * kBdsHalo;   // vector elements a wave keeps

// The distances d > 0 of the system's entries: bit d.
__device__ inline uint32_t bds_dist(unsigned long long doffs) { return (uint32_t)(doffs >> 32) & ~1u; }

// Whether the system's distances allow diagonal storage.  Worth it where two
// thirds of the diagonals' places hold an entry; systems that may advance in
// one workgroup keep SELL-64, which those steps read.
__device__ inline int bds_candidate(const BSys &S)
{
    if (S.err || S.bw > kBandMaxBw || S.nslices <= kWgMaxSlices) return 0;
    const uint32_t up = bds_dist(S.doffs), low = (uint32_t)S.doffs;   // low: distance d at bit 32 - d
    const int nh = __popc(up);
    if (nh < 1 || nh > kBdsMax || (__brev(up) << 1) != low) return 0;
    if ((int64_t)(2 * nh + 1) * S.n * 2 > 3 * S.nnz) return 0;
    return nh;
}

// Wave per slice, SELL-64 in place: every entry must have its mirror image, bit
// for bit, and every slice room for the diagonals.
__device__ inline void bds_verify(const BArena &a, const BSys &S, int64_t entry0, int32_t sys, int sl)
{
    const int nh = bds_candidate(S);
    if (!nh) return;
    const int lane = threadIdx.x & 63, row = sl * 64 + lane, len = a.rowlen[row];
    const int64_t base = entry0 + a.slice_off[sl] + lane;
    int bad = a.slice_w[sl] < nh + 1;
    for (int k = 0; k < len; ++k) {
        const int c = a.col[base + (int64_t)k * 64];
        if (c == row) continue;
        const int64_t pb = entry0 + a.slice_off[c >> 6] + (c & 63);
        const int pl = a.rowlen[c];
        int found = 0;
        for (int t = 0; t < pl; ++t) {
            const int pc = a.col[pb + (int64_t)t * 64];
            if (pc < row) continue;
            found = pc == row && __double_as_longlong(a.v64[pb + (int64_t)t * 64]) ==
                                     __double_as_longlong(a.v64[base + (int64_t)k * 64]);
            break;
        }
        if (!found) bad = 1;
    }
    if (__any(bad) && lane == 0) atomicOr(&a.sys[sys].ds_bad, 1);
}

// Wave per slice: the slice's values become its diagonals, in place (a slice's
// entries are read by its own wave alone, all before the first store).
__device__ inline void bds_convert(const BArena &a, const BSys &S, int sl)
{
    if (!S.ds) return;
    const int lane = threadIdx.x & 63, row = sl * 64 + lane, len = a.rowlen[row];
    const int64_t base = S.entry0 + a.slice_off[sl] + lane;
    int k = 0;
    while (k < len && a.col[base + (int64_t)k * 64] < row) ++k;
    double v[kBdsMax + 1];
    uint32_t m = bds_dist(S.doffs) | 1u;   // the main diagonal first
#pragma unroll
    for (int t = 0; t <= kBdsMax; ++t) {
        v[t] = NAN;
        if (m && k < len && a.col[base + (int64_t)k * 64] == row + __builtin_ctz(m)) v[t] = a.v64[base + (int64_t)k++ * 64];
        m &= m - 1u;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
#pragma unroll
    for (int t = 0; t <= kBdsMax; ++t)
        if (t <= S.ds) {
            a.v64[base + (int64_t)t * 64] = v[t];
            a.v32[base + (int64_t)t * 64] = (float)v[t];
        }
}

// Row sums of slice sl with the vector elements g(row); lu: the wave's LDS.
// own: the row's element.
template <typename T, typename G>
__device__ inline T bds_sum(const BArena &a, const StepSys &S, const T *val, int sl, T *lu, const G &g, T &own)
{
    const int lane = threadIdx.x & 63, row = sl * 64 + lane;
    const int nh = S.ds;
    const uint32_t dist = bds_dist(S.doffs);
    const bool top = sl == S.slice0;
    // one scalar base, the previous slice's places first
    const int64_t off0 = a.slice_off[top ? sl : sl - 1];
    const uint32_t ahead = (uint32_t)(a.slice_off[sl] - off0);
    const T *p = val + S.entry0 + off0;
    T lo[kBdsMax], hi[kBdsMax];
    const T mid = p[ahead + lane];
    uint32_t m = dist;
#pragma unroll
    for (int t = 0; t < kBdsMax; ++t) {
        lo[t] = hi[t] = T(NAN);
        if (t >= nh) continue;
        const int d = __builtin_ctz(m);
        m &= m - 1u;
        const uint32_t at = (uint32_t)((t + 1) * 64 + lane);
        hi[t] = p[ahead + at];
        const bool here = lane >= d;
        lo[t] = p[here ? ahead + at - d : at + 64 - d];
        if (top && !here) lo[t] = T(NAN);
    }
    const int reach = 31 - __builtin_clz(dist);
    const int h = lane < reach ? lane - reach : lane + reach;
    const bool halo = lane < reach || lane >= 64 - reach;
    const int first = S.row0, last = S.row0 + S.nslices * 64 - 1;
    own = g(row);
    T out = T(0);
    if (halo) out = g(max(first, min(sl * 64 + h, last)));
    lu[kBdsHalo + lane] = own;
    if (halo) lu[kBdsHalo + h] = out;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const T *u = lu + kBdsHalo + lane;
    T acc = T(0);
    m = dist;
#pragma unroll
    for (int t = kBdsMax - 1; t >= 0; --t) {
        if (t >= nh) continue;
        const int d = 31 - __builtin_clz(m);
        m &= ~(1u << d);
        const T f = fma_b<T>(lo[t], u[-d], acc);
        acc = lo[t] == lo[t] ? f : acc;
    }
    {
        const T f = fma_b<T>(mid, own, acc);
        acc = mid == mid ? f : acc;
    }
    m = dist;
#pragma unroll
    for (int t = 0; t < kBdsMax; ++t) {
        if (t >= nh) continue;
        const int d = __builtin_ctz(m);
        m &= m - 1u;
        const T f = fma_b<T>(hi[t], u[d], acc);
        acc = hi[t] == hi[t] ? f : acc;
    }
    return acc;
}

// As cg_product and residual for a system in diagonal storage.
template <typename T>
__device__ inline double bds_product(const BArena &a, const StepSys &S, const T *val, const T *r, T *dA, T *dB, T *q,
                                     int sl, T *lu)
{
    const int row = sl * 64 + (int)(threadIdx.x & 63);
    const int j = S.ph_it;
    const bool first = j == 0;
    const T beta = (T)S.beta;
    T *dnew = (j & 1) ? dB : dA;
    const T *dold = (j & 1) ? dA : dB;
    T dn;
    const T acc = bds_sum<T>(a, S, val, sl, lu, [&](int i) { return first ? r[i] : fma_b<T>(beta, dold[i], r[i]); }, dn);
    dnew[row] = dn;
    q[row] = acc;
    if (sizeof(T) == 4) return wave_dot32(a.acc32, (float)dn, (float)acc);
    return wave_dot((double)dn, (double)acc);
}

__device__ inline double bds_residual(const BArena &a, const StepSys &S, bool restart, int sl, double *lu)
{
    const int row = sl * 64 + (int)(threadIdx.x & 63);
    const int src = restart ? S.src : (int)kSrcX64;
    const float *xs = src == kSrcSnap ? a.snap32 + (size_t)S.snap_ci * ((size_t)a.max_slices * 64) : a.x32;
    double xv;
    const double acc = bds_sum<double>(
        a, S, a.v64, sl, lu,
        [&](int i) { return src == kSrcX64 ? a.x64[i] : src == kSrcZero ? 0.0 : (double)xs[i]; }, xv);
    const double res = a.b64[row] - acc;
    if (restart) {
        if (src != kSrcX64) a.x64[row] = xv;
        a.r64[row] = res;
    }
    return wave_dot(res, res);
}

}  // namespace batch
}  // namespace mpcg
