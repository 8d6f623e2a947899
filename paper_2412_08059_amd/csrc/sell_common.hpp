// Device helpers shared by the SELL-64 kernels: fma in the working
// precision, wave and block sums, the fixed-order reduction of per-block
// partials, and the XCD-aware walk of slice groups.

#pragma once

#include "mpcg_internal.hpp"
#include "wave_ops.hpp"

#include <cmath>

namespace mpcg {

// Row r of ingest's sample, one in each kDsSample-th of the rows (may be >= n).
__device__ inline int64_t ds_sample_row(int r, int32_t n)
{
    const int64_t step = ((int64_t)n + kDsSample - 1) / kDsSample;
    return (int64_t)r * step + (r * 2654435761u >> 7) % (uint64_t)step;
}

template <typename T> __device__ inline T fma_t(T a, T b, T c);
template <> __device__ inline float fma_t<float>(float a, float b, float c) { return fmaf(a, b, c); }
template <> __device__ inline double fma_t<double>(double a, double b, double c) { return fma(a, b, c); }

// Block sum (kBlock threads): butterfly in each wave, then waves 0..3 in
// order.  Valid in thread 0; sm (kBlock / 64 doubles) may be reused after it.
__device__ inline double sell_block_sum(double v, double *sm)
{
    v = wave_sum_all(v);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) sm[w] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < kBlock / 64; ++i) s += sm[i];
    __syncthreads();
    return s;
}

// The same sum delivered to every thread with one barrier.  sm must not be
// written again by the kernel (each sum has a slot array of its own).
__device__ inline double block_total(double v, double *sm)
{
    v = wave_sum_all(v);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    for (int i = 0; i < kBlock / 64; ++i) s += sm[i];
    return s;
}

// This thread's share of cnt <= kMaxGrid partials, added in index order.  All
// loads are issued at once; a share past cnt adds +0.0, which leaves the
// sum's bits unchanged (the running sum starts at +0.0 and so is never -0.0).
__device__ inline double partials_share(const double *p, int cnt)
{
    double pv[kMaxGrid / kBlock];
#pragma unroll
    for (int k = 0; k < kMaxGrid / kBlock; ++k) {
        const int i = threadIdx.x + k * kBlock;
        pv[k] = i < cnt ? p[i] : 0.0;
    }
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < kMaxGrid / kBlock; ++k) acc += pv[k];
    return acc;
}

// FP32 accumulation (dot_acc = 1): the same trees in float; partials are
// stored widened to double and narrowed back, both exact.
__device__ inline float sell_block_sum_f(float v, double *sm)
{
    v = wave_sum_all(v);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) sm[w] = (double)v;
    __syncthreads();
    float s = 0.0f;
    if (threadIdx.x == 0)
        for (int i = 0; i < kBlock / 64; ++i) s += (float)sm[i];
    __syncthreads();
    return s;
}

__device__ inline double block_total_f(float v, double *sm)
{
    v = wave_sum_all(v);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = (double)v;
    __syncthreads();
    float s = 0.0f;
    for (int i = 0; i < kBlock / 64; ++i) s += (float)sm[i];
    return (double)s;
}

__device__ inline float partials_share_f(const double *p, int cnt)
{
    float acc = 0.0f;
    for (int i = threadIdx.x; i < cnt; i += kBlock) acc += (float)p[i];
    return acc;
}

// Sum of the previous kernel's partials in the precision dot_acc asks for:
// every block gets the same bits.
__device__ inline double partials_total(bool f32, const double *p, int cnt, double *sm)
{
    return f32 ? block_total_f(partials_share_f(p, cnt), sm) : block_total(partials_share(p, cnt), sm);
}

// ---- head of a CG product kernel (all storage formats)
//
// The stop flag, the previous iteration's scalars and the update's partials
// are independent loads: every thread issues them together at the start (the
// scalars are uniform), so the head costs one memory latency and one barrier
// where reading the flag, then the partials, then the scalars costs three of
// each.  A stale scalar cannot be picked up: a launch writes only the parity
// slots of its own iteration and reads those of the one before.
struct CgHead {
    bool skip;        // the recurrence has stopped: nothing to do
    bool xdone;       // x already holds x_it
    bool f32acc;      // dot_acc = 1 (FP32 phase)
    double rho, g;    // rho_it (alpha, beta) and gamma_it = r.r (stop test, v)
    double gp, rhop;  // the same of iteration it - 1
    double alph;      // alpha_{it-1}
    double thr;
    int32_t maxit;
};

// live: a word in host memory that the host reads once a group of iterations
// has run; the launch in which the recurrence stops clears it, and so does
// every one after it (a copy of the device state for each group cost the
// stream a launch and two gaps, 5 us).
__device__ inline void host_stopped(int32_t *live)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) __hip_atomic_store(live, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

template <typename T>
__device__ inline CgHead cg_head(const DevState *st, const double *up, int nup, int pc, int it, int it0, double *sm,
                                 double *sm2, int32_t *live)
{
    CgHead h;
    const int32_t stop = st->stop_it, xit = st->x_it;
    const int pv = (it - 1) & 1;
    h.gp = st->gr[pv];
    h.rhop = st->gam[pv];
    h.alph = st->alph[pv];
    h.thr = st->thr;
    h.maxit = st->maxit;
    h.f32acc = sizeof(T) == 4 && st->acc32;
    h.rho = h.g = 0.0;
    h.xdone = xit == it;
    h.skip = stop < it;
    if (h.skip) host_stopped(live);
    if (h.skip || it == it0) return h;
    h.rho = partials_total(h.f32acc, up, nup, sm);
    h.g = pc ? partials_total(h.f32acc, up + nup, nup, sm2) : h.rho;   // equal without a preconditioner
    return h;
}

// The stop test of iteration it and what block 0 records of it; returns
// whether the recurrence stops here.
__device__ inline bool cg_head_decide(DevState *st, const CgHead &h, int it, int32_t *live)
{
    const bool conv = sqrt(h.g) <= h.thr;
    const bool cap = !conv && it >= h.maxit;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->gam[it & 1] = h.rho;
        st->gr[it & 1] = h.g;
        const int k = it - 1;
        if (k < st->k0rec && k < kK0Max) st->ratios[k] = sqrt(h.g) / sqrt(h.gp);
        if (conv || cap) {
            st->gamma = h.g;
            st->iter = it;
            st->reason = conv ? kConverged : kMaxit;
            st->stop_it = it;
            st->live = 0;
            host_stopped(live);
        }
    }
    return conv || cap;
}

__device__ inline void record_crossings(DevState *st, unsigned cross, int it, double g)
{
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    for (int t = 0; t < kNumEps; ++t) {
        if (!(cross & (1u << t))) continue;
        st->cross_iter[t] = it;
        st->cross_gamma[t] = g;
    }
}

// Slice groups (kBlock / 64 slices, one per wave) of an XCD's contiguous
// range (in proportion to its blocks) are dealt round-robin to that XCD's
// blocks: at any moment the blocks of one XCD work on a narrow window of
// consecutive rows, so the rows that a stencil's neighbour planes gather are
// still in that XCD's L2.  The ranges come from the host with the launch: two
// 64-bit divisions per wave are several hundred scalar instructions.
struct SliceWalk {
    int g, g_end, step;   // group index, end, stride
};

// As a table: diagonal storage and the Jacobi iterations (FP64 CG product of the
// 1 M band 19.0 us; 22.0 with the divisions, 21.4 with the numbers below).
__device__ inline SliceWalk slice_walk(const WalkTab &t)
{
    const int x = blockIdx.x % kNumXcd, i = blockIdx.x / kNumXcd;
    SliceWalk w;
    w.g = t.first[x] + i;
    w.g_end = t.first[x + 1];
    w.step = t.blocks[x];
    return w;
}

// As numbers: the SELL products, which lose by reading the table at the block's
// index, however early.  CG products, us with the table, read first, and with
// the numbers: FP64 7-point 128^3 43.8, 42.7, 41.1; 19-point 100^3 45.7, 44.1,
// 42.5; 1 M rows of half-width 9 45.9, 44.0, 42.3; 5-point 1001^2 20.9, 20.2,
// 19.5; FP32 of these 24.6 to 13.5, 24.1 to 13.1, 23.4 to 12.7.  (One loses: the
// unsplit product of a random graph of 1 M rows, 420 and 431.)
__device__ inline SliceWalk slice_walk(const WalkNum &t)
{
    const int x = blockIdx.x % kNumXcd, i = blockIdx.x / kNumXcd;
    SliceWalk w;
    w.g = walk_first(t, x) + i;
    w.g_end = walk_first(t, x + 1);
    w.step = walk_blocks(t, x);
    return w;
}

}  // namespace mpcg
