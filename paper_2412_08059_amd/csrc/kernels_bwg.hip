// Steps of small systems, one workgroup per system (gfx950).
//
// A step of the batch is two launches over all listed slices; with systems of
// a few thousand rows each launch is mostly latency (gaps, and chains of work
// list, state, slice and matrix loads).  While no listed system is larger (or
// has more entries than one workgroup reads in that time, wg_max_entries), a
// workgroup takes its system through up to `steps` steps instead: the state in
// LDS, x, r and d of its rows and their first E entries in registers, d (or
// the x of a residual) also in LDS for the gathers, entries past E read where
// they lie.  The state machine and every sum are those of the step kernels
// (per-slice partials added by one wave), so a system may pass from one form
// to the other at any step and its bits do not show it.
//
// Thread T owns rows T + 1024 k, k < R: slice W + 16 k belongs to wave W.  An
// entry past a row's length is -0.0 times an LDS element that holds +0.0.
//
// What bounds it: the five barriers of a step and the scalars one lane forms
// between them (512 systems of 1,000 rows, two workgroups a CU: 2.7 us a step
// for all of them).  Batches, ms, two launches a step and this: 512 trees of
// 1,000 rows 20.7 and 5.6, 100 of 300 .. 1,000 rows (FP64) 6.9 and 2.4, 64 mixed
// systems of 1,000 .. 2,000 rows 10.7 and 5.1, of 1,000 .. 4,000 rows with
// features 21.3 and 16.7 (what is left there is the 2BFS).  Half or twice the
// entries in registers: within 1%.

#include "batch_step.hpp"

#include <cstddef>

namespace mpcg {
namespace batch {

namespace {

constexpr int kWgThreads = 1024;
constexpr int kWgWaves = kWgThreads / 64;

// Sum of the system's slice partials (at most 64), first wave, every lane: the
// order of the step kernels' block sum, whose other terms are zeros.
__device__ inline double wg_sum(const double *part, int ns, bool f32)
{
    const int lane = threadIdx.x & 63;
    if (f32) {
        const float v = lane < ns ? 0.0f + (float)part[lane] : 0.0f;
        return (double)(0.0f + wave_sum_all(v));
    }
    const double v = lane < ns ? 0.0 + part[lane] : 0.0;
    return 0.0 + wave_sum_all(v);
}

// Entries from .. len - 1 of a row, gathered from LDS and added to acc in order.
template <typename T>
__device__ inline T wg_entries(const int32_t *col, const T *val, const T *s_d, int32_t row0, int from, int len, T acc)
{
    constexpr int kAhead = 4;
    for (int k0 = from; k0 < len; k0 += kAhead) {
        int c[kAhead];
        T v[kAhead];
#pragma unroll
        for (int t = 0; t < kAhead; ++t)
            if (k0 + t < len) {
                c[t] = col[(int64_t)(k0 + t) * 64];
                v[t] = val[(int64_t)(k0 + t) * 64];
            }
#pragma unroll
        for (int t = 0; t < kAhead; ++t)
            if (k0 + t < len) acc = fma_b<T>(v[t], s_d[c[t] - row0], acc);
    }
    return acc;
}

// CG steps of the system's phase until it ends or no step is left.
template <typename T, int R, int E>
__device__ inline void wg_cg(const BArena &a, BSys &S, const T *val, T *xg, T *rg, T *dA, T *dB, T *s_d, double *part,
                             int &left, bool hold)
{
    constexpr int kZero = R * kWgThreads;   // the LDS element that holds +0.0
    const int tid = threadIdx.x, lane = tid & 63, W = tid >> 6;
    const int ns = S.nslices, row0 = S.row0, mode = S.mode;
    T x[R], r[R], d[R], mv[R][E];
    uint32_t mi[R][(E + 1) / 2];   // LDS byte addresses of the columns, two per register
    int len[R];
    int64_t at[R];
    {
        const T *dold = (S.ph_it & 1) ? dA : dB;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const bool on = W + k * kWgWaves < ns;
            const int row = row0 + (on ? tid + k * kWgThreads : lane);
            x[k] = xg[row];
            r[k] = rg[row];
            d[k] = dold[row];
            len[k] = on ? a.rowlen[row] : 0;
            at[k] = S.entry0 + a.slice_off[row >> 6] + lane;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const bool in = e < len[k];
                const int64_t p = at[k] + (in ? (int64_t)e * 64 : 0);
                uint32_t b = (uint32_t)kZero * (uint32_t)sizeof(T);
                mv[k][e] = T(-0.0);
                if (in) {
                    b = (uint32_t)(a.col[p] - row0) * (uint32_t)sizeof(T);
                    mv[k][e] = val[p];
                }
                if (e & 1) mi[k][e / 2] |= b << 16;
                else mi[k][e / 2] = b;
            }
        }
    }
    if (tid == 0) s_d[kZero] = T(0);
    const bool f32 = sizeof(T) == 4 && a.acc32;
#pragma clang loop unroll(disable)
    for (;;) {
        int own = tid;   // opaque: addresses are formed where they are used
        asm volatile("" : "+v"(own));
        const bool first = S.ph_it == 0;
        const T beta = (T)S.beta;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            d[k] = first ? r[k] : fma_b<T>(beta, d[k], r[k]);
            s_d[own + k * kWgThreads] = d[k];
        }
        __syncthreads();
        T q[R];
#pragma unroll
        for (int k = 0; k < R; ++k) {
            T acc = T(0);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const uint32_t b = (e & 1) ? mi[k][e / 2] >> 16 : mi[k][e / 2] & 0xffffu;
                acc = fma_b<T>(mv[k][e], *reinterpret_cast<const T *>(reinterpret_cast<const char *>(s_d) + b), acc);
            }
            if (__any(len[k] > E)) acc = wg_entries<T>(a.col + at[k], val + at[k], s_d, row0, E, len[k], acc);
            q[k] = acc;
            const double p = sizeof(T) == 4 ? wave_dot32(f32, (float)d[k], (float)acc)
                                            : wave_dot((double)d[k], (double)acc);
            if (lane == 0) part[W + k * kWgWaves] = p;
        }
        __syncthreads();
        if (W == 0) {
            const double v = wg_sum(part, ns, f32);
            if (tid == 0) step_product_done(S, mode, v);
        }
        __syncthreads();
        --left;
        if (!S.upd) break;   // breakdown
        const T alpha = (T)S.alpha;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            x[k] = fma_b<T>(alpha, d[k], x[k]);
            r[k] = fma_b<T>(-alpha, q[k], r[k]);
            const double p = sizeof(T) == 4 ? wave_dot32(f32, (float)r[k], (float)r[k])
                                            : wave_dot((double)r[k], (double)r[k]);
            if (lane == 0) part[W + k * kWgWaves] = p;
        }
        __syncthreads();
        if (W == 0) {
            const double g = wg_sum(part, ns, f32);
            if (tid == 0) step_update_done(S, hold, g);
        }
        __syncthreads();
        const int due = S.snap_mask;   // run-ahead: candidates first crossed here
        if (due) {
            for (int t = 0; t < kNumEps; ++t)
                if ((due >> t) & 1)
                    for (int k = 0; k < R; ++k)
                        if (W + k * kWgWaves < ns)
                            a.snap32[(size_t)t * ((size_t)a.max_slices * 64) + row0 + own + k * kWgThreads] =
                                (float)x[k];
            __syncthreads();
            if (tid == 0) S.snap_mask = 0;
        }
        if (S.mode != mode || left == 0) break;
    }
    T *dn = (S.ph_it & 1) ? dA : dB;   // the next step's previous direction
#pragma unroll
    for (int k = 0; k < R; ++k)
        if (W + k * kWgWaves < ns) {
            const int row = row0 + tid + k * kWgThreads;
            xg[row] = x[k];
            rg[row] = r[k];
            dn[row] = d[k];
        }
    __syncthreads();
}

// The restart's or the final check's residual.
template <int R>
__device__ inline void wg_residual(const BArena &a, BSys &S, double *s_d, double *part)
{
    const int tid = threadIdx.x, lane = tid & 63, W = tid >> 6;
    const int ns = S.nslices, row0 = S.row0, mode = S.mode;
    const bool restart = mode == kRestart;
    const int src = restart ? S.src : (int)kSrcX64;
    const float *xs = src == kSrcSnap ? a.snap32 + (size_t)S.snap_ci * ((size_t)a.max_slices * 64) : a.x32;
    for (int k = 0; k < R; ++k) {
        if (W + k * kWgWaves >= ns) break;
        const int i = tid + k * kWgThreads;
        const double xv = src == kSrcX64 ? a.x64[row0 + i] : src == kSrcZero ? 0.0 : (double)xs[row0 + i];
        s_d[i] = xv;
        if (restart) a.x64[row0 + i] = xv;
    }
    __syncthreads();
    for (int k = 0; k < R; ++k) {
        if (W + k * kWgWaves >= ns) break;
        const int row = row0 + tid + k * kWgThreads;
        const int64_t at = S.entry0 + a.slice_off[row >> 6] + lane;
        const double acc = wg_entries<double>(a.col + at, a.v64 + at, s_d, row0, 0, a.rowlen[row], 0.0);
        const double res = a.b64[row] - acc;
        if (restart) a.r64[row] = res;
        const double p = wave_dot(res, res);
        if (lane == 0) part[W + k * kWgWaves] = p;
    }
    __syncthreads();
    if (W == 0) {
        const double v = wg_sum(part, ns, false);
        if (tid == 0) step_product_done(S, mode, v);
    }
    __syncthreads();
}

}  // namespace

// R rows a thread; of each row E32 entries in registers in FP32, E64 in FP64.
template <int R, int E32, int E64, int WAVES>
__global__ void __launch_bounds__(kWgThreads, WAVES) k_b_wg(BArena a, int32_t steps)
{
    __shared__ BSys S;
    __shared__ double s_d[R * kWgThreads + 1], part[64];
    if ((int)blockIdx.x >= a.step_cnt[1]) return;
    constexpr int kWords = (int)(sizeof(BSys) / 4);
    static_assert(kWords <= kWgThreads, "one word a thread");
    uint32_t *g = reinterpret_cast<uint32_t *>(a.sys + a.step_sys[blockIdx.x]);
    uint32_t *l = reinterpret_cast<uint32_t *>(&S);
    const int tid = threadIdx.x, W = tid >> 6;
    if (tid < kWords) l[tid] = g[tid];
    __syncthreads();
    const bool hold = a.step_cnt[1] > a.hold_above;
    const int due = S.snap_mask;
    if (due) {   // left by a step of the other form
        for (int t = 0; t < kNumEps; ++t)
            if ((due >> t) & 1)
                for (int k = 0; k < R; ++k)
                    if (W + k * kWgWaves < S.nslices) {
                        const int row = S.row0 + tid + k * kWgThreads;
                        a.snap32[(size_t)t * ((size_t)a.max_slices * 64) + row] = a.x32[row];
                    }
        __syncthreads();
        if (tid == 0) S.snap_mask = 0;
        __syncthreads();
    }
    int left = steps;
    while (left > 0) {
        const int mode = S.mode;
        if (mode == kCg32)
            wg_cg<float, R, E32>(a, S, a.v32, a.x32, a.r32, a.dA32, a.dB32, reinterpret_cast<float *>(s_d), part, left,
                                 hold);
        else if (mode == kCg64)
            wg_cg<double, R, E64>(a, S, a.v64, a.x64, a.r64, a.dA64, a.dB64, s_d, part, left, hold);
        else if (mode == kRestart || mode == kResid) {
            wg_residual<R>(a, S, s_d, part);
            --left;
        } else break;
    }
    // the fields of the recurrence only: those of the 2BFS belong to another stream
    constexpr int kFrom = (int)(offsetof(BSys, mode) / 4), kTo = (int)(offsetof(BSys, bfs_mode) / 4);
    if (tid >= kFrom && tid < kTo) g[tid] = l[tid];
}

// The list's largest system gives the rows per thread: one row leaves room for
// two workgroups a CU (64 registers), which hide each other's barriers.
void launch_wg_steps(hipStream_t s, const BArena &a, int32_t nsys, int32_t max_slices, int32_t steps)
{
    if (nsys <= 0) return;
    if (max_slices <= kWgWaves)
        hipLaunchKernelGGL((k_b_wg<1, 16, 8, 8>), dim3(nsys), dim3(kWgThreads), 0, s, a, steps);
    else if (max_slices <= 2 * kWgWaves)
        hipLaunchKernelGGL((k_b_wg<2, 12, 8, 4>), dim3(nsys), dim3(kWgThreads), 0, s, a, steps);
    else
        hipLaunchKernelGGL((k_b_wg<4, 5, 4, 4>), dim3(nsys), dim3(kWgThreads), 0, s, a, steps);
}

}  // namespace batch
}  // namespace mpcg
