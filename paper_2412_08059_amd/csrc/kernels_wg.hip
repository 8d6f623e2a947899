// CG iterations of a small system in one workgroup (gfx950).
//
// Up to a few thousand rows an iteration's arithmetic takes well under a
// microsecond of the chip, and the two launches of the general path cost about
// 10 us: the gap between dependent launches, and in each a chain of loads
// through the caches (stop flag and partials, then the vectors).  Here one
// workgroup keeps the matrix and x, r and d of its rows in registers, d also in
// LDS for the gathers, and runs `iters` iterations per launch.
//
// Thread T owns rows T + 1024 k, k < R, with at most E entries each.  An entry
// past a row's length is -0.0 times an LDS element that holds +0.0: its product
// -0.0 leaves any sum as it is, so the row chains need no guard.
//
// The bits are those of the general path, whose sums are partials over blocks
// of rows added in a fixed order: a product block sums 256 consecutive rows (a
// term per thread, the waves in order), an update block 1,024 of them as
// chains of four 256 apart.  The scalars (delta and alpha; rho, the stop test
// and beta) are formed by the first wave and handed round through LDS: done by
// all sixteen, the divisions and square roots alone took longer than the
// product.
//
// Between launches the phase's state is the general path's (x without its
// last update, the previous direction in the buffer of its parity, the scalars
// of the last iteration), except that up[0] holds the sum of the update's
// partials instead of the partials.
//
// What bounds it: the five barriers and what one wave does between them
// (1,024 rows of 5 entries: 1.8 us an iteration), then instruction issue of
// the row chains (4,096 rows of 5 entries 3.0 us, 3,375 of 7 5.3 us; two
// launches take 9.5 to 11).

#include "mpcg_internal.hpp"
#include "sell_common.hpp"

#include <cmath>

namespace mpcg {

namespace {
constexpr int kWgThreads = 1024;

template <typename T> struct WgArgs {
    int32_t n, it, it0, iters, grid;   // grid: product blocks (partial slots)
    WalkTab walk;
    const int32_t *rp, *col;           // CSR
    const double *val;
    T *x, *r, *dA, *dB, *snap;
    double *up;
    DevState *st;
};

// What the first wave hands round.
struct WgShared {
    double alpha, beta, rho;
    int32_t stop;          // 1: the recurrence ends here
    uint32_t cross;        // run-ahead candidates first crossed here
};

// Wave sums of R values per lane, in butterfly order.  R = 4: value k in the
// lanes 16 k .. 16 k + 15; R = 2: in the lanes 32 k .. 32 k + 31.  A swap of
// two values' halves adds both with one addition.
template <int STEP> __device__ inline double swap_add(double a, double b)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, a), v = __builtin_bit_cast(uint64_t, b);
    uint32_t lo[2], hi[2];
    if (STEP == 32) {
        const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)v, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(v >> 32), false, false);
        lo[0] = l[0]; lo[1] = l[1]; hi[0] = h[0]; hi[1] = h[1];
    } else {
        const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)v, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(v >> 32), false, false);
        lo[0] = l[0]; lo[1] = l[1]; hi[0] = h[0]; hi[1] = h[1];
    }
    return __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) +
           __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
}
template <int R> __device__ inline double wave_sums(const double (&v)[R])
{
    double s;
    if (R == 4) {
        s = swap_add<16>(swap_add<32>(v[0], v[R > 2 ? 2 : 0]), swap_add<32>(v[R > 1 ? 1 : 0], v[R > 3 ? 3 : 0]));
    } else if (R == 2) {
        s = lane_add<16>(swap_add<32>(v[0], v[R > 1 ? 1 : 0]));
    } else {
        s = lane_add<16>(lane_add<32>(v[0]));
    }
    s = lane_add<8>(s);
    s = lane_add<4>(s);
    s = lane_add<2>(s);
    return lane_add<1>(s);
}

// Sum of the first wave's lanes 0 .. 15 (the others hold zeros, whose
// additions change nothing), in every lane.
__device__ inline double sum16(double s)
{
    s = lane_add<8>(s);
    s = lane_add<4>(s);
    s = lane_add<2>(s);
    s = lane_add<1>(s);
    const uint64_t u = __builtin_bit_cast(uint64_t, s);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)u);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
    return 0.0 + __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
}  // namespace

template <typename T, int R, int E>
__global__ void __launch_bounds__(kWgThreads) k_wg_cg(WgArgs<T> a)
{
    static_assert(R == 1 || R == 2 || R == 4, "rows per thread");
    constexpr int kRows = R * kWgThreads;
    __shared__ T s_d[kRows + 1], s_r[kRows];   // the direction (and a zero), the new residual
    __shared__ double s_pp[16 * R], s_pu[4 * R];
    __shared__ WgShared sh;
    DevState *st = a.st;
    const int tid = threadIdx.x, lane = tid & 63, W = tid >> 6, n = a.n;
    if (st->stop_it < a.it) return;

    T x[R], r[R], dl[R], mv[R][E];
    uint32_t mi[R][(E + 1) / 2];   // LDS byte addresses of the columns, two per register
    {
        const T *dold = (a.it & 1) ? a.dB : a.dA;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int row = tid + k * kWgThreads, i = min(row, n - 1);
            x[k] = a.x[i];
            r[k] = a.r[i];
            dl[k] = dold[i];
            const int lo = a.rp[i], len = row < n ? a.rp[i + 1] - lo : 0;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const bool in = e < len;
                const int at = in ? lo + e : lo;
                mv[k][e] = in ? (T)a.val[at] : T(-0.0);
                const uint32_t b = (uint32_t)(in ? a.col[at] : kRows) * (uint32_t)sizeof(T);
                if (e & 1) mi[k][e / 2] |= b << 16;
                else mi[k][e / 2] = b;
            }
        }
    }
    if (tid == 0) s_d[kRows] = T(0);

    // the first wave's scalars
    const int pv = (a.it - 1) & 1;
    double gp = st->gr[pv], rhop = st->gam[pv];
    const double thr = st->thr;
    const int32_t maxit = st->maxit, k0rec = st->k0rec, spec_k0 = st->spec_k0;
    const bool spec = a.snap && st->spec_on;
    double rho = a.it == a.it0 ? st->gam[a.it & 1] : a.up[0];
    uint32_t crossed = 0;
    if (spec)
        for (int k = 0; k < kNumEps; ++k)
            if (st->cross_iter[k] >= 0) crossed |= 1u << k;
    T alpha_prev = (T)st->alph[pv];
    const bool xdone0 = st->x_it == a.it;   // x already holds x_it

    // r, x and the direction of iteration it - 1 (it with next_dir)
    auto store = [&](int it, bool next_dir, int own) {
        T *db = ((it + next_dir) & 1) ? a.dB : a.dA;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int row = own + k * kWgThreads;
            if (row < n) {
                a.x[row] = x[k];
                a.r[row] = r[k];
                db[row] = dl[k];
            }
        }
    };
    // rho_it, the stop test and beta_it (first wave), it > it0
    auto head = [&](int it) {
        const bool conv = sqrt(rho) <= thr;
        const bool cap = !conv && it >= maxit;
        uint32_t cross = 0;
        if (spec && it >= spec_k0) {
            const double rg = sqrt(rho);
            for (int k = 0; k < kNumEps; ++k)
                if (!((crossed >> k) & 1) && rg <= st->spec_thr[k]) cross |= 1u << k;
            crossed |= cross;
        }
        if (tid != 0) return;
        sh.beta = (double)(T)(rho / rhop);
        sh.stop = conv || cap;
        sh.cross = cross;
        st->gam[it & 1] = rho;
        st->gr[it & 1] = rho;
        const int k = it - 1;
        if (k < k0rec && k < kK0Max) st->ratios[k] = sqrt(rho) / sqrt(gp);
        for (int j = 0; j < kNumEps; ++j)
            if ((cross >> j) & 1) {
                st->cross_iter[j] = it;
                st->cross_gamma[j] = rho;
            }
        if (conv || cap) {
            st->gamma = rho;
            st->iter = it;
            st->reason = conv ? kConverged : kMaxit;
            st->stop_it = it;
            st->live = 0;
            a.up[0] = rho;   // a resumed phase starts from it
        }
    };
    if (W == 0 && a.it != a.it0) head(a.it);
    __syncthreads();

    int it = a.it;
    const int it_end = a.it + a.iters;
#pragma clang loop unroll(disable)
    for (; it < it_end; ++it) {
        T beta = T(0);
        // opaque per iteration: addresses are formed where they are used, not
        // kept in registers (and spilled) across the loop
        int own = tid;
        asm volatile("" : "+v"(own));
        if (it != a.it0) {
            beta = (T)sh.beta;
            const uint32_t cross = sh.cross;
            if (!(it == a.it && xdone0)) {
#pragma unroll
                for (int k = 0; k < R; ++k) x[k] = fma_t<T>(alpha_prev, dl[k], x[k]);
            }
            if (cross)
                for (int j = 0; j < kNumEps; ++j)
                    if ((cross >> j) & 1)
                        for (int k = 0; k < R; ++k)
                            if (own + k * kWgThreads < n) a.snap[(size_t)j * n + own + k * kWgThreads] = x[k];
            if (sh.stop) {
                store(it, false, own);
                return;
            }
        }
        // d = r + beta d_old
#pragma unroll
        for (int k = 0; k < R; ++k) {
            dl[k] = fma_t<T>(beta, dl[k], r[k]);
            s_d[own + k * kWgThreads] = dl[k];
        }
        __syncthreads();
        // q = A d, d.q
        T q[R];
        double pq[R];
#pragma unroll
        for (int k = 0; k < R; ++k) {
            T acc = T(0);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const uint32_t b = (e & 1) ? mi[k][e / 2] >> 16 : mi[k][e / 2] & 0xffffu;
                acc = fma_t<T>(mv[k][e], *reinterpret_cast<const T *>(reinterpret_cast<const char *>(s_d) + b), acc);
            }
            q[k] = acc;
            pq[k] = own + k * kWgThreads < n ? fma((double)dl[k], (double)acc, 0.0) : 0.0;
        }
        const double ws = wave_sums<R>(pq);
        if ((lane & (64 / R - 1)) == 0) s_pp[16 * (lane / (64 / R)) + W] = ws;
        __syncthreads();
        if (W == 0) {   // block sums at the lane of their slot, then the slots' sum
            double s = 0.0;
            if (lane < a.grid) {
                const int g = a.walk.first[lane % kNumXcd] + lane / kNumXcd;   // 256 rows: four wave sums
#pragma unroll
                for (int w = 0; w < 4; ++w) s += s_pp[4 * g + w];
            }
            const double delta = sum16(s);
            const bool bad = !isfinite(delta) || !(delta > 0.0);
            const T alpha = (T)(rho / delta);
            if (tid == 0) {
                sh.alpha = (double)alpha;
                sh.stop = bad;
                st->delta = delta;
                if (bad) {
                    st->gamma = it == a.it0 ? st->gr[it & 1] : rho;
                    st->iter = it;
                    st->reason = isfinite(delta) ? kNotSpd : kNonFinite;
                    st->stop_it = it;
                    st->live = 0;
                } else {
                    st->alpha = (double)alpha;
                    st->alph[it & 1] = (double)alpha;
                }
            }
        }
        __syncthreads();
        if (sh.stop) {
            store(it, true, own);
            return;
        }
        const T alpha = (T)sh.alpha;
        alpha_prev = alpha;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            r[k] = fma_t<T>(-alpha, q[k], r[k]);
            s_r[own + k * kWgThreads] = r[k];
        }
        __syncthreads();
        if (tid < R * kBlock) {   // thread (c, t): rows 1024 c + t + 256 j in a chain
            const int row = (tid / kBlock) * kWgThreads + tid % kBlock;
            double s2 = 0.0;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (row + j * kBlock < n) {
                    const T rn = s_r[row + j * kBlock];
                    s2 = fma((double)rn, (double)rn, s2);
                }
            s2 = wave_sum_all(s2);
            if (lane == 0) s_pu[W] = s2;
        }
        __syncthreads();
        if (W == 0) {
            double s = 0.0;
            if (lane < R && lane * kWgThreads < n) {
#pragma unroll
                for (int w = 0; w < 4; ++w) s += s_pu[4 * lane + w];
            }
            gp = rho;
            rhop = rho;
            rho = sum16(s);
            if (it + 1 < it_end) head(it + 1);
        }
        __syncthreads();
    }
    store(it, false, tid);
    if (tid == 0) a.up[0] = rho;
}

template <typename T, int R, int E> static void wg_go(hipStream_t s, const WgArgs<T> &a)
{
    hipLaunchKernelGGL((k_wg_cg<T, R, E>), dim3(1), dim3(kWgThreads), 0, s, a);
}

// Rows and entries that some instance holds: 4 rows of 7 entries a thread (28
// values), 2 of 17, 1 of 32.  Solves against two launches an iteration, us:
// 64^2 grid 2,440 -> 770, 32^2 1,200 -> 350, 15^3 2,090 -> 1,110, 1,000-row band
// of 17 entries 2,530 -> 650, 1,000-row random graph 710 -> 310.  With the
// matrix streamed from the L2 instead (any n up to 4,096) the same band took
// 3,400 and the graph 980: what does not fit the registers stays with the two
// launches.
bool wg_fits(int64_t n, int32_t max_row)
{
    return (n <= 4 * kWgThreads && max_row <= 7) || (n <= 2 * kWgThreads && max_row <= 17) ||
           (n <= kWgThreads && max_row <= 32);
}

template <typename T>
void launch_wg_cg(hipStream_t s, const int32_t *rp, const int32_t *col, const double *val, int32_t n, int32_t max_row,
                  int grid, T *x, T *r, T *dA, T *dB, T *snap, double *up, int it, int it0, int iters, DevState *st)
{
    WgArgs<T> a{};
    a.n = n; a.it = it; a.it0 = it0; a.iters = iters; a.grid = grid;
    a.walk = walk_tab((n + 63) / 64, grid);
    a.rp = rp; a.col = col; a.val = val;
    a.x = x; a.r = r; a.dA = dA; a.dB = dB; a.snap = snap; a.up = up; a.st = st;
    if (n <= kWgThreads) {
        if (max_row <= 7) wg_go<T, 1, 7>(s, a);
        else if (max_row <= 17) wg_go<T, 1, 17>(s, a);
        else wg_go<T, 1, 32>(s, a);
    } else if (n <= 2 * kWgThreads) {
        if (max_row <= 7) wg_go<T, 2, 7>(s, a);
        else wg_go<T, 2, 17>(s, a);
    } else {
        if (max_row <= 5) wg_go<T, 4, 5>(s, a);
        else wg_go<T, 4, 7>(s, a);
    }
}

template void launch_wg_cg<float>(hipStream_t, const int32_t *, const int32_t *, const double *, int32_t, int32_t, int,
                                  float *, float *, float *, float *, float *, double *, int, int, int, DevState *);
template void launch_wg_cg<double>(hipStream_t, const int32_t *, const int32_t *, const double *, int32_t, int32_t, int,
                                   double *, double *, double *, double *, double *, double *, int, int, int,
                                   DevState *);

}  // namespace mpcg
