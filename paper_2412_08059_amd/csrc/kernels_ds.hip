// Diagonal storage: the matrix as its main and upper diagonals (gfx950,
// wave64), for symmetric matrices whose entries lie on few diagonals (grids
// and bands: at most kDsMax distances |i - j| > 0).
//
// Plane 0 holds a_ii, plane j the entries a_{i, i + d_j}; an entry that the
// pattern does not have is a NaN (stored values are finite, so the NaN says
// "absent" without a mask).  The lower entry a_{i, i - d_j} is the upper
// entry of row i - d_j, so a product reads
//   main and upper planes  once, straight through, and
//   the lower entries      from lines of the same planes that the rows d_j
//                          earlier have just brought into the L2,
// and no column indices and no row lengths at all: (nh + 1) values per row
// where SELL-64 moves 2 nh + 1 values, as many 16-bit columns and a row
// pointer (7-point stencil in FP64: 32 instead of 74 bytes a row; FP32 16
// instead of 46).  Every address follows from the row alone, so all loads of
// a slice are independent of each other.
//
// Each lane walks its row's diagonals from the lowest to the highest, which
// is CSR order, with one fma chain starting from 0 and absent entries
// skipped: the bits of the SELL and CSR kernels.  Blocks walk the same slice
// groups as there and leave partials of the same rows.
//
// What bounds it: the bytes above plus the vectors (gathers of r and d hit
// the L2).  One FP64 CG product on the 128^3 stencil needs 168 MB instead of
// 255 MB (counted: 170 MB read and 50 MB written; rows a plane of the grid apart
// are not always in the same XCD's L2 any more).

#include "jacobi_common.hpp"

#include <cmath>
#include <type_traits>

namespace mpcg {

// ------------------------------------------------------------- ingest --

// Sampled offsets (one block): the distances |i - j| > 0 of kDsSample rows
// spread over the matrix, a thread per entry.  Up to 63 they are bits of a
// mask, beyond that slots claimed by compare-and-swap.  The upper entries' mirror
// images have been looked up by blocks of k_ingest_rows (the dependent loads took
// 6 us here, of a 2M-row band's 0.37 ms): a matrix that is symmetric only to
// rounding is then not a candidate.  Other distances than the sampled ones, or an
// unequal pair outside the sample, are found out by k_ds_rows, which costs a
// second ingest but no result (7-point stencil, 49^3 rows 0.08 ms, 128^3 0.27).
struct DsSample {
    unsigned long long near;      // bit d: distance d
    int32_t far[kDsMax], misfit;
};

__device__ inline void ds_sample(int lo, int hi, int64_t i, const int32_t *col, int32_t n, int64_t nnz, int64_t cap,
                                 int ds, DevState *st, DsSample *sm)
{
    // (lo, hi): the sampled row's entries, none for a thread without a row
    const int j = threadIdx.x % kDsRowMax;
    if (hi - lo > kDsRowMax) sm->misfit = 1;
    if (lo + j < hi) {
        const int32_t c = col[lo + j];
        const int64_t diff = (int64_t)c - i;
        const int64_t d = diff < 0 ? -diff : diff;
        if (d > 0 && d < 64) {
            atomicOr(&sm->near, 1ull << d);
        } else if (d >= 64 && d < n) {   // a column out of range is found by the entries' pass
            int t = 0;
            for (; t < kDsMax; ++t) {   // plain reads first: a taken slot keeps its distance
                int old = *(volatile int32_t *)&sm->far[t];
                if (old == 0) old = atomicCAS(&sm->far[t], 0, (int)d);
                if (old == 0 || old == (int)d) break;
            }
            if (t == kDsMax) sm->misfit = 1;
        }
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    const int nnear = __popcll(sm->near);
    int nh = nnear, nfar = 0;
    while (nfar < kDsMax && sm->far[nfar]) ++nfar;
    nh += nfar;
    if (sm->misfit || nh > kDsMax) {
        st->ds_many = 1;
        return;
    }
    if (!ds || nh == 0) return;
    // Worth it when at least two thirds of the diagonals' places hold an
    // entry: each place costs a gather whether or not it does.
    if ((int64_t)(2 * nh + 1) * n * 2 > 3 * nnz || (int64_t)(nh + 1) * ds_stride(n) > cap) return;
    if (n >= (1 << 28) || (int64_t)(nh + 1) * ds_stride(n) * 8 >= (1ll << 32)) return;   // 32-bit byte offsets
    unsigned long long m = sm->near;
    for (int t = 0; t < nnear; ++t, m &= m - 1) st->ds_d[t] = __builtin_ctzll(m);
    int prev = 0;
    for (int t = nnear; t < nh; ++t) {   // the far ones, ascending
        int next = kNoStop;
        for (int k = 0; k < nfar; ++k)
            if (sm->far[k] > prev && sm->far[k] < next) next = sm->far[k];
        st->ds_d[t] = next;
        prev = next;
    }
    st->ds_nh = nh;
    st->ds_cand = 1;
}

// One block after k_ingest_rows: clears the device state, folds the blocks'
// statistics into it, samples the distances (if the row pointers are usable;
// for diagonal storage if ds), and unless diagonal storage takes the matrix
// forms the SELL slice offsets (exclusive scan of the padded slice sizes).
__global__ void __launch_bounds__(1024)
k_ingest_fold(const int32_t *blk, int32_t nblk, const int32_t *rp, const int32_t *col, int32_t n, int64_t nnz,
              const int64_t *wid, int64_t *off, int64_t cap, int ds, DevState *st)
{
    __shared__ int32_t fold[3][1024 / 64];
    __shared__ int64_t part[1024 / 64];
    __shared__ DsSample smp;
    __shared__ int32_t cand;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    for (int i = t; i < (int)(sizeof(DevState) / sizeof(int32_t)); i += 1024) reinterpret_cast<int32_t *>(st)[i] = 0;
    // the sampled row's pointers, loaded beside the statistics
    const int r = t / kDsRowMax;
    const int64_t row = ds_sample_row(r, n);
    const bool has = r < kDsSample && row < n;
    const int rlo = has ? rp[row] : 0, rhi = has ? rp[row + 1] : 0;
    int unequal = 0;   // with ds: some sampled entry has no equal mirror image
    for (int k = 0; k < kDsMirrorBlocks; ++k) unequal |= blk[3 * nblk + k];
    int e = 0, l = 0, bd = 0;
    for (int i = t; i < nblk; i += 1024) {
        e |= blk[3 * i];
        l = l > blk[3 * i + 1] ? l : blk[3 * i + 1];
        bd = bd > blk[3 * i + 2] ? bd : blk[3 * i + 2];
    }
    auto larger = [](int x, int y) { return x > y ? x : y; };
    e = wave_fold(e, [](int x, int y) { return x | y; });
    l = wave_fold(l, larger);
    bd = wave_fold(bd, larger);
    if (lane == 0) {
        fold[0][w] = e;
        fold[1][w] = l;
        fold[2][w] = bd;
    }
    if (t == 0) smp.near = 0;
    if (t < kDsMax) smp.far[t] = 0;
    if (t == kDsMax) smp.misfit = 0;
    __syncthreads();
    for (int k = 0; k < 1024 / 64; ++k) {
        e |= fold[0][k];
        l = larger(l, fold[1][k]);
        bd = larger(bd, fold[2][k]);
    }
    if (t == 0) {
        st->ing_err = e;
        st->max_row = l;
        st->max_band = bd;
    }
    // a row with more entries than kDsMax distances can give is not diagonal
    // storage's, sampled or not
    if (l > kDsRowMax || unequal) ds = 0;
    if (!(e & kErrRowPtr)) ds_sample(rlo, rhi, row, col, n, nnz, cap, ds, st, &smp);   // else ds_cand is 0
    if (t == 0) cand = st->ds_cand;
    __syncthreads();
    if (cand) return;
    // per thread a run of slices; the runs' sums scanned in the waves and over them
    const int nsl = (n + 63) / 64, per = (nsl + 1023) / 1024;
    const int a = min(t * per, nsl), b = min(a + per, nsl);
    int64_t sum = 0;
    for (int i = a; i < b; ++i) sum += wid[i];
    int64_t inc = sum;
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t v = __shfl_up(inc, o, 64);
        if (lane >= o) inc += v;
    }
    if (lane == 63) part[w] = inc;
    __syncthreads();
    int64_t run = inc - sum;
    for (int k = 0; k < w; ++k) run += part[k];
    for (int i = a; i < b; ++i) {
        off[i] = run;
        run += wid[i];
    }
    if (t == 1023) {
        off[nsl] = run;
        st->sell_total = run;
    }
}

void launch_ingest_fold(hipStream_t s, const int32_t *blk, const int32_t *rp, const int32_t *col, int32_t n, int64_t nnz,
                        const int64_t *wid, int64_t *off, int64_t cap, int ds, DevState *st)
{
    hipLaunchKernelGGL(k_ingest_fold, dim3(1), dim3(1024), 0, s, blk, (n + kBlock - 1) / kBlock, rp, col, n, nnz,
                       wid, off, cap, ds, st);
}

constexpr int kDsNear = 32;   // largest distance of the kernels that keep a slice's vector elements in LDS

// The entries of rows r .. r + nrows - 1 (cnt of them, from lo) into a wave's LDS.
__device__ inline void ds_stage(const int32_t *__restrict__ col, const double *__restrict__ val, int lo, int cnt,
                                int32_t *sc, double *sv)
{
    const int lane = threadIdx.x & 63;
    for (int k0 = 0; k0 < cnt; k0 += 256) {
        int c[4];
        double v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = k0 + j * 64 + lane;
            if (k < cnt) {
                c[j] = col[lo + k];
                v[j] = val[lo + k];
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = k0 + j * 64 + lane;
            if (k < cnt) {
                sc[k] = c[j];
                sv[k] = v[j];
            }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// One slice of a near matrix: the planes and the check of its lower entries in
// one pass.  A lower entry's partner row is in the slice or one of the `reach`
// rows before it, whose upper entries the first lanes pick up beforehand (the
// slice before reads the same lines); the slice's and these rows' upper entries
// then meet in LDS.
__device__ inline void ds_near_slice(const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
                                     const double *__restrict__ val, int32_t n, int r0, const int32_t (&d)[kDsMax],
                                     int nh, int64_t S, double *p64, float *p32, double *dg64, float *dg32, int32_t *sc,
                                     double *sv, int &miss, int &err)
{
    const int lane = threadIdx.x & 63;
    const int reach = d[nh - 1], nrows = min(64, n - r0), row = r0 + lane;
    // slice 0 has no rows before it
    const int nbefore = r0 ? reach : 0, h0 = r0 - nbefore;
    const int hs = rp[h0 + min(lane, nbefore)], he = rp[h0 + min(lane + 1, nbefore)];
    const int ps = rp[r0 + min(lane, nrows)], pe = rp[r0 + min(lane + 1, nrows)];
    const int hlo = rp[h0], lo = rp[r0], hi = rp[r0 + nrows];
    if (lo - hlo > 64 * kDsRowMax || hi - lo > 64 * kDsRowMax) {   // a row too long to match
        miss = 1;
        return;
    }
    double before[kDsMax], low[kDsMax], up[kDsMax];
    ds_stage(col, val, hlo, lo - hlo, sc, sv);
    {
        const int hr = h0 + lane;
        int k = hs - hlo;
        const int ke = he - hlo;
        while (k < ke && sc[k] <= hr) ++k;
#pragma unroll
        for (int t = 0; t < kDsMax; ++t) {
            before[t] = NAN;
            if (t < nh && k < ke && sc[k] == hr + d[t]) before[t] = sv[k++];
        }
    }
    __builtin_amdgcn_wave_barrier();
    ds_stage(col, val, lo, hi - lo, sc, sv);
    int k = ps - lo;
    const int ke = pe - lo;
    auto take = [&](int c) {   // the next entry if it is column c
        if (k >= ke || sc[k] != c) return (double)NAN;
        const double v = sv[k++];
        if (!isfinite(v)) err |= kErrNonFiniteA;
        return v;
    };
#pragma unroll
    for (int t = kDsMax - 1; t >= 0; --t) low[t] = t < nh ? take(row - d[t]) : NAN;
    const double mid = take(row);
#pragma unroll
    for (int t = 0; t < kDsMax; ++t) up[t] = t < nh ? take(row + d[t]) : NAN;
    if (k != ke) miss = 1;
    if (row < n) {
        p64[row] = mid;
        if (p32) p32[row] = (float)mid;
        if (dg64) {
            const double dv = mid == mid ? mid : 0.0;
            dg64[row] = dv;
            dg32[row] = (float)dv;
            if (!(dv > 0.0) || !isfinite(dv) || !((float)dv > 0.0f) || !isfinite((float)dv)) err |= kErrDiag;
        }
#pragma unroll
        for (int t = 0; t < kDsMax; ++t)
            if (t < nh) {
                p64[(t + 1) * S + row] = up[t];
                if (p32) p32[(t + 1) * S + row] = (float)up[t];
            }
    }
    __builtin_amdgcn_wave_barrier();
    constexpr int kMeet = 64 + kDsNear;
    static_assert(kDsMax * kMeet <= 64 * kDsRowMax, "the upper entries take the staged entries' place");
#pragma unroll
    for (int t = 0; t < kDsMax; ++t) {
        if (lane < reach) sv[t * kMeet + lane] = r0 ? before[t] : NAN;
        sv[t * kMeet + reach + lane] = up[t];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < kDsMax; ++t) {
        if (t >= nh) continue;
        const double u = sv[t * kMeet + reach + lane - d[t]];
        const bool here = low[t] == low[t], there = u == u;
        if (here != there || (here && __double_as_longlong(u) != __double_as_longlong(low[t]))) miss = 1;
    }
    __builtin_amdgcn_wave_barrier();
}

// Wave per 64 rows: the rows' entries are staged in LDS with coalesced loads,
// then each lane walks its row along the diagonals.  VERIFY 0: the planes (and
// diag(A) for Jacobi), values finite, every entry on a sampled diagonal.
// VERIFY 1, after it: every lower entry equals the upper one of its partner
// row, bit for bit, and every upper entry has one (absent = NaN on both
// sides), i.e. the matrix is symmetric.  Near matrices have both in the first
// launch: 2 M-row band of half-width 8, 298 -> 160 us, of which the matrix and
// the planes need 110.
template <int VERIFY>
__global__ void __launch_bounds__(kBlock)
k_ds_rows(const int32_t *__restrict__ rp, const int32_t *__restrict__ col, const double *__restrict__ val,
          int32_t n, int32_t nslices, double *p64, float *p32, double *dg64, float *dg32, DevState *st)
{
    __shared__ int32_t s_col[kBlock / 64][64 * kDsRowMax];
    __shared__ double s_val[kBlock / 64][64 * kDsRowMax];
    if (!st->ds_cand || (VERIFY && st->ds_miss)) return;
    const int nh = st->ds_nh;
    const int64_t S = ds_stride(n);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int32_t *sc = s_col[w];
    double *sv = s_val[w];
    int miss = 0, err = 0;
    const bool near = st->ds_d[nh - 1] <= kDsNear;
    if (VERIFY && near) return;
    int32_t d[kDsMax];
    for (int t = 0; t < kDsMax; ++t) d[t] = t < nh ? st->ds_d[t] : 0;
    for (int s = blockIdx.x * (kBlock / 64) + w; s < nslices; s += gridDim.x * (kBlock / 64)) {
        const int r0 = s * 64;
        if (near) {
            ds_near_slice(rp, col, val, n, r0, d, nh, S, p64, p32, dg64, dg32, sc, sv, miss, err);
            continue;
        }
        const int nrows = min(64, n - r0);
        const int row = r0 + lane;
        const bool has = lane < nrows;
        const int rpl = rp[r0 + min(lane, nrows)];
        const int rph = rp[r0 + min(lane + 1, nrows)];
        const int lo = __builtin_amdgcn_readfirstlane(rpl);
        const int hi = rp[r0 + nrows];
        const int cnt = hi - lo;
        if (cnt > 64 * kDsRowMax) {   // a row too long to match
            miss = 1;
            continue;
        }
        ds_stage(col, val, lo, cnt, sc, sv);
        if (has) {
            int k = rpl - lo;
            const int ke = rph - lo;
            for (int t = -nh; t <= nh; ++t) {
                const int d = t < 0 ? -st->ds_d[-t - 1] : (t > 0 ? st->ds_d[t - 1] : 0);
                const int64_t c = (int64_t)row + d;
                const bool here = k < ke && c >= 0 && c < n && sc[k] == (int)c;
                const double v = here ? sv[k] : NAN;
                k += here;
                if (!VERIFY) {
                    if (here && !isfinite(v)) err |= kErrNonFiniteA;
                    if (t >= 0) {
                        p64[t * S + row] = v;
                        if (p32) p32[t * S + row] = (float)v;
                    }
                    if (t == 0 && dg64) {
                        const double dv = here ? v : 0.0;
                        dg64[row] = dv;
                        dg32[row] = (float)dv;
                        if (!(dv > 0.0) || !isfinite(dv) || !((float)dv > 0.0f) || !isfinite((float)dv)) err |= kErrDiag;
                    }
                } else if (t < 0 && c >= 0) {
                    const double u = p64[(int64_t)(-t) * S + c];
                    const bool there = u == u;
                    if (here != there || (here && __double_as_longlong(u) != __double_as_longlong(v))) miss = 1;
                }
            }
            if (!VERIFY && k != ke) miss = 1;
        }
        __builtin_amdgcn_wave_barrier();
    }
    // upper entries that reach past the last row do not exist (c < n above),
    // so every upper entry's partner row has looked at it
    for (int o = 32; o > 0; o >>= 1) {
        err |= __shfl_xor(err, o, 64);
        miss |= __shfl_xor(miss, o, 64);
    }
    if (lane == 0 && err) atomicOr(&st->ing_err, err);
    if (lane == 0 && miss) atomicOr(&st->ds_miss, 1);
}

void launch_ds_ingest(hipStream_t s, const int32_t *rp, const int32_t *col, const double *val, int32_t n, double *p64,
                      float *p32, double *dg64, float *dg32, DevState *st)
{
    const int nslices = (n + 63) / 64;
    int g = (nslices + kBlock / 64 - 1) / (kBlock / 64);
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL((k_ds_rows<0>), dim3(g), dim3(kBlock), 0, s, rp, col, val, n, nslices, p64, p32, dg64, dg32, st);
    hipLaunchKernelGGL((k_ds_rows<1>), dim3(g), dim3(kBlock), 0, s, rp, col, val, n, nslices, p64, p32, dg64, dg32, st);
}

// -------------------------------------------------------------- products --

enum DsMode { kDsCg = 0, kDsRestart = 1, kDsResid = 2 };

template <typename T>
struct DsArgs {
    const T *p;         // planes
    uint32_t S;         // bytes from one plane to the next
    int32_t d[kDsMax];
    int32_t n, nslices;
    int32_t it, it0, nup, pc;
    WalkTab walk;
    const T *r;
    T *dA, *dB, *q, *x, *snap;
    const double *up;
    double *part;
    DevState *st;
    int32_t *live;      // cleared in host memory when the recurrence has stopped
    // restart, residual
    const float *x32;
    const double *x64in, *b, *dg;
    double *x64out, *rout, *dz, *z;
};

// A vector or plane element at a byte offset below 2^32 (ds_sample keeps the
// planes within it): one scalar base and a 32-bit lane offset, so an address
// costs one addition and no 64-bit pointer per diagonal is kept.
template <typename T> __device__ inline T ds_at(const T *p, uint32_t byte)
{
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(p) + byte);
}

// The row's sum over its diagonals, lowest first: sum of v * g(byte offset of
// the column's vector element).
// EDGE: the slice holds rows whose diagonals leave the matrix (or rows past
// its end); their offsets are clamped into it and the products skipped.
// NEAR: every distance is at most kDsNear, and the slice's 64 + 2 reach
// vector elements lie in `lu` (LDS): each was formed once instead of once per
// diagonal, and a row's loads from memory are its matrix entries alone.
template <int NH, bool EDGE, bool NEAR, bool SKIP_MAIN, typename T, typename G>
__device__ inline T ds_row(const T *p, uint32_t S, const int32_t *d, int32_t n, int32_t row, int lane, const T *lu,
                           const G &g)
{
    constexpr int W = (int)sizeof(T);
    constexpr int CH = NEAR ? (W == 8 ? 9 : 17) : 7;   // diagonals whose loads are issued together
    const int32_t last = (n - 1) * W;
    // The row's offset is opaque to the loop optimiser, which otherwise keeps
    // every diagonal's offset in a register of its own across the slices and
    // spills them (band of half-width 8, FP32 product: 28.5 us instead of 12.8).
    int32_t rb = row * W;
    asm("" : "+v"(rb));
    const int32_t rc = EDGE ? min(rb, last) : rb;
    const T *lr = lu + d[NH - 1] + lane;
    T acc = T(0);
#pragma unroll
    for (int t0 = -NH; t0 <= NH; t0 += CH) {
        T v[CH], u[CH];
        bool ok[CH];
#pragma unroll
        for (int k = 0; k < CH; ++k) {
            const int t = t0 + k;
            if (t > NH || (SKIP_MAIN && t == 0)) continue;
            const int32_t off = t < 0 ? -d[-t - 1] : (t > 0 ? d[t - 1] : 0);
            const int32_t c = rb + off * W;
            const int32_t cc = EDGE ? max(0, min(c, last)) : c;
            ok[k] = !EDGE || c == cc;
            v[k] = ds_at(p, (uint32_t)(t < 0 ? cc : rc) + (uint32_t)(t < 0 ? -t : t) * S);
            u[k] = NEAR ? lr[off] : g((uint32_t)cc);
        }
#pragma unroll
        for (int k = 0; k < CH; ++k) {
            const int t = t0 + k;
            if (t > NH || (SKIP_MAIN && t == 0)) continue;
            const T f = fma_t<T>(v[k], u[k], acc);
            acc = ok[k] && v[k] == v[k] ? f : acc;
        }
    }
    return acc;
}

template <int NH, bool NEAR, bool SKIP_MAIN, typename T, typename G>
__device__ inline T ds_sum(const T *p, uint32_t S, const int32_t *d, int32_t n, int32_t rb, int lane, T *lu, const G &g)
{
    const int32_t reach = d[NH - 1];   // the largest distance
    if (NEAR) {
        // own element, and one of the halo's (lanes of both ends of the wave)
        const int32_t h = lane < reach ? lane - reach : lane + reach;
        const bool halo = lane < reach || lane >= 64 - reach;
        const T own = g((uint32_t)min(rb + lane, n - 1) * (uint32_t)sizeof(T));
        T out = T(0);
        if (halo) out = g((uint32_t)max(0, min(rb + h, n - 1)) * (uint32_t)sizeof(T));
        __builtin_amdgcn_wave_barrier();   // the previous slice's reads are done
        lu[reach + lane] = own;
        if (halo) lu[reach + h] = out;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if (rb >= reach && rb + 63 + reach < n)
        return ds_row<NH, false, NEAR, SKIP_MAIN, T>(p, S, d, n, rb + lane, lane, lu, g);
    return ds_row<NH, true, NEAR, SKIP_MAIN, T>(p, S, d, n, rb + lane, lane, lu, g);
}

// A slice's operands for a CG product, all loaded at once: the matrix, d_old
// and r of the columns (NEAR: of the slice and of its halo, else one per
// diagonal), x of the rows.  LOOP: a wave takes several slices in turn.
template <int NH, bool NEAR, bool LOOP, typename T> struct DsSlice {
    static constexpr int K = 2 * NH + 1, C = NEAR ? 2 : K, OWN = NEAR ? 0 : NH;
    T v[K], d[C], r[C], x;

    __device__ inline void load(const DsArgs<T> &a, const T *dold, int rb, int lane)
    {
        constexpr int W = (int)sizeof(T);
        int32_t row = rb + lane;
        if (LOOP) asm("" : "+v"(row));   // opaque: see ds_row
        const int32_t last = a.n - 1, rc = min(row, last);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int t = k - NH;
            const int32_t c = row + (t < 0 ? -a.d[-t - 1] : (t > 0 ? a.d[t - 1] : 0));
            v[k] = T(NAN);   // no entry
            if (!NEAR) d[k] = r[k] = T(0);
            if (c >= 0 && c <= last) {
                v[k] = ds_at(a.p, (uint32_t)((t < 0 ? c : rc) * W) + (uint32_t)(t < 0 ? -t : t) * a.S);
                if (!NEAR) {
                    d[k] = ds_at(dold, (uint32_t)(c * W));
                    r[k] = ds_at(a.r, (uint32_t)(c * W));
                }
            }
        }
        if (NEAR) {
            const int reach = a.d[NH - 1], h = lane < reach ? lane - reach : lane + reach;
            const uint32_t o = (uint32_t)(rc * W), ho = (uint32_t)(max(0, min(rb + h, last)) * W);
            d[0] = ds_at(dold, o);
            r[0] = ds_at(a.r, o);
            d[C - 1] = ds_at(dold, ho);
            r[C - 1] = ds_at(a.r, ho);
        }
        x = ds_at(a.x, (uint32_t)(rc * W));
    }

    // The row's sum of v * (r + beta d_old).
    __device__ inline T sum(const DsArgs<T> &a, T beta, int lane, T *lu) const
    {
        int at = a.d[NH - 1] + lane;
        if (LOOP) asm("" : "+v"(at));
        if (NEAR) {
            const int reach = a.d[NH - 1], h = lane < reach ? lane - reach : lane + reach;
            if (LOOP) __builtin_amdgcn_wave_barrier();   // the previous slice's reads are done
            lu[reach + lane] = fma_t<T>(beta, d[0], r[0]);
            if (lane < reach || lane >= 64 - reach) lu[reach + h] = fma_t<T>(beta, d[C - 1], r[C - 1]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        T acc = T(0);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int t = k - NH;
            const int32_t off = t < 0 ? -a.d[-t - 1] : (t > 0 ? a.d[t - 1] : 0);
            const T u = NEAR ? lu[at + off] : fma_t<T>(beta, d[NEAR ? 0 : k], r[NEAR ? 0 : k]);
            const T f = fma_t<T>(v[k], u, acc);
            acc = v[k] == v[k] ? f : acc;
        }
        return acc;
    }
};

// How a wave takes its slices: one after the other, their diagonals loaded as
// they are walked (kDsWalk); or each loaded whole, the first before the
// iteration's scalars are known: its only slice (kDsOne), or several (kDsLoop).
enum DsPre { kDsWalk = 0, kDsOne = 1, kDsLoop = 2 };

template <int MODE, typename T, int NH, bool NEAR, int PRE>
__global__ void __launch_bounds__(kBlock, PRE == kDsWalk ? 8 : PRE == kDsOne ? 4 : 5)
__attribute__((amdgpu_num_sgpr(kSgprCap))) k_ds(DsArgs<T> a)
{
    static_assert(PRE == kDsWalk || MODE == kDsCg, "the products of a phase");
    constexpr int NV = MODE == kDsRestart ? 3 : 1;
    __shared__ double sm[kBlock / 64];
    __shared__ T s_u[kBlock / 64][NEAR ? 64 + 2 * kDsNear : 1];
    DevState *st = a.st;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    T *lu = s_u[wv];

    T beta = T(0), alpha_prev = T(0);
    bool x_pending = false, f32acc = false;
    const T *dold = nullptr;
    T *dnew = nullptr;
    DsSlice<NH, NEAR, PRE == kDsLoop, T> one;
    SliceWalk ow = slice_walk(a.walk);
    int osl = ow.g < ow.g_end ? ow.g * (kBlock / 64) + wv : a.nslices;
    if (PRE && osl < a.nslices) one.load(a, (a.it & 1) ? a.dB : a.dA, osl * 64, lane);
    if (MODE == kDsCg) {
        __shared__ double sm_rho[kBlock / 64], sm_g[kBlock / 64];
        const int it = a.it;
        const CgHead h = cg_head<T>(st, a.up, a.nup, a.pc, it, a.it0, sm_rho, sm_g, a.live);
        if (h.skip) return;
        f32acc = h.f32acc;
        dold = (it & 1) ? a.dB : a.dA;
        dnew = (it & 1) ? a.dA : a.dB;
        if (it != a.it0) {
            alpha_prev = (T)h.alph;
            const bool stop = cg_head_decide(st, h, it, a.live);
            const unsigned cross = a.snap ? spec_crossings(st, it, h.g) : 0u;
            if (stop || cross) {
                // the iterate x_it of this block's rows, then its run-ahead copies
                for (SliceWalk w = slice_walk(a.walk); w.g < w.g_end; w.g += w.step) {
                    const int i = w.g * kBlock + tid;
                    if (i >= a.n) continue;
                    const T xn = h.xdone ? a.x[i] : fma_t<T>(alpha_prev, dold[i], a.x[i]);
                    if (!h.xdone) a.x[i] = xn;
                    for (int t = 0; t < kNumEps; ++t)
                        if (cross & (1u << t)) a.snap[(size_t)t * a.n + i] = xn;
                }
                record_crossings(st, cross, it, h.g);
                if (stop) return;
            } else {
                x_pending = !h.xdone;
            }
            beta = (T)(h.rho / h.rhop);
        }
    }

    double s[NV];
    for (int j = 0; j < NV; ++j) s[j] = 0.0;
    float sf = 0.0f;   // d.q in FP32 (dot_acc = 1)
    if (PRE) {
        while (osl < a.nslices) {
            const int row = osl * 64 + lane;
            const T acc = one.sum(a, beta, lane, lu);
            if (row < a.n) {
                const T dof = one.d[one.OWN];
                if (x_pending) a.x[row] = fma_t<T>(alpha_prev, dof, one.x);
                const T dn = fma_t<T>(beta, dof, one.r[one.OWN]);
                dnew[row] = dn;
                a.q[row] = acc;
                if (f32acc) sf = fmaf((float)dn, (float)acc, sf);
                else s[0] = fma((double)dn, (double)acc, s[0]);
            }
            if (PRE == kDsOne) break;
            ow.g += ow.step;
            if (ow.g >= ow.g_end) break;
            osl = ow.g * (kBlock / 64) + wv;
            if (osl >= a.nslices) break;
            one.load(a, dold, osl * 64, lane);
        }
    } else {
        for (SliceWalk w = slice_walk(a.walk); w.g < w.g_end; w.g += w.step) {
            const int sl = w.g * (kBlock / 64) + wv;
            if (sl >= a.nslices) continue;
            const int rb = sl * 64;
            const int row = rb + lane;
            const bool has = row < a.n;
            T acc;
            if (MODE == kDsCg)
                acc = ds_sum<NH, NEAR, false, T>(a.p, a.S, a.d, a.n, rb, lane, lu,
                                           [&](uint32_t c) { return fma_t<T>(beta, ds_at(dold, c), ds_at(a.r, c)); });
            else if (a.x32)
                acc = ds_sum<NH, NEAR, false, T>(a.p, a.S, a.d, a.n, rb, lane, lu,
                                           [&](uint32_t c) { return (T)ds_at(a.x32, c / 2); });
            else
                acc = ds_sum<NH, NEAR, false, T>(a.p, a.S, a.d, a.n, rb, lane, lu,
                                           [&](uint32_t c) { return (T)ds_at(a.x64in, c); });
            if (!has) continue;
            if (MODE == kDsCg) {
                const T dof = dold[row];
                if (x_pending) a.x[row] = fma_t<T>(alpha_prev, dof, a.x[row]);
                const T dn = fma_t<T>(beta, dof, a.r[row]);
                dnew[row] = dn;
                a.q[row] = acc;
                if (f32acc) sf = fmaf((float)dn, (float)acc, sf);
                else s[0] = fma((double)dn, (double)acc, s[0]);
            } else {
                const double bv = a.b[row];
                const double res = bv - (double)acc;
                if (MODE == kDsRestart) {
                    if (a.x32) a.x64out[row] = (double)a.x32[row];
                    a.rout[row] = res;
                    a.dz[row] = 0.0;
                    s[1 % NV] = fma(bv, bv, s[1 % NV]);
                    double zv = res;
                    if (a.dg) {
                        zv = res / a.dg[row];
                        a.z[row] = zv;
                    }
                    s[2 % NV] = fma(res, zv, s[2 % NV]);
                }
                s[0] = fma(res, res, s[0]);
            }
        }
    }
    if (f32acc) {
        const float bs = sell_block_sum_f(sf, sm);
        if (tid == 0) a.part[blockIdx.x] = (double)bs;
        return;
    }
    for (int j = 0; j < NV; ++j) {
        const double bs = sell_block_sum(s[j], sm);
        if (tid == 0) a.part[(size_t)blockIdx.x * NV + j] = bs;
    }
}

// One Jacobi iteration (see kernels_jacobi.hip): off-diagonal sum, residual
// of the iterate, next iterate; a_ii is plane 0.
template <typename T, int NH, bool NEAR>
__global__ void __launch_bounds__(kBlock, 8) __attribute__((amdgpu_num_sgpr(kSgprCap)))
k_ds_jac(JacArgs<T> a, DsPlanes<T> m)
{
    __shared__ double sm[kBlock / 64], sm_head[kBlock / 64];
    __shared__ T s_u[kBlock / 64][NEAR ? 64 + 2 * kDsNear : 1];
    if (jac_prologue<T>(a, sm_head)) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const T *x = (a.k & 1) ? a.x1 : a.x0;
    T *xn = (a.k & 1) ? a.x0 : a.x1;
    double s2 = 0.0;
    for (SliceWalk w = slice_walk(a.walk); w.g < w.g_end; w.g += w.step) {
        const int sl = w.g * (kBlock / 64) + wv;
        if (sl >= a.nslices) continue;
        const int rb = sl * 64;
        const int row = rb + lane;
        const T acc = ds_sum<NH, NEAR, true, T>(m.p, m.S, m.d, a.n, rb, lane, s_u[wv], [&](uint32_t c) { return ds_at(x, c); });
        if (row >= a.n) continue;
        const T d = m.p[row];
        const T t = a.b[row] - acc;
        const T r = fma_t<T>(-d, x[row], t);
        xn[row] = t / d;
        s2 = fma((double)r, (double)r, s2);
    }
    const double bs = sell_block_sum(s2, sm);
    if (tid == 0) a.part[(size_t)(a.k & 1) * a.np + blockIdx.x] = bs;
}

// f(integral_constant<NH>, bool_constant<NEAR>) for the matrix's distances
template <typename F> static void ds_dispatch(const DsMat &m, const F &f)
{
    const bool near = m.d[m.nh - 1] <= kDsNear;
    auto with = [&](auto nh) {
        if (near) f(nh, std::true_type());
        else f(nh, std::false_type());
    };
    switch (m.nh) {
    case 1: with(std::integral_constant<int, 1>()); break;
    case 2: with(std::integral_constant<int, 2>()); break;
    case 3: with(std::integral_constant<int, 3>()); break;
    case 4: with(std::integral_constant<int, 4>()); break;
    case 5: with(std::integral_constant<int, 5>()); break;
    case 6: with(std::integral_constant<int, 6>()); break;
    case 7: with(std::integral_constant<int, 7>()); break;
    default: with(std::integral_constant<int, 8>()); break;
    }
}

template <typename T> static const T *ds_vals(const DsMat &m);
template <> const float *ds_vals<float>(const DsMat &m) { return m.p32; }
template <> const double *ds_vals<double>(const DsMat &m) { return m.p64; }

template <typename T> static DsArgs<T> ds_args(const DsMat &m, int grid)
{
    DsArgs<T> a{};
    a.p = ds_vals<T>(m);
    a.S = (uint32_t)(ds_stride(m.n) * sizeof(T));
    for (int t = 0; t < kDsMax; ++t) a.d[t] = m.d[t];
    a.n = m.n;
    a.nslices = (m.n + 63) / 64;
    a.walk = walk_tab(a.nslices, grid);
    return a;
}

// Slices are loaded whole in FP64 where their registers leave at least four
// waves on a SIMD: every near matrix, far ones up to three distances.  The
// first slice's loads run beside the partials' and all of a slice's loads are
// in flight at once, which is worth more than the other four waves.  FP64 CG
// product, us before and after: band of half-width 8, n = 100,000 5.9 -> 4.9,
// 500,000 15.8 -> 11.9, 2 M 45.1 -> 34.2; 7-point 49^3 5.1 -> 4.8, 128^3
// 34.9 -> 32.4; 5-point 300^2 4.5 -> 4.0, 1001^2 14.9 -> 14.2.  With eight
// waves (64 registers) the same kernels spill: the band at 2 M took 302.  In
// FP32, half the registers in flight either way, the walk is as fast or
// faster (128^3 15.6 against 15.8, 1001^2 8.0 against 8.5).
template <typename T, int NH, bool NEAR> constexpr bool ds_pre = sizeof(T) == 8 && (NEAR || NH <= 3);

template <int MODE, typename T> static void ds_launch(hipStream_t s, const DsMat &m, int grid, const DsArgs<T> &a)
{
    ds_dispatch(m, [&](auto nh, auto near) {
        constexpr int NH = decltype(nh)::value;
        constexpr bool NEAR = decltype(near)::value;
        if constexpr (MODE == kDsCg && ds_pre<T, NH, NEAR>) {
            if (a.nslices <= grid * (kBlock / 64))   // then no wave has two
                hipLaunchKernelGGL((k_ds<MODE, T, NH, NEAR, kDsOne>), dim3(grid), dim3(kBlock), 0, s, a);
            else hipLaunchKernelGGL((k_ds<MODE, T, NH, NEAR, kDsLoop>), dim3(grid), dim3(kBlock), 0, s, a);
        } else {
            hipLaunchKernelGGL((k_ds<MODE, T, NH, NEAR, kDsWalk>), dim3(grid), dim3(kBlock), 0, s, a);
        }
    });
}

template <typename T>
void launch_ds_cg_spmv(hipStream_t s, const DsMat &m, int grid, const T *r, T *dA, T *dB, T *q, const double *up,
                       int nup, double *part, int it, int it0, T *x, T *snap, int pc, DevState *st, int32_t *live)
{
    DsArgs<T> a = ds_args<T>(m, grid);
    a.it = it; a.it0 = it0; a.r = r; a.dA = dA; a.dB = dB; a.q = q; a.up = up; a.nup = nup;
    a.x = x; a.snap = snap; a.pc = pc; a.part = part; a.st = st; a.live = live;
    ds_launch<kDsCg, T>(s, m, grid, a);
}

void launch_ds_restart(hipStream_t s, const DsMat &m, int grid, const float *x32, double *x64, const double *b,
                       double *r, double *dA, double *dB, int it0, const double *dg, double *z, double *part,
                       DevState *st)
{
    DsArgs<double> a = ds_args<double>(m, grid);
    a.x32 = x32; a.x64in = x64; a.x64out = x64; a.b = b; a.rout = r; a.dz = (it0 & 1) ? dB : dA;
    a.dg = dg; a.z = z; a.part = part; a.st = st;
    ds_launch<kDsRestart, double>(s, m, grid, a);
}

void launch_ds_resid(hipStream_t s, const DsMat &m, int grid, const double *x64, const double *b, double *part,
                     DevState *st)
{
    DsArgs<double> a = ds_args<double>(m, grid);
    a.x64in = x64; a.b = b; a.part = part; a.st = st;
    ds_launch<kDsResid, double>(s, m, grid, a);
}

template <typename T> void launch_ds_jacobi(hipStream_t s, const DsMat &m, const JacArgs<T> &a)
{
    DsPlanes<T> p{};
    p.p = ds_vals<T>(m);
    p.S = (uint32_t)(ds_stride(m.n) * sizeof(T));
    for (int t = 0; t < kDsMax; ++t) p.d[t] = m.d[t];
    ds_dispatch(m, [&](auto nh, auto near) {
        hipLaunchKernelGGL((k_ds_jac<T, decltype(nh)::value, decltype(near)::value>), dim3(a.np), dim3(kBlock), 0, s, a, p);
    });
}

template void launch_ds_cg_spmv<float>(hipStream_t, const DsMat &, int, const float *, float *, float *, float *,
                                       const double *, int, double *, int, int, float *, float *, int, DevState *,
                                       int32_t *);
template void launch_ds_cg_spmv<double>(hipStream_t, const DsMat &, int, const double *, double *, double *, double *,
                                        const double *, int, double *, int, int, double *, double *, int, DevState *,
                                        int32_t *);
template void launch_ds_jacobi<float>(hipStream_t, const DsMat &, const JacArgs<float> &);
template void launch_ds_jacobi<double>(hipStream_t, const DsMat &, const JacArgs<double> &);

}  // namespace mpcg
