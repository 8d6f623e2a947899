// BFS of narrow bands (|i - j| <= kSegBand) in segments (gfx950, wave64).
//
// A band's BFS is a chain of about n / 8 levels of a few vertices each; run
// level by level, even in registers, it costs n / 8 dependent steps (a 1M
// band: 2 x 125,000 levels, 80 ms).  Here the rows are cut into segments of
// 2,048 and the chain into two short ones:
//
//   k_seg_local  per segment and boundary row (its first and last 8 rows) the
//                distances to the other boundary rows inside the segment: all
//                segments at once, at most 2,048 levels;
//   k_seg_join   the distances from one segment's boundary rows across the
//                cut to its neighbour's: min-plus products of the above;
//   k_seg_chain  one wave: distances from the source to every boundary row, a
//                16-vector and one 8 x 16 min-plus product per segment, forward
//                and backward until a pass changes nothing;
//   k_seg_fill   per segment, all at once: levels from its boundary rows, each
//                entering at its distance, give every row its distance.
//
// An edge spans at most 8 rows, so a shortest path changes segment only from
// one's boundary rows to the next one's, and inside a segment it is a shortest
// path of that segment's rows alone: the distances are the BFS's, exactly.
// Passes are bounded; a path that turns at more segments than that leaves the
// guard set and the queue kernels take the sweep.
//
// Inside a segment a level is formed on bits, 32 rows per lane: the union over
// the offsets d of the frontier shifted by d (one v_alignbit with the
// neighbouring lane's word, fetched with one DPP move) and the rows that store
// an entry at -d, less the visited rows.  What bounds it: instruction issue,
// about 60 vector instructions a level.  Features of a 1M band 79 -> 1.6 ms, of
// 4M rows 322 -> 4.7 ms.

#include "mpcg_internal.hpp"
#include "wave_ops.hpp"

#include <type_traits>

namespace mpcg {

constexpr int kSegWords = 64;                  // words (lanes) of a segment
constexpr int kSegRows = 32 * kSegWords;
constexpr int kSegBnd = 2 * kSegBand;          // boundary rows: the first and the last kSegBand
constexpr int kSegInf = 0x3fffffff;
constexpr uint16_t kSegInf16 = 0xffff;
constexpr int kSegMaxRel = 1 << 13;            // levels a segment's fill may span (13 bit planes)
constexpr int kSegPasses = 64;                 // chain passes before giving up

static_assert(kSegBnd == 16, "the chain's lane layout is 4 groups of 16 boundary rows");

// value of the lane below / above, 0 at the wave's ends
__device__ inline uint32_t lane_below(uint32_t v) { return dpp_u32<0x138>(v); }
__device__ inline uint32_t lane_above(uint32_t v) { return dpp_u32<0x130>(v); }

// mask t < kSegBand: rows that store an entry at offset -(t + 1); mask
// kSegBand + t: at offset t + 1.  The pattern is symmetric, so these are also
// the rows that row v - (t + 1) (v + t + 1) reaches.
struct SegBufs {
    uint32_t *mask;        // 2 kSegBand masks, nwords apart
    uint16_t *local;       // per segment, kSegBnd x kSegBnd
    uint16_t *fwd, *bwd;   // per cut, kSegBand x kSegBnd
    int32_t *dist;         // per segment, kSegBnd
    int32_t n, nwords, nseg;
};

static SegBufs seg_bufs(const BfsBufs &b)
{
    SegBufs s{};
    s.n = b.n;
    s.nwords = b.nwords;
    s.nseg = (b.n + kSegRows - 1) / kSegRows;
    s.mask = b.dm;   // 16 masks, as the diagonal levels' (at most one of the two is in use)
    char *at = reinterpret_cast<char *>(b.q0);   // 8 bytes a row; 1,088 bytes a segment are used
    auto take = [&](size_t bytes) {
        char *q = at;
        at += (bytes + 255) & ~(size_t)255;
        return q;
    };
    s.local = reinterpret_cast<uint16_t *>(take(sizeof(uint16_t) * kSegBnd * kSegBnd * (size_t)s.nseg));
    s.fwd = reinterpret_cast<uint16_t *>(take(sizeof(uint16_t) * kSegBand * kSegBnd * (size_t)s.nseg));
    s.bwd = reinterpret_cast<uint16_t *>(take(sizeof(uint16_t) * kSegBand * kSegBnd * (size_t)s.nseg));
    s.dist = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * kSegBnd * (size_t)s.nseg));
    return s;
}

// Wave per 64 rows: presence bits by ballot, entries staged in LDS.
__global__ void __launch_bounds__(kBlock)
k_seg_masks(const int32_t *__restrict__ rp, const int32_t *__restrict__ col, SegBufs b)
{
    constexpr int kMax = 2 * kSegBand + 1;   // entries of a row of a band that narrow
    __shared__ int32_t s_col[kBlock / 64][64 * kMax];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int32_t *sc = s_col[w];
    const int nsl = (b.n + 63) / 64;
    for (int s = blockIdx.x * (kBlock / 64) + w; s < nsl; s += gridDim.x * (kBlock / 64)) {
        const int r0 = s * 64, nrows = min(64, b.n - r0);
        const int row = r0 + lane;
        const int rpl = rp[r0 + min(lane, nrows)], rph = rp[r0 + min(lane + 1, nrows)];
        const int lo = __builtin_amdgcn_readfirstlane(rpl);
        const int cnt = min(rp[r0 + nrows] - lo, 64 * kMax);
        for (int k0 = 0; k0 < cnt; k0 += 256) {
            int c[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (k0 + j * 64 + lane < cnt) c[j] = col[lo + k0 + j * 64 + lane];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (k0 + j * 64 + lane < cnt) sc[k0 + j * 64 + lane] = c[j];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        uint32_t have = 0;   // bit d + kSegBand: an entry at offset d
        for (int k = rpl - lo; k < min(rph - lo, cnt); ++k) {
            const int d = sc[k] - row;
            if (d >= -kSegBand && d <= kSegBand && sc[k] >= 0 && sc[k] < b.n) have |= 1u << (d + kSegBand);
        }
#pragma unroll
        for (int t = 0; t < 2 * kSegBand; ++t) {
            const int d = t < kSegBand ? -(t + 1) : t - kSegBand + 1;
            const unsigned long long bits = __ballot(lane < nrows && ((have >> (d + kSegBand)) & 1));
            if (lane < 2 && 2 * s + lane < b.nwords)
                b.mask[(size_t)t * b.nwords + 2 * s + lane] = (uint32_t)(bits >> (32 * lane));
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// A segment's masks in registers (lane = word); zero past the matrix.
template <int W> struct SegMasks {
    uint32_t up[W], dn[W];   // rows that the row d below (above) reaches
};

template <int W> __device__ inline SegMasks<W> seg_load(const SegBufs &b, int seg)
{
    SegMasks<W> m;
    const int word = seg * kSegWords + (threadIdx.x & 63);
#pragma unroll
    for (int t = 0; t < W; ++t) {
        m.up[t] = word < b.nwords ? b.mask[(size_t)t * b.nwords + word] : 0u;
        m.dn[t] = word < b.nwords ? b.mask[(size_t)(kSegBand + t) * b.nwords + word] : 0u;
    }
    return m;
}

// The rows reached from the frontier F within the segment.
template <int W> __device__ inline uint32_t seg_step(const SegMasks<W> &m, uint32_t F)
{
    const uint32_t lo = lane_below(F), hi = lane_above(F);
    uint32_t nx = 0;
#pragma unroll
    for (int t = 0; t < W; ++t) {
        nx |= __builtin_amdgcn_alignbit(F, lo, 31 - t) & m.up[t];   // rows v = u + t + 1
        nx |= __builtin_amdgcn_alignbit(hi, F, t + 1) & m.dn[t];    // rows v = u - t - 1
    }
    return nx;
}

// Distances inside the segment from the rows of F (level 0) to its boundary
// rows: lane j < kSegBnd returns boundary row j's, kSegInf if not reached.
template <int W> __device__ inline int seg_bfs(const SegMasks<W> &m, uint32_t F)
{
    const int lane = threadIdx.x & 63;
    uint32_t V = F;
    int out = kSegInf;
    for (int lev = 0; lev <= kSegRows; ++lev) {
        const uint32_t first = __builtin_amdgcn_readlane(F, 0) & ((1u << kSegBand) - 1);
        const uint32_t last = (uint32_t)__builtin_amdgcn_readlane(F, 63) >> (32 - kSegBand);
        const uint32_t hit = first | (last << kSegBand);
        if (hit && lane < kSegBnd && ((hit >> lane) & 1)) out = lev;
        if (__ballot(F != 0) == 0ull) break;
        F = seg_step<W>(m, F) & ~V;
        V |= F;
    }
    return out;
}

// boundary row j of a segment as (lane, bit)
__device__ inline uint32_t seg_bnd_word(int j)
{
    const int lane = threadIdx.x & 63;
    if (j < kSegBand) return lane == 0 ? 1u << j : 0u;
    return lane == 63 ? 1u << (32 - kSegBnd + j) : 0u;
}

template <int W> __global__ void __launch_bounds__(kBlock) k_seg_local(SegBufs b)
{
    const int w = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int seg = w / kSegBnd, src = w % kSegBnd;
    if (seg >= b.nseg) return;
    const int row = seg * kSegRows + (src < kSegBand ? src : kSegRows - kSegBnd + src);
    const SegMasks<W> m = seg_load<W>(b, seg);
    const int d = seg_bfs<W>(m, row < b.n ? seg_bnd_word(src) : 0u);
    if (lane < kSegBnd)
        b.local[((size_t)seg * kSegBnd + src) * kSegBnd + lane] = d < kSegInf ? (uint16_t)d : kSegInf16;
}

// Cut between segments k and k + 1, thread per (i, j): fwd from last row i of
// k to boundary row j of k + 1, bwd from first row i of k + 1 to boundary row
// j of k; one edge across the cut, then the segment's own distances.
__global__ void __launch_bounds__(kBlock) k_seg_join(SegBufs b)
{
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t k = t / (kSegBand * kSegBnd);
    if (k >= b.nseg - 1) return;
    const int i = (int)(t / kSegBnd) % kSegBand, j = (int)(t % kSegBnd);
    const int64_t cut = (k + 1) * kSegRows;   // first row of segment k + 1
    int f = kSegInf, r = kSegInf;
    for (int a = 0; a < kSegBand; ++a) {
        // last row i of k is cut - kSegBand + i, first row a of k + 1 is cut + a
        const int df = kSegBand - i + a;       // their distance
        if (df <= kSegBand && cut + a < b.n) {
            const int64_t v = cut + a;         // stores the row df below it?
            if ((b.mask[(size_t)(df - 1) * b.nwords + (v >> 5)] >> (v & 31)) & 1) {
                const int d = b.local[((size_t)(k + 1) * kSegBnd + a) * kSegBnd + j];
                if (d != kSegInf16) f = min(f, d + 1);
            }
        }
        const int db = kSegBand - a + i;       // first row i of k + 1, last row a of k
        if (db <= kSegBand && cut + i < b.n) {
            const int64_t v = cut - kSegBand + a;   // stores the row db above it?
            if ((b.mask[(size_t)(kSegBand + db - 1) * b.nwords + (v >> 5)] >> (v & 31)) & 1) {
                const int d = b.local[((size_t)k * kSegBnd + kSegBand + a) * kSegBnd + j];
                if (d != kSegInf16) r = min(r, d + 1);
            }
        }
    }
    // lane layout of the chain: (pair of i, j, which of the pair)
    const size_t at = (size_t)k * kSegBand * kSegBnd + ((size_t)(i / 2) * kSegBnd + j) * 2 + (i & 1);
    b.fwd[at] = f < kSegInf16 ? (uint16_t)f : kSegInf16;
    b.bwd[at] = r < kSegInf16 ? (uint16_t)r : kSegInf16;
}

__device__ inline int min_group(int v)   // over the four lanes 16 apart
{
    const LanePair p = lane_pair<16>((uint32_t)v);
    v = min((int)p.a, (int)p.b);
    const LanePair q = lane_pair<32>((uint32_t)v);
    return min((int)q.a, (int)q.b);
}

// One pass over the segments in one direction.  cur: boundary distances of
// the segment it stands on (lane l: row l & 15, the four groups alike).
// Returns whether a distance fell.
template <bool FWD> __device__ inline bool seg_pass(const SegBufs &b)
{
    constexpr int D = 8;   // cuts whose loads are in flight
    const int lane = threadIdx.x & 63, j = lane & 15, g = lane >> 4;
    const int from = (FWD ? kSegBand : 0) + 2 * g;   // the two rows this lane's group starts from
    const uint32_t *c32 = reinterpret_cast<const uint32_t *>(FWD ? b.fwd : b.bwd);
    const int ncut = b.nseg - 1;
    bool fell = false;
    int cur = b.dist[(size_t)(FWD ? 0 : b.nseg - 1) * kSegBnd + j];
    uint32_t c[D];
    int nd[D];
    auto cut_of = [&](int s) { return FWD ? s : ncut - 1 - s; };
    auto load = [&](int s, uint32_t &cc, int &dd) {
        if (s >= ncut) return;
        const int k = cut_of(s);
        cc = c32[(size_t)k * (kSegBand * kSegBnd / 2) + lane];
        dd = b.dist[(size_t)(FWD ? k + 1 : k) * kSegBnd + j];
    };
#pragma unroll
    for (int u = 0; u < D; ++u) load(u, c[u], nd[u]);
    for (int s0 = 0; s0 < ncut; s0 += D) {
        uint32_t c2[D];
        int nd2[D];
#pragma unroll
        for (int u = 0; u < D; ++u) load(s0 + D + u, c2[u], nd2[u]);
#pragma unroll
        for (int u = 0; u < D; ++u) {
            if (s0 + u >= ncut) break;
            const int a0 = __shfl(cur, from, 64), a1 = __shfl(cur, from + 1, 64);
            const int w0 = (int)(c[u] & 0xffff), w1 = (int)(c[u] >> 16);
            int t = min(w0 == kSegInf16 ? kSegInf : a0 + w0, w1 == kSegInf16 ? kSegInf : a1 + w1);
            t = min(min_group(t), kSegInf);
            const int old = nd[u];
            cur = min(old, t);
            if (__ballot(cur < old) != 0ull) {
                fell = true;
                const int k = cut_of(s0 + u);
                if (lane < kSegBnd) b.dist[(size_t)(FWD ? k + 1 : k) * kSegBnd + lane] = cur;
            }
        }
#pragma unroll
        for (int u = 0; u < D; ++u) {
            c[u] = c2[u];
            nd[u] = nd2[u];
        }
    }
    return fell;
}

// Boundary distances from the source (one wave).
template <int W> __global__ void __launch_bounds__(64) k_seg_chain(SegBufs b, int32_t src, DevState *st)
{
    const int lane = threadIdx.x;
    const int seg = src / kSegRows, loc = src % kSegRows;
    for (int64_t i = lane; i < (int64_t)b.nseg * kSegBnd; i += 64) b.dist[i] = kSegInf;
    const SegMasks<W> m = seg_load<W>(b, seg);
    const int d = seg_bfs<W>(m, lane == loc / 32 ? 1u << (loc & 31) : 0u);
    __threadfence_block();
    if (lane < kSegBnd) b.dist[(size_t)seg * kSegBnd + lane] = d;
    __threadfence_block();
    bool fell = true;
    int pass = 0;
    for (; fell && pass < kSegPasses; pass += 2) {
        fell = seg_pass<true>(b);
        __threadfence_block();
        const bool back = seg_pass<false>(b);
        __threadfence_block();
        fell = back;   // a forward pass follows only what a backward one changed
    }
    if (lane == 0) {
        st->bfs_visited = 0;
        st->comp_best = 0;
        st->bfs_done = 0;
        st->bfs_ecc = 0;
        st->bfs_far = src;
        if (fell) st->guard = 1;
    }
}

// Wave per segment: every row's distance (dist, if given), and the segment's
// visited rows and farthest row (largest distance, then smallest index).
template <int W> __global__ void __launch_bounds__(64) k_seg_fill(SegBufs b, int32_t src, int32_t *dist, DevState *st)
{
    __shared__ int32_t s_d[64 * 33];
    const int lane = threadIdx.x, seg = blockIdx.x;
    const SegMasks<W> m = seg_load<W>(b, seg);
    // lanes 0 and 63 hold the boundary rows' entry levels, first and last
    int seed[kSegBand];
    int lo = kSegInf, hi = -1;
#pragma unroll
    for (int i = 0; i < kSegBand; ++i) {
        const int j = lane == 0 ? i : kSegBand + i;
        seed[i] = lane == 0 || lane == 63 ? b.dist[(size_t)seg * kSegBnd + j] : kSegInf;
        if (seed[i] < kSegInf) {
            lo = min(lo, seed[i]);
            hi = max(hi, seed[i]);
        }
    }
    const int ls = src / kSegRows == seg ? src % kSegRows : -1;   // the source's own segment
    if (ls >= 0) {
        lo = 0;
        hi = max(hi, 0);
    }
    for (int o = 32; o > 0; o >>= 1) {
        lo = min(lo, __shfl_xor(lo, o, 64));
        hi = max(hi, __shfl_xor(hi, o, 64));
    }
    lo = __builtin_amdgcn_readfirstlane(lo);
    hi = __builtin_amdgcn_readfirstlane(hi);
    const int sh = lane == 0 ? 0 : 32 - kSegBand;
    uint32_t F = 0, V = 0, lastF = 0, plane[13];
#pragma unroll
    for (int k = 0; k < 13; ++k) plane[k] = 0;
    int lastlev = 0;
    if (lo < kSegInf) {
        bool over = false;
        for (int lev = lo;; ++lev) {
            uint32_t nx = lev == lo ? 0u : seg_step<W>(m, F);
            if (lev <= hi) {
                uint32_t in = 0;
#pragma unroll
                for (int i = 0; i < kSegBand; ++i) in |= seed[i] == lev ? 1u << i : 0u;
                nx |= in << sh;
                if (lev == 0 && ls >= 0 && lane == ls / 32) nx |= 1u << (ls & 31);
            }
            F = nx & ~V;
            V |= F;
            if (__ballot(F != 0) == 0ull) {
                if (lev >= hi) break;
            } else {
                lastF = F;
                lastlev = lev;
            }
            const int rel = lev - lo;
            if (rel >= kSegMaxRel) {
                over = true;
                break;
            }
            if (dist) {
#pragma unroll
                for (int k = 0; k < 13; ++k) plane[k] |= F & (0u - ((uint32_t)(rel >> k) & 1u));
            }
        }
        if (over && lane == 0) st->guard = 1;
        // visited rows, farthest row
        int cnt = __popc(V);
        for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
        const unsigned long long has = __ballot(lastF != 0);
        const int l0 = __builtin_ctzll(has);
        const uint32_t w0 = __builtin_amdgcn_readlane(lastF, l0);
        if (lane == 0) {
            const uint32_t row = (uint32_t)seg * kSegRows + (uint32_t)l0 * 32 + (uint32_t)__builtin_ctz(w0);
            atomicAdd(reinterpret_cast<unsigned long long *>(&st->bfs_visited), (unsigned long long)cnt);
            atomicMax(reinterpret_cast<unsigned long long *>(&st->comp_best),
                      ((unsigned long long)(uint32_t)lastlev << 32) | (0xffffffffu - row));
        }
    }
    if (!dist) return;
    for (int r = 0; r < 32; ++r) {
        int d = 0;
#pragma unroll
        for (int k = 0; k < 13; ++k) d |= (int)((plane[k] >> r) & 1u) << k;
        s_d[lane * 33 + r] = (V >> r) & 1u ? lo + d : -1;
    }
    __syncthreads();
    for (int i = lane; i < kSegRows; i += 64) {
        const int64_t row = (int64_t)seg * kSegRows + i;
        if (row < b.n) dist[row] = s_d[(i >> 5) * 33 + (i & 31)];
    }
}

template <typename F> static void seg_dispatch(int band, const F &f)
{
    if (band <= 1) f(std::integral_constant<int, 1>());
    else if (band <= 2) f(std::integral_constant<int, 2>());
    else if (band <= 4) f(std::integral_constant<int, 4>());
    else f(std::integral_constant<int, 8>());
}

void launch_seg_prepare(hipStream_t s, const BfsBufs &bb)
{
    const SegBufs b = seg_bufs(bb);
    int g = ((b.n + 63) / 64 + kBlock / 64 - 1) / (kBlock / 64);
    if (g > 8192) g = 8192;
    hipLaunchKernelGGL(k_seg_masks, dim3(g), dim3(kBlock), 0, s, bb.rp, bb.col, b);
    const int64_t waves = (int64_t)b.nseg * kSegBnd;
    seg_dispatch(bb.band, [&](auto w) {
        hipLaunchKernelGGL((k_seg_local<decltype(w)::value>), dim3((unsigned)((waves + 3) / 4)), dim3(kBlock), 0, s, b);
    });
    const int64_t threads = (int64_t)(b.nseg - 1) * kSegBand * kSegBnd;
    if (threads > 0)
        hipLaunchKernelGGL(k_seg_join, dim3((unsigned)((threads + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, b);
}

void launch_seg_sweep(hipStream_t s, const BfsBufs &bb, int32_t src, bool want_dist)
{
    const SegBufs b = seg_bufs(bb);
    seg_dispatch(bb.band, [&](auto w) {
        constexpr int W = decltype(w)::value;
        hipLaunchKernelGGL((k_seg_chain<W>), dim3(1), dim3(64), 0, s, b, src, bb.st);
        hipLaunchKernelGGL((k_seg_fill<W>), dim3(b.nseg), dim3(64), 0, s, b, src, want_dist ? bb.dist : nullptr, bb.st);
    });
}

}  // namespace mpcg
