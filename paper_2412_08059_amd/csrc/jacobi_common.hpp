// Arguments and the stop decision shared by the Jacobi-iteration kernels
// (kernels_jacobi.hip describes the scheme).

#pragma once

#include "mpcg_internal.hpp"
#include "sell_common.hpp"

namespace mpcg {

template <typename T>
struct JacArgs {
    // SELL-64 copy (SELL kernel) or CSR (CSR kernel)
    const int32_t *rp;
    const void *scol;
    const T *sval;
    const int64_t *off;
    const int32_t *col;
    const T *val;
    int32_t n, nslices;
    WalkTab walk;
    int32_t k, maxit, abs_tol, np;
    double eps;
    const T *b;
    const T *dg;
    T *x0, *x1;       // xs[0], xs[1]
    double *part;     // 2 * np partials
    DevState *st;
};

// Stop decision of launch k (block-uniform); returns true when the block exits.
template <typename T>
__device__ inline bool jac_prologue(const JacArgs<T> &a, double *sm)
{
    DevState *st = a.st;
    const int k = a.k;
    const double thr = st->thr;
    // stop_it = k - 1 is block 0's decision in this launch, which the waves of
    // a block can see or miss: only an earlier stop skips the barrier below
    if (st->stop_it < k - 1) return true;
    if (k == 0) {
        const double bb = partials_total(false, a.part + a.np, a.np, sm);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            st->bnorm2 = bb;
            st->thr = a.abs_tol ? a.eps : a.eps * sqrt(bb);
        }
        return false;
    }
    const double g = partials_total(false, a.part + (size_t)((k - 1) & 1) * a.np, a.np, sm);
    const bool bad = !(g == g) || isinf(g);
    const bool conv = !bad && sqrt(g) <= thr;
    const bool cap = !conv && !bad && k - 1 >= a.maxit;
    if (!(conv || cap || bad)) return false;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->gamma = g;
        st->iter = k - 1;
        st->reason = conv ? kConverged : (bad ? kNonFinite : kMaxit);
        st->stop_it = k - 1;
        st->live = 0;
    }
    return true;
}

// Diagonal storage (kernels_ds.hip) as a kernel argument.
template <typename T>
struct DsPlanes {
    const T *p;
    uint32_t S;   // bytes from one plane to the next
    int32_t d[kDsMax];
};

template <typename T> void launch_ds_jacobi(hipStream_t s, const DsMat &m, const JacArgs<T> &a);

}  // namespace mpcg
