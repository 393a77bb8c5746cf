// dd_gmres.h -- device side of the coarsest-level GMRES bookkeeping shared by
// the reduction kernels and by the stencil kernel that starts an Arnoldi step.
//
// The norm of a new basis vector is left as partial sums by the kernel that
// makes it.  The first kernel of the next step adds them (each workgroup for
// itself: at most 256 values) for the factor of its input, and one extra
// workgroup per right-hand side folds the finished column into the state
// meanwhile: neither waits for the other, and the update kernel needs no last
// workgroup that runs the rotations while the device is idle (16^4, FP64:
// update 13.0 us with them, 4.7 us without; 6x3^3, FP32, four right-hand
// sides: 18.7 -> 5.5 us).  A stop found there may be seen by some workgroups of
// that launch and is seen by every kernel after it; what the first kernel writes
// for such a right-hand side is scratch.
#pragma once
#include "dd_kernels.h"

namespace dd {

// sum over the chunk partials of ||w||^2 of right-hand side r, in every lane of
// the calling wave
__device__ __forceinline__ double gm_norm2(const cx<double>* __restrict__ npart, int nc, int r) {
    double s = 0;
    for (int c = threadIdx.x & 63; c < nc; c += 64) s += npart[(size_t)r * nc + c].re;
    return wave_sum(s);
}

// factor of the stored basis vector that `isc` names, for right-hand side r
__device__ __forceinline__ double gm_factor(const InScale& isc, int r) {
    if (!isc.npart) return isc.st[r].sc[isc.j];
    const double n2 = gm_norm2(isc.npart, isc.nc, r);
    return n2 > 0 ? 1.0 / sqrt(n2) : 0.0;
}

// fold column j (inner products h[0..j], ||w||^2 = hn2) into the state of
// one RHS, by a whole workgroup (at least 64 threads): the inner products and
// the previous rotations are first staged in LDS by many threads at once, then
// one thread runs the rotation chain with the running entry in registers (the
// global-memory form waits on one load per rotation)
__device__ __forceinline__ void gm_column_wg(GmDev* st, int j, const cx<double>* h, double hn2) {
    __shared__ cx<double> hs[33], css[32], sns[32];
    const int t = threadIdx.x;
    if (t <= j) hs[t] = h[t];
    if (t < j) {
        css[t] = st->cs[t];
        sns[t] = st->sn[t];
    }
    __syncthreads();
    if (t == 0) {
        cx<double>* col = st->H + (size_t)j * 33;
        const double hn = sqrt(hn2);
        cx<double> a = hs[0];
        for (int i = 0; i < j; i++) {  // previous rotations; col[i] is final after rotation i
            const cx<double> b = hs[i + 1];
            col[i] = conj(css[i]) * a + conj(sns[i]) * b;
            a = -(sns[i] * a) + css[i] * b;
        }
        const cx<double> b = cx<double>{hn, 0.0};
        const double den = sqrt(norm2(a) + norm2(b));
        cx<double> c, s;
        if (den == 0.0) { c = cx<double>{1.0, 0.0}; s = czero<double>(); }
        else { c = cx<double>{a.re / den, a.im / den}; s = cx<double>{b.re / den, b.im / den}; }
        st->cs[j] = c;
        st->sn[j] = s;
        col[j] = conj(c) * a + conj(s) * b;
        col[j + 1] = czero<double>();
        const cx<double> gj = st->g[j], gn = -(s * gj);
        st->g[j + 1] = gn;
        st->g[j] = conj(c) * gj;
        const int its = st->its + 1;
        st->its = its;
        st->j = j + 1;
        int stop = 0;
        if (st->fixed > 0) stop = its >= st->fixed;
        else stop = (sqrt(norm2(gn)) <= st->tol_abs) || (its >= st->maxit);
        if (hn == 0.0) stop = 1;
        st->scale = (hn > 0) ? 1.0 / hn : 0.0;
        st->sc[j + 1] = st->scale;   // the new basis vector keeps its factor
        st->stop = stop;
    }
}

// Whether this wave sees right-hand side r running (the same in all its lanes).
// Beside a fold the flag may be raised while the launch runs, so the waves of a
// workgroup may differ: one thread's reading, kept in `run`, decides for all behind
// the first barrier, and no wave leaves before it.  (Waves that went on without the
// others would read input pointers in LDS that nobody had stored.)  What a wave
// asks for ahead of the barrier goes by its own reading.
template <bool FOLD>
__device__ __forceinline__ bool wg_enter(const Mask& mk, int r, int& run) {
    const int on = __builtin_amdgcn_readfirstlane((int)mk.on(r));
    if (FOLD && threadIdx.x == 0) run = on;
    return on != 0;
}

// The extra workgroup of the first kernel of a step: column isc.j - 1 of
// right-hand side r, from the partial norms and the inner products at
// isc.h + r * isc.hstride.
__device__ __forceinline__ void gm_fold(const InScale& isc, int r) {
    GmDev* st = const_cast<GmDev*>(isc.st) + r;
    if (st->stop) return;
    const double n2 = gm_norm2(isc.npart, isc.nc, r);
    gm_column_wg(st, isc.j - 1, isc.h + (size_t)r * isc.hstride, n2);
}

}  // namespace dd
