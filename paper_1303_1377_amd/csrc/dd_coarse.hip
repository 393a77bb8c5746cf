// dd_coarse.hip -- kernels on coarse levels (nd = 2N unknowns per site).
//
//   coarse stencil D_c ............ nearest-neighbour blocks of P^H D P (Sec. 3.2)
//   odd-even pieces ............... Schur complement A_oo - D_oe A_ee^{-1} D_eo (Sec. 5)
//   self-block inverses ........... dense Gauss-Jordan in FP64
//   coarse SAP, P^H, P, Gram-Schmidt, assembly of the next coarser operator
//                                   (recursive application, Sec. 3 and 5)
//
// Vectors are [parity][layout index][nd] (a site's unknowns contiguous);
// operator blocks are column-major so that the thread owning row r reads
// consecutive addresses across the wavefront.
#include <algorithm>
#include <mutex>
#include <stdexcept>
#include <type_traits>

#include "dd_gmres.h"

namespace dd {

static inline int nblk_of(long n, int b) { return (int)((n + b - 1) / b); }

// ---------------------------------------------------------------------------
// out(x) = [post Minv] ( self(x) in1(x) + hop_sign * sum_k M_{1+k}(x) in2(x_k) )
// One workgroup per site.  The site's blocks used here lie back to back in
// memory (self, then the 8 hops, each column-major), so (block, column) pair
// q is column q of one nd-row panel.  The pairs are split evenly over the
// wavefronts and lane r accumulates row r: every load is coalesced.  On small
// coarse lattices (a few hundred sites) the kernel is bound by memory latency,
// not bandwidth, so each lane issues the loads of its first pairs (and of its
// columns of the self-block inverse) before the site's input vectors
// (hop sign folded in) are staged in LDS: block entries and inputs are in
// flight together.  Partial rows meet in LDS.
// ---------------------------------------------------------------------------
static constexpr int CA_WAVES = 12;
// block entries and inverse-block columns a lane loads at once (fewer in
// FP64, where they take twice the registers)
template <class S> struct CaPre {
    static constexpr int N = sizeof(S) > 4 ? 24 : 30;
    static constexpr int INV = sizeof(S) > 4 ? 4 : 8;
};

// FOLD: the first kernel of an Arnoldi step, which also folds the step before
// (compiled apart: the fold's registers cost the FP16-storage row kernel a wave
// per SIMD, 80 -> 90 registers, 8^4 sites of 32 unknowns 36 -> 41 us)
template <class T, class S, bool FOLD = true>
__global__ void __launch_bounds__(64 * CA_WAVES) k_coarse_apply(CoarseOp<T, S> op, int par, int self_mode,
                                                                const cx<T>* __restrict__ in1, int hop_sign,
                                                                const cx<T>* in2, int post_inv, cx<T>* out,
                                                                Mask mk, long ld, InScale isc, int nsite) {
    __shared__ int run;
    if constexpr (FOLD) {
        if ((int)blockIdx.x >= nsite) {   // the extra workgroup
            gm_fold(isc, blockIdx.y);
            return;
        }
    }
    const bool early = wg_enter<FOLD>(mk, blockIdx.y, run);
    if (!FOLD && !early) return;
    {
        const long off = blockIdx.y * ld;
        if (in1) in1 += off;
        if (in2) in2 += off;
        out += off;
    }
    __shared__ cx<T> part[CA_WAVES][64];
    __shared__ cx<T> X[9 * 64];            // staged inputs [slot][nd] (nd <= 64)
    __shared__ const cx<T>* vin[9];
    const Geom g = op.g;
    const int nd = op.nd;
    const int nw = blockDim.x >> 6, w = threadIdx.x >> 6, r = threadIdx.x & 63;
    int p, i;
    if (par < 0) { p = blockIdx.x >= g.vh; i = blockIdx.x - p * g.vh; }
    else { p = par; i = blockIdx.x; }
    const size_t gs = (size_t)p * g.vh + i;
    const size_t nn = (size_t)nd * nd;
    const int nself = (self_mode == CS_SELF || self_mode == CS_SELFINV) ? 1 : 0;
    // first block of the panel: the self block, its inverse, or the first hop
    const cx<S>* panel = (self_mode == CS_SELFINV) ? op.Minv + gs * nn : op.M + (gs * 9 + 1 - nself) * nn;
    // input vectors of the panel's column slots: thread k < 8 finds neighbour k
    if (threadIdx.x == 0 && nself) vin[0] = in1 + gs * nd;
    if (hop_sign != 0 && threadIdx.x < 8) {
        int x[4];
        cb_coords(g, p, i, x);
        vin[nself + threadIdx.x] = in2 + nb_global(g, p, x, threadIdx.x) * nd;
    }
    const int ns = nself + (hop_sign != 0 ? 8 : 0);
    const int Q = ns * nd;
    const int per = (Q + nw - 1) / nw;
    const int q0 = w * per, q1 = min(Q, q0 + per);
    const bool row = r < nd;
    const cx<S>* A = panel + r;
    constexpr int CA_PRE = CaPre<S>::N;
    cx<S> a[CA_PRE];
    auto load_pairs = [&](int qb) {
#pragma unroll
        for (int u = 0; u < CA_PRE; u++)
            a[u] = (row && qb + u < q1) ? A[(size_t)(qb + u) * nd] : cx<S>{S(0), S(0)};
    };
    const int per2 = (nd + nw - 1) / nw;
    const int c0 = w * per2, c1 = min(nd, c0 + per2);
    const cx<S>* Ainv = op.Minv + gs * nn + r;
    constexpr int CA_INV = CaPre<S>::INV;
    cx<S> b[CA_INV];
    auto load_inv = [&](int cb) {
#pragma unroll
        for (int u = 0; u < CA_INV; u++)
            b[u] = (row && cb + u < c1) ? Ainv[(size_t)(cb + u) * nd] : cx<S>{S(0), S(0)};
    };
    T f1 = T(1), f2 = T(hop_sign < 0 ? -1 : 1);
    auto ahead = [&]() {   // in flight while the inputs are staged
        load_pairs(q0);
        if (post_inv) load_inv(c0);
        if (isc.st) {
            const T f = T(FOLD ? gm_factor(isc, blockIdx.y) : isc.st[blockIdx.y].sc[isc.j]);
            if (isc.which & 1) f1 *= f;
            if (isc.which & 2) f2 *= f;
        }
    };
    if (early) ahead();
    __syncthreads();
    if constexpr (FOLD) {
        if (!run) return;
        if (!early) ahead();
    }
    for (int e = threadIdx.x; e < Q; e += blockDim.x) {
        const int s2 = e / nd;
        X[e] = ((s2 >= nself) ? f2 : f1) * vin[s2][e - s2 * nd];
    }
    __syncthreads();
    cx<T> acc = czero<T>();
    for (int qb = q0; qb < q1; qb += CA_PRE) {
        if (qb != q0) load_pairs(qb);
#pragma unroll
        for (int u = 0; u < CA_PRE; u++)
            if (qb + u < q1) acc += ccast<T>(a[u]) * X[qb + u];
    }
    part[w][r] = acc;
    __syncthreads();
    cx<T> tot = czero<T>();
    if (w == 0 && row) {
        tot = (self_mode == CS_IDENT) ? f1 * in1[gs * nd + r] : czero<T>();
        for (int q = 0; q < nw; q++) tot += part[q][r];
    }
    if (!post_inv) {
        if (w == 0 && row) out[gs * nd + r] = tot;
        return;
    }
    if (w == 0) X[r] = tot;
    __syncthreads();
    cx<T> a3 = czero<T>();
    for (int cb = c0; cb < c1; cb += CA_INV) {
        if (cb != c0) load_inv(cb);
#pragma unroll
        for (int u = 0; u < CA_INV; u++)
            if (cb + u < c1) a3 += ccast<T>(b[u]) * X[cb + u];
    }
    part[w][r] = a3;
    __syncthreads();
    if (w == 0 && row) {
        cx<T> s2 = czero<T>();
        for (int q = 0; q < nw; q++) s2 += part[q][r];
        out[gs * nd + r] = s2;
    }
}

// ---------------------------------------------------------------------------
// Multi-RHS coarse stencil on the matrix cores.  For one site and k <= 16
// right-hand sides the apply is a sum of complex products
//     C (nd x k) += M_s (nd x nd) X_s (nd x k),   s = self + 8 hops,
// which runs as real MFMA tiles on the split real / imaginary parts:
//     C_re += M_re X_re - M_im X_im,   C_im += M_re X_im + M_im X_re.
// Up to eight right-hand sides take one tile for both parts (half the
// instructions).  Workgroup = one site; a wave owns 16 rows of C (nd <= 64).  The
// k right-hand-side columns of every X_s are staged once in LDS (one coalesced
// pass per RHS), so each block entry is read once for all right-hand sides.
// The FP32 form uses v_mfma_f32_16x16x4_f32 on FP32 blocks; the FP16-storage
// form uses v_mfma_f32_16x16x16_f16 with the blocks as stored and X rounded to
// FP16 (FP32 accumulation in both).
//   16x16xK tile layout (lane l = 16 q + j):  A row j, k-slice q;  B column j,
//   k-slice q;  D column j, rows 4q .. 4q+3 in the four result registers.
// ---------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

template <class S> struct MfmaK;
template <> struct MfmaK<float> { static constexpr int K = 4; };       // k per instruction, FP32 inputs
template <> struct MfmaK<_Float16> { static constexpr int K = 16; };   // k per instruction, FP16 inputs

__device__ __forceinline__ f32x4 mma(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mma(f16x4 a, f16x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0);
}

// columns of X staged in LDS for a batch of nr right-hand sides (the tile
// has 16): a batch of four needs a quarter of the LDS of sixteen, so more
// workgroups share a CU
__host__ __device__ __forceinline__ int mfma_cols(int nr) { return nr <= 4 ? 4 : (nr <= 8 ? 8 : 16); }

// The A fragments of one block for the wave's tile: rows r = 16 w + (lane & 15),
// k-slices of NS instruction steps.  Outside the block the last row or column is
// read again (no branch around a load): rows past it are never stored, columns
// past it meet rows of X that hold zeros.
template <class S, int NS>
struct TileFrags {
    using F = typename std::conditional<std::is_same<S, float>::value, float, f16x4>::type;
    F re[NS], im[NS];
    __device__ __forceinline__ void load(const cx<S>* __restrict__ A, int nd, int r, int q, int t0 = 0, int step = 1) {
        constexpr int KL = MfmaK<S>::K / 4;
#pragma unroll
        for (int t = 0; t < NS; t++) {
            const int c0 = (t0 + t * step) * MfmaK<S>::K + q * KL;
            if constexpr (std::is_same<S, float>::value) {
                const cx<float> a = A[min(c0, nd - 1) * nd + min(r, nd - 1)];
                re[t] = a.re;
                im[t] = a.im;
            } else {
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const cx<_Float16> a = A[min(c0 + u, nd - 1) * nd + min(r, nd - 1)];
                    re[t][u] = a.re;
                    im[t][u] = a.im;
                }
            }
        }
    }
    // C += A X for X staged as [row][2 xs] reals: columns j < xs the real, xs + j the
    // imaginary parts of right-hand side j.  PACK (xs <= 8): one tile holds both,
    //   [C_re | C_im] += A_re [X_re | X_im] + A_im [-X_im | X_re],
    // two instructions per step; otherwise two tiles and four instructions.
    template <bool PACK>
    __device__ __forceinline__ void multiply(const S* __restrict__ X, int xs, int lane, f32x4& c0, f32x4& c1, int t0 = 0,
                                             int step = 1) const {
        constexpr int K = MfmaK<S>::K, KL = K / 4;
        const int q = lane >> 4, j = lane & 15, cols = 2 * xs;
        auto frag = [&](int t, int col, bool on) {
            const S* x = X + ((t0 + t * step) * K + q * KL) * cols + col;
            if constexpr (std::is_same<S, float>::value) {
                return on ? x[0] : 0.f;
            } else {
                f16x4 v = {};
                if (on)
#pragma unroll
                    for (int u = 0; u < 4; u++) v[u] = x[u * cols];
                return v;
            }
        };
        if constexpr (PACK) {
            const bool on = j < cols;
            const bool lo = j < xs;
            const int js = lo ? j + xs : j - xs;
#pragma unroll
            for (int t = 0; t < NS; t++) {
                const F b = frag(t, j, on);
                F s = frag(t, js, on);
                s = lo ? -s : s;
                c0 = mma(re[t], b, c0);
                c0 = mma(im[t], s, c0);
            }
        } else {
#pragma unroll
            for (int t = 0; t < NS; t++) {
                const F br = frag(t, j, true), bi = frag(t, xs + j, true), ni = -im[t];
                c0 = mma(re[t], br, c0);
                c0 = mma(ni, bi, c0);
                c1 = mma(re[t], bi, c1);
                c1 = mma(im[t], br, c1);
            }
        }
    }
};

// Waves: (row tile, slot group): group g of MG multiplies the slots g, g + MG,
// ...; the groups' partial tiles meet in LDS.
//   MG = 3: a wave loads the fragments of all its slots before anything else, so
//   the whole panel of the site is in flight while its inputs are staged.  For
//   lattices of few sites, where one site's latency is the launch's: 64x32^3
//   coarsest level (256 sites a launch, FP32, four RHS) 20 -> 14 us.
//   MG = 1: small workgroups that load one block ahead; eight share a CU and hide
//   each other's waits, which beats the deeper loads once every CU has several
//   sites: 64x32^3 level 1 (8192 sites) 284 -> 213 us (4.4 TB/s), against 360 us
//   for MG = 3.
// Both forms timed for 1 to 30 test vectors N (2 N unknowns), 256 to 16384 sites
// and 2 to 16 right-hand sides.  With two row tiles or more the line is 1024 sites:
// FP32, N = 10..16, MG = 3 takes 0.7-0.8 of the time of MG = 1 at 512 sites, 1.0-1.2
// at 1024; FP16 storage, N = 20, 0.72 and 1.3 (FP32, N >= 20, crosses earlier: 0.77 at
// 256, 1.2 at 512).  With one tile (N <= 8) it is 2048: 0.8-1.0 at 1296, 0.9-1.2 at
// 2592; and as the one wave of MG = 1 stages all nine slots, MG = 3 serves every
// size from 128 entries per slot on (16384 sites, FP32, N = 5..8, eight RHS: 0.85).
template <class S, int NS, int MG> struct MfmaWg {
    static constexpr int NT = 64 * MG * ((NS * MfmaK<S>::K + 15) / 16);
};
// ND: the unknowns per site where they are known to the compiler (0: op.nd)
template <class S, int NS, bool PACK, int ND, int MG>
__global__ void __launch_bounds__((MfmaWg<S, NS, MG>::NT)) k_coarse_apply_mfma(CoarseOp<float, S> op, int par, int self_mode,
                                                                   const cx<float>* __restrict__ in1, int hop_sign,
                                                                   const cx<float>* in2, int post_inv, cx<float>* out,
                                                                   Mask mk, long ld, int nr, InScale isc, int nsite) {
    if ((int)blockIdx.x >= nsite) {   // the extra workgroups of a first Arnoldi kernel
        gm_fold(isc, blockIdx.x - nsite);
        return;
    }
    constexpr int K = MfmaK<S>::K, NDK = NS * K;
    constexpr bool F16 = std::is_same<S, _Float16>::value;
    constexpr int NSI = (NS + MG - 1) / MG;         // steps of the inverse block per group
    extern __shared__ __align__(16) char smem_raw[];
    __shared__ float fac[2][16], sc[16];
    const Geom g = op.g;
    const int nd = ND ? ND : op.nd, xs = mfma_cols(nr), cols = 2 * xs;
    const int ntile = (nd + 15) / 16;
    S* X = reinterpret_cast<S*>(smem_raw);          // [9][NDK][cols]
    f32x4* red = reinterpret_cast<f32x4*>(X + 9 * NDK * cols);   // [MG - 1][ntile][PACK ? 1 : 2][64]
    int p, i;
    if (par < 0) { p = blockIdx.x >= g.vh; i = blockIdx.x - p * g.vh; }
    else { p = par; i = blockIdx.x; }
    const size_t gs = (size_t)p * g.vh + i;
    const size_t nn = (size_t)nd * nd;
    const int t = threadIdx.x, nt = blockDim.x, nw = nt >> 6;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63, q = lane >> 4, j = lane & 15;
    const int w = wv % ntile, grp = wv / ntile;
    const int r = 16 * w + j;
    const int nself = (self_mode == CS_SELF || self_mode == CS_SELFINV) ? 1 : 0;
    const int ns = nself + (hop_sign != 0 ? 8 : 0);
    // lane k holds flag and factor of right-hand side k: one load for all (beside a
    // fold the waves may see a flag before and after it is raised: such a column is
    // staged and stored in part, and nothing reads it)
    const bool mine = lane < nr && mk.on(lane);
    double f0 = (isc.st && !isc.npart && lane < nr) ? isc.st[lane].sc[isc.j] : 1.0;
    const unsigned on = (unsigned)__ballot(mine);
    // Staging of X: wave wv takes the slots wv, wv + nw, ... (its neighbour is
    // uniform), entries lane, lane + 64, ... of [RHS][row], row fastest so each
    // input is read contiguously.  Loads return in order, so the inputs of the
    // first PS slots (SR entries a lane) are asked for before the block fragments.
    constexpr int SR = 3, PS = MG == 1 ? 3 : 1;   // entries per slot and slots asked for ahead
    int x[4];
    cb_coords(g, p, i, x);
    // MG = 1: lane k finds neighbour k; a wave that stages several slots would find
    // them one after another (8^4 sites of 4 unknowns, FP32, two RHS: 16.4 -> 14.2 us).
    // With MG = 3 a wave has one slot, or three (one by one is 4 % faster there: 24
    // against 25 us at 512 sites of 36 unknowns)
    int nb = 0;
    if constexpr (MG == 1) nb = (int)nb_global(g, p, x, lane & 7);
    auto input = [&](int sl) {
        if (sl < nself) return in1 + gs * nd;
        const int k = sl - nself;
        if constexpr (MG == 1) return in2 + (size_t)__builtin_amdgcn_readlane(nb, k) * nd;
        else return in2 + nb_global(g, p, x, k) * nd;
    };
    auto entry = [&](const cx<float>* v, int e) {
        const int k = e / NDK, c = e - k * NDK;
        return (k < nr && c < nd && ((on >> k) & 1u)) ? v[(size_t)k * ld + c] : czero<float>();
    };
    cx<float> pre[PS][SR];
#pragma unroll
    for (int a = 0; a < PS; a++)
        if (wv + a * nw < ns) {
            const cx<float>* v = input(wv + a * nw);
#pragma unroll
            for (int u = 0; u < SR; u++) pre[a][u] = entry(v, lane + 64 * u);
        }
    // factors of the inputs; the hop sign goes into them
    auto put_factor = [&](int k, double fk) {
        const float s = (float)fk;
        fac[0][k] = (isc.which & 1) ? s : 1.f;
        fac[1][k] = ((isc.which & 2) ? s : 1.f) * (hop_sign < 0 ? -1.f : 1.f);
        sc[k] = 0.f;
    };
    if (isc.npart) {
        for (int k = wv; k < nr; k += nw) {
            const double fk = gm_factor(isc, k);
            if (lane == 0) put_factor(k, fk);
        }
    } else if (wv == 0 && lane < nr) {
        put_factor(lane, f0);
    }
    // columns of the tile beyond the batch: their inputs are zero, so they stay zero
    if (wv == 0 && lane >= nr && lane < xs) put_factor(lane, 1.0);
    auto block = [&](int sl) {
        return sl < nself ? (self_mode == CS_SELF ? op.M + gs * 9 * nn : op.Minv + gs * nn) : op.M + (gs * 9 + 1 + sl - nself) * nn;
    };
    TileFrags<S, NS> f[MG == 1 ? 2 : MG];
    TileFrags<S, NSI> fi;
#pragma unroll
    for (int u = 0; u < MG; u++)
        if (grp + u * MG < ns) f[u].load(block(grp + u * MG), nd, r, q);
    __syncthreads();
    // body(slot, RHS, row, value) over the wave's entries
    auto staged = [&](auto&& body) {
        auto one = [&](int sl, int e, cx<float> val) {
            if (e >= xs * NDK) return;
            const int k = e / NDK;
            body(sl, k, e - k * NDK, fac[sl >= nself][k] * val);
        };
#pragma unroll
        for (int a = 0; a < PS; a++)
            if (wv + a * nw < ns)
#pragma unroll
                for (int u = 0; u < SR; u++) one(wv + a * nw, lane + 64 * u, pre[a][u]);
        for (int sl = wv; sl < ns; sl += nw) {   // what was not asked for ahead
            const int e0 = sl < wv + PS * nw ? 64 * SR : 0;
            if (e0 >= xs * NDK) continue;
            const cx<float>* v = input(sl);
            for (int e = lane + e0; e < xs * NDK; e += 64) one(sl, e, entry(v, e));
        }
    };
    // FP16 form: column k of every slot is divided by sc[k], the largest modulus
    // of the column's reals over the slots, so that the rounded inputs lie in
    // [-1, 1] whatever the vector's magnitude; the products are scaled back in FP32
    if constexpr (F16) {
        staged([&](int, int k, int, cx<float> v) {
            const float m = fmaxf(fabsf(v.re), fabsf(v.im));
            if (m > 0.f) atomicMax(reinterpret_cast<int*>(sc) + k, __float_as_int(m));
        });
        __syncthreads();
    }
    staged([&](int sl, int k, int c, cx<float> v) {
        float s = 1.f;
        if constexpr (F16) s = sc[k] > 0.f ? 1.f / sc[k] : 0.f;
        S* o = X + (sl * NDK + c) * cols + k;
        o[0] = F16 ? S(v.re * s) : S(v.re);
        o[xs] = F16 ? S(v.im * s) : S(v.im);
    });
    __syncthreads();
    f32x4 c0 = {0.f, 0.f, 0.f, 0.f}, c1 = {0.f, 0.f, 0.f, 0.f};
    // MG = 1 sums every slot from zero: chains of 2 nd products, not 18 nd, round
    // less (the groups of MG = 3 cut them as well)
    auto multiply = [&](const TileFrags<S, NS>& a, int sl) {
        const S* x = X + sl * NDK * cols;
        if constexpr (MG == 1) {
            f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
            a.template multiply<PACK>(x, xs, lane, s0, s1);
            c0 += s0;
            c1 += s1;
        } else {
            a.template multiply<PACK>(x, xs, lane, c0, c1);
        }
    };
    auto load_inverse = [&]() {
        if (post_inv) fi.load(op.Minv + gs * nn, nd, r, q, grp, MG);
    };
    if constexpr (MG == 1) {
        // block sl + 1 loads while block sl multiplies
        for (int sl = 0; sl < ns; sl += 2) {
            if (sl + 1 < ns) f[1].load(block(sl + 1), nd, r, q);
            multiply(f[0], sl);
            if (sl + 1 >= ns) break;
            if (sl + 2 < ns) f[0].load(block(sl + 2), nd, r, q);
            multiply(f[1], sl + 1);
        }
        load_inverse();
    } else {
#pragma unroll
        for (int u = 0; u < MG; u++) {
            if (grp + u * MG < ns) multiply(f[u], grp + u * MG);
            if (u == 0) load_inverse();   // into the first slot's registers
        }
    }
    // the groups' partial tiles, added in order by group 0
    auto meet = [&]() {
        if constexpr (MG == 1) {
            __syncthreads();
            return;
        }
        if (grp) {
            f32x4* o = red + ((grp - 1) * ntile + w) * (PACK ? 1 : 2) * 64 + lane;
            o[0] = c0;
            if constexpr (!PACK) o[64] = c1;
        }
        __syncthreads();
        if (grp == 0)
            for (int u = 1; u < MG; u++) {
                const f32x4* o = red + ((u - 1) * ntile + w) * (PACK ? 1 : 2) * 64 + lane;
                c0 += o[0];
                if constexpr (!PACK) c1 += o[64];
            }
    };
    meet();
    // the lane's column: RHS k, real part (and in c1, or in lane + xs, the imaginary one)
    const int k = PACK ? (j & (xs - 1)) : j;
    const bool have = grp == 0 && (PACK ? j < cols : true);
    if (grp == 0) {
        if constexpr (F16) {
            c0 *= sc[k];
            c1 *= sc[k];
        }
        if (self_mode == CS_IDENT && have && k < nr && ((on >> k) & 1u)) {
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const int row = 16 * w + 4 * q + v;
                if (row < nd) {
                    const cx<float> a = fac[0][k] * in1[(size_t)k * ld + gs * nd + row];
                    c0[v] += (PACK && j >= xs) ? a.im : a.re;
                    if constexpr (!PACK) c1[v] += a.im;
                }
            }
        }
    }
    auto store = [&]() {
        if (grp) return;
#pragma unroll
        for (int v = 0; v < 4; v++) {
            const float im = PACK ? __shfl(c0[v], lane + xs, 64) : c1[v];
            const int row = 16 * w + 4 * q + v;
            if (j < xs && k < nr && ((on >> k) & 1u) && row < nd)
                out[(size_t)k * ld + gs * nd + row] = cx<float>{c0[v], im};
        }
    };
    if (!post_inv) {
        store();
        return;
    }
    // post multiplication by the self-block inverse: the result is the new X
    // (zero rows up to the last step; FP16 form scaled per column as above)
    for (int e = nd * cols + t; e < max(NS, NSI * MG) * K * cols; e += nt) X[e] = S(0.f);
    float s = 1.f;
    if constexpr (F16) {
        __syncthreads();
        if (t < 16) sc[t] = 0.f;
        __syncthreads();
        if (have) {
            float m = 0.f;
#pragma unroll
            for (int v = 0; v < 4; v++)
                if (16 * w + 4 * q + v < nd) m = fmaxf(m, PACK ? fabsf(c0[v]) : fmaxf(fabsf(c0[v]), fabsf(c1[v])));
            if (m > 0.f) atomicMax(reinterpret_cast<int*>(sc) + k, __float_as_int(m));
        }
        __syncthreads();
        s = sc[k] > 0.f ? 1.f / sc[k] : 0.f;
    }
    if (have)
#pragma unroll
        for (int v = 0; v < 4; v++) {
            const int row = 16 * w + 4 * q + v;
            if (row < nd) {
                X[row * cols + j] = F16 ? S(c0[v] * s) : S(c0[v]);
                if constexpr (!PACK) X[row * cols + xs + j] = F16 ? S(c1[v] * s) : S(c1[v]);
            }
        }
    __syncthreads();
    c0 = f32x4{0.f, 0.f, 0.f, 0.f};
    c1 = c0;
    fi.template multiply<PACK>(X, xs, lane, c0, c1, grp, MG);
    meet();
    if constexpr (F16) {
        c0 *= sc[k];
        c1 *= sc[k];
    }
    store();
}

template <class S, int NS, bool PACK, int ND, int MG>
static void mfma_go(const CoarseOp<float, S>& op, int nsite, int par, int self_mode, const cx<float>* in1, int hop_sign,
                    const cx<float>* in2, bool post_inv, cx<float>* out, hipStream_t s, Mask mk, int nr, long ld, InScale isc) {
    const int ntile = (op.nd + 15) / 16;
    // the inverse's steps are dealt round robin: its last ones may lie past NDK
    const int rows = std::max(9 * NS, (NS + MG - 1) / MG * MG) * MfmaK<S>::K;
    const size_t lds = sizeof(S) * rows * 2 * mfma_cols(nr) + sizeof(f32x4) * (MG - 1) * ntile * (PACK ? 1 : 2) * 64;
    static std::mutex mu;
    static size_t configured = 65536;
    {
        std::lock_guard<std::mutex> lock(mu);
        if (lds > configured && hipFuncSetAttribute((const void*)k_coarse_apply_mfma<S, NS, PACK, ND, MG>,
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) == hipSuccess)
            configured = lds;
    }
    k_coarse_apply_mfma<S, NS, PACK, ND, MG><<<nsite + (isc.npart ? nr : 0), 64 * MG * ntile, lds, s>>>(
        op, par, self_mode, in1, hop_sign, in2, post_inv ? 1 : 0, out, mk, ld, nr, isc, nsite);
}

// instruction steps of a block column, rounded up to the compiled forms.  40
// unknowns (20 test vectors, the default of dd_default_params) take their own up to
// eight right-hand sides: with bounds and strides known, FP16 storage takes 54 us
// against 68 (4096 sites, two RHS) and 110 against 143 (8192), FP32 187 against 203
// (8192, four RHS)
template <class S>
static void mfma_launch(const CoarseOp<float, S>& op, int nsite, int par, int self_mode, const cx<float>* in1, int hop_sign,
                        const cx<float>* in2, bool post_inv, cx<float>* out, hipStream_t s, Mask mk, int nr, long ld,
                        InScale isc) {
    auto pick = [&](auto ns) {
        constexpr int NS = decltype(ns)::value;
        const bool one = op.nd <= 16;
        const bool split = nsite < (one ? 2048 : 1024) || (one && NS * MfmaK<S>::K * mfma_cols(nr) >= 128);
        auto go = [&](auto pack, auto n) {
            constexpr bool P = decltype(pack)::value;
            constexpr int ND = decltype(n)::value;
            if (split) mfma_go<S, NS, P, ND, 3>(op, nsite, par, self_mode, in1, hop_sign, in2, post_inv, out, s, mk, nr, ld, isc);
            else mfma_go<S, NS, P, ND, 1>(op, nsite, par, self_mode, in1, hop_sign, in2, post_inv, out, s, mk, nr, ld, isc);
        };
        constexpr std::integral_constant<int, 0> any{};
        if constexpr (NS == (40 + MfmaK<S>::K - 1) / MfmaK<S>::K)
            if (op.nd == 40 && nr <= 8) return go(std::true_type{}, std::integral_constant<int, 40>{});
        if (nr <= 8) go(std::true_type{}, any);
        else go(std::false_type{}, any);
    };
    const int steps = (op.nd + MfmaK<S>::K - 1) / MfmaK<S>::K;
    if constexpr (std::is_same<S, float>::value) {
        if (steps <= 1) pick(std::integral_constant<int, 1>{});
        else if (steps <= 2) pick(std::integral_constant<int, 2>{});
        else if (steps <= 4) pick(std::integral_constant<int, 4>{});
        else if (steps <= 5) pick(std::integral_constant<int, 5>{});
        else if (steps <= 8) pick(std::integral_constant<int, 8>{});
        else if (steps <= 10) pick(std::integral_constant<int, 10>{});
        else if (steps <= 12) pick(std::integral_constant<int, 12>{});
        else pick(std::integral_constant<int, 16>{});
    } else {
        if (steps <= 1) pick(std::integral_constant<int, 1>{});
        else if (steps <= 2) pick(std::integral_constant<int, 2>{});
        else if (steps <= 3) pick(std::integral_constant<int, 3>{});
        else pick(std::integral_constant<int, 4>{});
    }
}

// ---------------------------------------------------------------------------
// The same stencil split by rows: workgroup = (site, chunk of RC rows) with RC
// rows of a block column making one 128-byte line, so a small coarse lattice
// still spreads over every CU.  Lane (rl, cg) of a wavefront accumulates row
// rl of the chunk over the columns q = cg, cg + CG, ... of the site's panel
// (self block, then the 8 hop blocks, or the 8 folded blocks B_k); the column
// groups meet through lane shuffles and the wavefronts in LDS.  No post
// multiplication: the folded blocks carry the self inverse where it is needed.
// ---------------------------------------------------------------------------
template <class T, class S, int RC, bool FOLD = true>
__global__ void __launch_bounds__(256) k_coarse_rows(CoarseOp<T, S> op, int par, int self_mode,
                                                     const cx<T>* __restrict__ in1, int hop_sign, int fold,
                                                     const cx<T>* in2, cx<T>* out, Mask mk, long ld, InScale isc,
                                                     int nwg) {
    constexpr int CG = 64 / RC;          // column groups per wavefront
    constexpr int PF = (CG >= 4) ? 12 * (8 / CG) : 24;   // block entries a lane loads at once
    __shared__ int run;
    if constexpr (FOLD) {
        if ((int)blockIdx.x >= nwg) {   // the extra workgroup
            gm_fold(isc, blockIdx.y);
            return;
        }
    }
    const bool early = wg_enter<FOLD>(mk, blockIdx.y, run);
    if (!FOLD && !early) return;
    {
        const long off = blockIdx.y * ld;
        if (in1) in1 += off;
        if (in2) in2 += off;
        out += off;
    }
    __shared__ cx<T> X[9 * 64];          // staged inputs [slot][nd] (nd <= 64), hop sign folded in
    __shared__ cx<T> part[4][RC];
    __shared__ const cx<T>* vin[9];
    const Geom g = op.g;
    const int nd = op.nd;
    const int nrc = (nd + RC - 1) / RC;
    const int site = blockIdx.x / nrc, rc = blockIdx.x - site * nrc;
    int p, i;
    if (par < 0) { p = site >= g.vh; i = site - p * g.vh; }
    else { p = par; i = site; }
    const size_t gs = (size_t)p * g.vh + i;
    const size_t nn = (size_t)nd * nd;
    const int nself = (self_mode == CS_SELF) ? 1 : 0;
    const cx<S>* panel = fold ? op.B + (size_t)i * 8 * nn : op.M + (gs * 9 + 1 - nself) * nn;
    // input vectors of the panel's column slots: thread k < 8 finds neighbour k
    if (threadIdx.x == 0 && nself) vin[0] = in1 + gs * nd;
    if (hop_sign != 0 && threadIdx.x < 8) {
        int x[4];
        cb_coords(g, p, i, x);
        vin[nself + threadIdx.x] = in2 + nb_global(g, p, x, threadIdx.x) * nd;
    }
    const int ns = nself + (hop_sign != 0 ? 8 : 0);
    const int Q = ns * nd;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, nw = blockDim.x >> 6;
    const int rl = lane % RC, cg = lane / RC;
    const int row = rc * RC + rl;
    const bool rok = row < nd;
    const int qs = w * CG + cg, qstep = nw * CG;
    const cx<S>* A = panel + (rok ? row : 0);
    cx<S> a[PF];
    auto load = [&](int qb) {
#pragma unroll
        for (int u = 0; u < PF; u++) {
            const int q = qb + u * qstep;
            a[u] = (rok && q < Q) ? A[(size_t)q * nd] : cx<S>{S(0), S(0)};
        }
    };
    // factors of the two inputs (stored GMRES basis vectors carry theirs in the state)
    T f1 = T(1), f2 = T(1);
    auto ahead = [&]() {   // in flight while the inputs are staged
        load(qs);
        if (isc.st) {
            const T f = T(FOLD ? gm_factor(isc, blockIdx.y) : isc.st[blockIdx.y].sc[isc.j]);
            if (isc.which & 1) f1 = f;
            if (isc.which & 2) f2 = f;
        }
        if (hop_sign < 0) f2 = -f2;
    };
    if (early) ahead();
    __syncthreads();
    if constexpr (FOLD) {
        if (!run) return;
        if (!early) ahead();
    }
    for (int e = t; e < Q; e += blockDim.x) {
        const int s2 = e / nd;
        const cx<T> v = vin[s2][e - s2 * nd];
        X[e] = ((s2 >= nself) ? f2 : f1) * v;
    }
    __syncthreads();
    cx<T> acc = czero<T>();
    for (int qb = qs; qb < Q; qb += PF * qstep) {
        if (qb != qs) load(qb);
#pragma unroll
        for (int u = 0; u < PF; u++) {
            const int q = qb + u * qstep;
            if (q < Q) acc += ccast<T>(a[u]) * X[q];
        }
    }
#pragma unroll
    for (int o = RC; o < 64; o <<= 1) {
        acc.re += __shfl_xor(acc.re, o, 64);
        acc.im += __shfl_xor(acc.im, o, 64);
    }
    if (cg == 0) part[w][rl] = acc;
    __syncthreads();
    if (w == 0 && cg == 0 && rok) {
        cx<T> tot = (self_mode == CS_IDENT) ? f1 * in1[gs * nd + row] : czero<T>();
        for (int q = 0; q < nw; q++) tot += part[q][rl];
        out[gs * nd + row] = tot;
    }
}

template <class T, class S>
static void launch_rows(const CoarseOp<T, S>& op, int par, int self_mode, const cx<T>* in1, int hop_sign, int fold,
                        const cx<T>* in2, cx<T>* out, hipStream_t s, Mask mk, int nr, long ld, InScale isc) {
    constexpr int RC = 128 / (int)sizeof(cx<S>);   // rows per 128-byte line
    const int nsite = (par < 0) ? 2 * op.g.vh : op.g.vh;
    const int nrc = (op.nd + RC - 1) / RC;
    auto go = [&](auto kernel) {
        dim3 grid(nsite * nrc + (isc.npart ? 1 : 0), nr);
        kernel<<<grid, 256, 0, s>>>(op, par, self_mode, in1, hop_sign, fold, in2, out, mk, ld, isc, nsite * nrc);
    };
    if (isc.npart) go(k_coarse_rows<T, S, RC, true>);
    else go(k_coarse_rows<T, S, RC, false>);
}

// B_k(x) = Minv(x) M_{1+k}(x): workgroup (even site i, hop k), FP64 sums
template <class T>
__global__ void k_coarse_fold(int nd, const cx<T>* __restrict__ M, const cx<T>* __restrict__ Minv,
                              cx<T>* __restrict__ B) {
    const int i = blockIdx.x, k = blockIdx.y;
    const size_t nn = (size_t)nd * nd;
    const cx<T>* Mi = Minv + (size_t)i * nn;
    const cx<T>* Mk = M + ((size_t)i * 9 + 1 + k) * nn;
    cx<T>* Bk = B + ((size_t)i * 8 + k) * nn;
    for (int e = threadIdx.x; e < (int)nn; e += blockDim.x) {
        const int c = e / nd, r = e - c * nd;   // column-major entry (r, c)
        cx<double> s = czero<double>();
        for (int q = 0; q < nd; q++) s += ccast<double>(Mi[(size_t)q * nd + r]) * ccast<double>(Mk[(size_t)c * nd + q]);
        Bk[e] = ccast<T>(s);
    }
}

template <class T>
void coarse_fold_inverse(const Geom& g, int nd, const cx<T>* M, const cx<T>* Minv, cx<T>* B, hipStream_t s) {
    dim3 grid(g.vh, 8);
    k_coarse_fold<T><<<grid, 256, 0, s>>>(nd, M, Minv, B);
}

template <class T, class S>
bool coarse_uses_mfma(const CoarseOp<T, S>& op, int nr) {
    return std::is_same<T, float>::value && op.mfma && nr >= 2 && nr <= 16 && op.nd <= 64;
}

template <class T, class S>
void coarse_apply_folded(const CoarseOp<T, S>& op, const cx<T>* in1, int hop_sign, const cx<T>* in2, cx<T>* out,
                         hipStream_t s, Mask mk, int nr, long ld, InScale isc) {
    if (!op.B || op.nd > 64) throw std::invalid_argument("coarse_apply_folded: no folded blocks on this level");
    launch_rows(op, 0, in1 ? CS_IDENT : CS_NONE, in1, hop_sign, 1, in2, out, s, mk, nr, ld, isc);
}

template <class T, class S>
void coarse_apply(const CoarseOp<T, S>& op, int par, int self_mode, const cx<T>* in1, int hop_sign, const cx<T>* in2,
                  bool post_inv, cx<T>* out, hipStream_t s, Mask mk, int nr, long ld, InScale isc) {
    const bool rows = !post_inv && self_mode != CS_SELFINV && op.nd <= 64;
    int nsite = (par < 0) ? 2 * op.g.vh : op.g.vh;
    if constexpr (std::is_same<T, float>::value) {
        // the matrix-core form serves FP32 arithmetic with 2..16 right-hand sides and nd <= 64
        if (op.mfma && nr >= 2 && nr <= 16 && op.nd <= 64) {
            mfma_launch<S>(op, nsite, par, self_mode, in1, hop_sign, in2, post_inv, out, s, mk, nr, ld, isc);
            return;
        }
    }
    // without the post multiplication by the inverse the row-split form applies
    if (rows) {
        launch_rows(op, par, self_mode, in1, hop_sign, 0, in2, out, s, mk, nr, ld, isc);
        return;
    }
    // the vector-unit kernel reads the site's blocks as one panel: the self
    // inverse is not stored next to the hop blocks
    if (self_mode == CS_SELFINV && hop_sign != 0)
        throw std::invalid_argument("coarse_apply: the self-block inverse combines with no hop term");
    int nslot = ((self_mode == CS_SELF || self_mode == CS_SELFINV) ? 1 : 0) + (hop_sign != 0 ? 8 : 0);
    // at most one prefetch batch of (block, column) pairs per wavefront where the
    // workgroup size allows
    int nw = std::max(1, std::min(CA_WAVES, (nslot * op.nd + CaPre<S>::N - 1) / CaPre<S>::N));
    if (post_inv) nw = std::max(nw, std::min(CA_WAVES, (op.nd + CaPre<S>::INV - 1) / CaPre<S>::INV));
    auto go = [&](auto kernel) {
        dim3 grid(nsite + (isc.npart ? 1 : 0), nr);
        kernel<<<grid, 64 * nw, 0, s>>>(op, par, self_mode, in1, hop_sign, in2, post_inv ? 1 : 0, out, mk, ld, isc, nsite);
    };
    if (isc.npart) go(k_coarse_apply<T, S, true>);
    else go(k_coarse_apply<T, S, false>);
}

// ---------------------------------------------------------------------------
// Persistent coarsest-level GMRES cycle (one cooperative launch).
//
// On small coarse lattices every Arnoldi step of the odd-even GMRES is a
// handful of tiny launches whose latency dominates.  This kernel runs all the
// steps of one restart cycle, for every RHS of the batch, inside one launch of
// G co-resident workgroups that meet at grid barriers:
//   A  t_e = A_ee^{-1} D_eo v_j          (even sites, spread over workgroups)
//   B  w   = A_oo v_j - D_oe t_e          (odd sites)
//   C  partial inner products V_i^H w    (odd entries cut into G chunks)
//   D  h = sum of the partials (fixed order, in every workgroup), w -= V h,
//      partial ||w||^2
//   E  ||w||, Givens update of the Hessenberg column (identical arithmetic
//      in every workgroup; workgroup 0 writes the GmDev state), w /= ||w||
// Each step is five barriers; the stop test is the device GMRES's own.  The
// barrier is a counter/generation pair updated with device-scope atomics; a
// wait that exceeds its spin limit raises `abort` and every workgroup leaves,
// so the kernel always drains.
// ---------------------------------------------------------------------------
static constexpr int COOP_NT = 256;
static constexpr int COOP_MAXR = 16;

__device__ __forceinline__ bool coop_barrier(unsigned* bar, int* abort_flag, unsigned nblk) {
    __syncthreads();
    __shared__ int ok_s;
    if (threadIdx.x == 0) {
        int ok = 1;
        __threadfence();
        const unsigned g = __hip_atomic_load(bar + 1, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned arrived = __hip_atomic_fetch_add(bar, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        if (arrived == nblk - 1) {
            __hip_atomic_store(bar, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(bar + 1, g + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            long spins = 0;
            while (__hip_atomic_load(bar + 1, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) == g) {
                if (__hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) { ok = 0; break; }
                if (++spins > (1L << 24)) {   // about a second: give up rather than hang
                    __hip_atomic_store(abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    ok = 0;
                    break;
                }
                __builtin_amdgcn_s_sleep(2);
            }
        }
        if (__hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) ok = 0;
        __threadfence();
        ok_s = ok;
    }
    __syncthreads();
    return ok_s != 0;
}

// out(site) = [post Minv] ( self(x) in1 + hop_sign sum_k M_k in2(x_k) ) for one
// site with the workgroup's 4 wavefronts (lane r owns row r; nd <= 64)
template <class T, class S>
__device__ __forceinline__ void coop_site_apply(const CoarseOp<T, S>& op, int p, int i, int self_mode,
                                                const cx<T>* in1, int hop_sign, const cx<T>* in2, bool post_inv,
                                                cx<T>* out, cx<T> (*part)[64], cx<T>* buf, const cx<S>** mat,
                                                const cx<T>** vin) {
    const Geom& g = op.g;
    const int nd = op.nd;
    const int t = threadIdx.x, w = t >> 6, r = t & 63;
    const size_t gs = (size_t)p * g.vh + i;
    const size_t nn = (size_t)nd * nd;
    const int nself = (self_mode == CS_SELF || self_mode == CS_SELFINV) ? 1 : 0;
    const int ns = nself + (hop_sign != 0 ? 8 : 0);
    if (t < ns) {
        if (t < nself) {
            mat[0] = (self_mode == CS_SELF) ? op.M + gs * 9 * nn : op.Minv + gs * nn;
            vin[0] = in1 + gs * nd;
        } else {
            const int k = t - nself;
            int x[4], y[4];
            cb_coords(g, p, i, x);
            nb_coords(g, x, k, y);
            mat[t] = op.M + (gs * 9 + 1 + k) * nn;
            vin[t] = in2 + ((size_t)(1 - p) * g.vh + cb_index(g, y)) * nd;
        }
    }
    __syncthreads();
    const int Q = ns * nd, per = (Q + 3) / 4;
    const int q0 = w * per, q1 = min(Q, q0 + per);
    cx<T> acc = czero<T>();
    if (r < nd) {
        int q = q0;
        while (q < q1) {
            const int sl = q / nd, c0 = q - sl * nd, c1 = min(nd, c0 + (q1 - q));
            const cx<S>* A = mat[sl] + r;
            const cx<T>* v = vin[sl];
            cx<T> a2 = czero<T>();
            for (int c = c0; c < c1; c++) a2 += ccast<T>(A[(size_t)c * nd]) * v[c];
            if (sl >= nself && hop_sign < 0) acc -= a2;
            else acc += a2;
            q += c1 - c0;
        }
    }
    part[w][r] = acc;
    __syncthreads();
    cx<T> tot = czero<T>();
    if (w == 0 && r < nd) {
        tot = (self_mode == CS_IDENT) ? in1[gs * nd + r] : czero<T>();
        for (int q = 0; q < 4; q++) tot += part[q][r];
    }
    if (!post_inv) {
        if (w == 0 && r < nd) out[gs * nd + r] = tot;
        __syncthreads();
        return;
    }
    if (w == 0) buf[r] = tot;
    __syncthreads();
    const int per2 = (nd + 3) / 4, c0 = w * per2, c1 = min(nd, c0 + per2);
    cx<T> a3 = czero<T>();
    if (r < nd) {
        const cx<S>* A = op.Minv + gs * nn + r;
        for (int c = c0; c < c1; c++) a3 += ccast<T>(A[(size_t)c * nd]) * buf[c];
    }
    part[w][r] = a3;
    __syncthreads();
    if (w == 0 && r < nd) {
        cx<T> s2 = czero<T>();
        for (int q = 0; q < 4; q++) s2 += part[q][r];
        out[gs * nd + r] = s2;
    }
    __syncthreads();
}

// sum of v over the workgroup (COOP_NT threads), returned to every thread
__device__ __forceinline__ double coop_sum(double v, double* sh) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0;
    for (int q = 0; q < COOP_NT / 64; q++) s += sh[q];
    return s;
}

__device__ __forceinline__ cx<double> cdivd(cx<double> a, cx<double> b) {
    double d = norm2(b);
    return cx<double>{(a.re * b.re + a.im * b.im) / d, (a.im * b.re - a.re * b.im) / d};
}

template <class T, class S>
__global__ void __launch_bounds__(COOP_NT) k_gmres_coop(CoarseOp<T, S> op, cx<T>* __restrict__ V, long ldv, long nfull,
                                                        cx<T>* tmp, GmDev* st, int nr, int m, cx<double>* part,
                                                        unsigned* bar, int* abort_flag) {
    __shared__ cx<T> ap_part[4][64];
    __shared__ cx<T> ap_buf[64];
    __shared__ const cx<S>* ap_mat[9];
    __shared__ const cx<T>* ap_vin[9];
    __shared__ double sh[COOP_NT / 64];
    __shared__ cx<double> cs_s[COOP_MAXR][32], sn_s[COOP_MAXR][32], g_s[COOP_MAXR][33], h_s[COOP_MAXR][33];
    __shared__ cx<double> col_s[COOP_MAXR][34];
    __shared__ int stop_s[COOP_MAXR], its_s[COOP_MAXR], fixed_s[COOP_MAXR], maxit_s[COOP_MAXR];
    __shared__ double tol_s[COOP_MAXR], hn_s[COOP_MAXR];
    const unsigned G = gridDim.x;
    const int wg = blockIdx.x, t = threadIdx.x;
    const int vh = op.g.vh;
    const long nh = (long)vh * op.nd;
    // private copy of the rotation state (every workgroup updates it identically)
    int j0 = 0;
    for (int r = 0; r < nr; r++) {
        const GmDev* sr = st + r;
        if (t < 32) { cs_s[r][t] = sr->cs[t]; sn_s[r][t] = sr->sn[t]; }
        if (t < 33) g_s[r][t] = sr->g[t];
        if (t == 0) {
            stop_s[r] = sr->stop;
            its_s[r] = sr->its;
            fixed_s[r] = sr->fixed;
            maxit_s[r] = sr->maxit;
            tol_s[r] = sr->tol_abs;
        }
        if (!sr->stop) j0 = sr->j;   // the running RHS share j
    }
    __syncthreads();
    const long chunk = (nh + G - 1) / G;
    const long e0 = min(nh, (long)wg * chunk), e1 = min(nh, e0 + chunk);
    for (int j = j0; j < m; j++) {
        int live = 0;
        for (int r = 0; r < nr; r++) live += !stop_s[r];
        if (!live) break;
        // A: t_e = A_ee^{-1} D_eo v_j (odd part of v_j)
        for (int s = wg; s < vh; s += G)
            for (int r = 0; r < nr; r++) {
                if (stop_s[r]) continue;
                const cx<T>* vj = V + (size_t)j * ldv + (size_t)r * nfull;
                coop_site_apply(op, 0, s, CS_NONE, (const cx<T>*)nullptr, 1, vj, true, tmp + (size_t)r * nfull,
                                ap_part, ap_buf, ap_mat, ap_vin);
            }
        if (!coop_barrier(bar, abort_flag, G)) return;
        // B: w = A_oo v_j - D_oe t_e, written as v_{j+1}
        for (int s = wg; s < vh; s += G)
            for (int r = 0; r < nr; r++) {
                if (stop_s[r]) continue;
                const cx<T>* vj = V + (size_t)j * ldv + (size_t)r * nfull;
                coop_site_apply(op, 1, s, CS_SELF, vj, -1, tmp + (size_t)r * nfull, false,
                                V + (size_t)(j + 1) * ldv + (size_t)r * nfull, ap_part, ap_buf, ap_mat, ap_vin);
            }
        if (!coop_barrier(bar, abort_flag, G)) return;
        // C: partial inner products over this workgroup's chunk of the odd entries
        for (int r = 0; r < nr; r++) {
            if (stop_s[r]) continue;
            const cx<T>* Vr = V + (size_t)r * nfull + nh;
            const cx<T>* w = Vr + (size_t)(j + 1) * ldv;
            for (int i = 0; i <= j; i++) {
                double re = 0, im = 0;
                for (long e = e0 + t; e < e1; e += COOP_NT) {
                    cx<T> a = Vr[(size_t)i * ldv + e], b = w[e];
                    re += (double)a.re * b.re + (double)a.im * b.im;
                    im += (double)a.re * b.im - (double)a.im * b.re;
                }
                re = coop_sum(re, sh);
                im = coop_sum(im, sh);
                if (t == 0) part[((size_t)r * 34 + i) * G + wg] = cx<double>{re, im};
            }
        }
        if (!coop_barrier(bar, abort_flag, G)) return;
        // D: h (fixed-order sum of the partials), w -= V h, partial ||w||^2
        for (int r = 0; r < nr; r++) {
            if (stop_s[r]) continue;
            for (int i = t; i <= j; i += COOP_NT) {
                cx<double> hsum = czero<double>();
                for (unsigned q = 0; q < G; q++) hsum += part[((size_t)r * 34 + i) * G + q];
                h_s[r][i] = hsum;
            }
        }
        __syncthreads();
        for (int r = 0; r < nr; r++) {
            if (stop_s[r]) continue;
            const cx<T>* Vr = V + (size_t)r * nfull + nh;
            cx<T>* w = V + (size_t)(j + 1) * ldv + (size_t)r * nfull + nh;
            double acc = 0;
            for (long e = e0 + t; e < e1; e += COOP_NT) {
                cx<T> we = w[e];
                for (int i = 0; i <= j; i++) we -= ccast<T>(h_s[r][i]) * Vr[(size_t)i * ldv + e];
                w[e] = we;
                acc += (double)norm2(we);
            }
            acc = coop_sum(acc, sh);
            if (t == 0) part[((size_t)r * 34 + 33) * G + wg] = cx<double>{acc, 0.0};
        }
        if (!coop_barrier(bar, abort_flag, G)) return;
        // E: ||w||, Givens update (same arithmetic as the step-by-step kernels), scale
        if (t < nr && !stop_s[t]) {
            const int r = t;
            double n2 = 0;
            for (unsigned q = 0; q < G; q++) n2 += part[((size_t)r * 34 + 33) * G + q].re;
            const double hn = sqrt(n2);
            cx<double>* col = col_s[r];
            for (int i = 0; i <= j; i++) col[i] = h_s[r][i];
            col[j + 1] = cx<double>{hn, 0.0};
            for (int i = 0; i < j; i++) {
                cx<double> a = col[i], b = col[i + 1];
                col[i] = conj(cs_s[r][i]) * a + conj(sn_s[r][i]) * b;
                col[i + 1] = -(sn_s[r][i] * a) + cs_s[r][i] * b;
            }
            cx<double> a = col[j], b = col[j + 1];
            const double den = sqrt(norm2(a) + norm2(b));
            if (den == 0.0) { cs_s[r][j] = cx<double>{1.0, 0.0}; sn_s[r][j] = czero<double>(); }
            else { cs_s[r][j] = cx<double>{a.re / den, a.im / den}; sn_s[r][j] = cx<double>{b.re / den, b.im / den}; }
            col[j] = conj(cs_s[r][j]) * a + conj(sn_s[r][j]) * b;
            col[j + 1] = czero<double>();
            g_s[r][j + 1] = -(sn_s[r][j] * g_s[r][j]);
            g_s[r][j] = conj(cs_s[r][j]) * g_s[r][j];
            its_s[r] += 1;
            const double resid = sqrt(norm2(g_s[r][j + 1]));
            int stop = (fixed_s[r] > 0) ? (its_s[r] >= fixed_s[r]) : ((resid <= tol_s[r]) || (its_s[r] >= maxit_s[r]));
            if (hn == 0.0) stop = 1;
            hn_s[r] = hn;
            if (wg == 0) {
                GmDev* sr = st + r;
                for (int i = 0; i <= j + 1; i++) sr->H[(size_t)j * 33 + i] = col[i];
                sr->cs[j] = cs_s[r][j];
                sr->sn[j] = sn_s[r][j];
                sr->g[j] = g_s[r][j];
                sr->g[j + 1] = g_s[r][j + 1];
                sr->its = its_s[r];
                sr->j = j + 1;
                sr->stop = stop;
                sr->scale = (hn > 0) ? 1.0 / hn : 0.0;
                sr->sc[j + 1] = 1.0;   // this kernel stores its basis vectors normalised
            }
            stop_s[r] = stop;
        }
        __syncthreads();
        for (int r = 0; r < nr; r++) {
            if (stop_s[r]) continue;   // (a RHS that stopped in this step is not scaled, as before)
            cx<T>* w = V + (size_t)(j + 1) * ldv + (size_t)r * nfull + nh;
            const T sc = T(1.0 / hn_s[r]);
            for (long e = e0 + t; e < e1; e += COOP_NT) w[e] = sc * w[e];
        }
        if (!coop_barrier(bar, abort_flag, G)) return;
    }
}

// Largest grid the cooperative launch admits (0 when not supported)
template <class T, class S>
int coarse_gmres_coop_max_grid() {
    int dev = 0, ncu = 0, per = 0, coop = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop) return 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, (const void*)k_gmres_coop<T, S>, COOP_NT, 0) != hipSuccess)
        return 0;
    return per * ncu;
}

template <class T, class S>
hipError_t coarse_gmres_coop(const CoarseOp<T, S>& op, cx<T>* V, long ldv, long nfull, cx<T>* tmp, GmDev* st, int nr,
                             int m, cx<double>* part, unsigned* bar, int* abort_flag, int grid, hipStream_t s) {
    if (nr > COOP_MAXR || op.nd > 64 || m > 32 || grid < 1) return hipErrorInvalidValue;
    CoarseOp<T, S> a0 = op;
    void* args[] = {&a0, &V, &ldv, &nfull, &tmp, &st, &nr, &m, &part, &bar, &abort_flag};
    return hipLaunchCooperativeKernel((const void*)k_gmres_coop<T, S>, dim3(grid), dim3(COOP_NT), args, 0, s);
}

// ---------------------------------------------------------------------------
// self-block inverse: Gauss-Jordan with partial pivoting on [A | I] in FP64
// ---------------------------------------------------------------------------
template <class T>
__global__ void k_coarse_selfinv(Geom g, int nd, const cx<T>* __restrict__ M, cx<T>* __restrict__ Minv, int* bad) {
    extern __shared__ char smem_raw[];
    cx<double>* a = reinterpret_cast<cx<double>*>(smem_raw);  // row-major [nd][2nd]
    __shared__ int piv;
    __shared__ double pmax[1024 / 64];
    __shared__ int pidx[1024 / 64];
    const size_t gs = blockIdx.x;
    const size_t nn = (size_t)nd * nd;
    const int t = threadIdx.x, nt = blockDim.x, w2 = 2 * nd;
    for (int e = t; e < nd * w2; e += nt) {
        int r = e / w2, c = e % w2;
        a[e] = (c < nd) ? ccast<double>(M[gs * 9 * nn + (size_t)c * nd + r]) : ((c - nd == r) ? cx<double>{1.0, 0.0} : czero<double>());
    }
    __syncthreads();
    int singular = 0;
    for (int c = 0; c < nd; c++) {
        // pivot search over rows c..nd-1
        double best = -1.0;
        int bi = c;
        for (int r = c + t; r < nd; r += nt) {
            double v = norm2(a[r * w2 + c]);
            if (v > best) { best = v; bi = r; }
        }
        for (int o = 32; o > 0; o >>= 1) {
            double ob = __shfl_xor(best, o, 64);
            int oi = __shfl_xor(bi, o, 64);
            if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
        }
        if ((t & 63) == 0) { pmax[t >> 6] = best; pidx[t >> 6] = bi; }
        __syncthreads();
        if (t == 0) {
            double b = pmax[0];
            int bidx = pidx[0];
            for (int q = 1; q < (nt + 63) / 64; q++)
                if (pmax[q] > b || (pmax[q] == b && pidx[q] < bidx)) { b = pmax[q]; bidx = pidx[q]; }
            piv = (b > 0.0) ? bidx : -1;
        }
        __syncthreads();
        int pr = piv;
        if (pr < 0) { singular = 1; break; }
        if (pr != c)
            for (int j = t; j < w2; j += nt) {
                cx<double> tmp = a[c * w2 + j]; a[c * w2 + j] = a[pr * w2 + j]; a[pr * w2 + j] = tmp;
            }
        __syncthreads();
        cx<double> pv = a[c * w2 + c];
        double d = norm2(pv);
        cx<double> ip = {pv.re / d, -pv.im / d};
        __syncthreads();
        for (int j = t; j < w2; j += nt) a[c * w2 + j] = a[c * w2 + j] * ip;
        __syncthreads();
        for (int e = t; e < nd * w2; e += nt) {
            int r = e / w2, j = e % w2;
            if (r == c) continue;
            cx<double> f = a[r * w2 + c];
            if (j == c) continue;
            a[e] -= f * a[c * w2 + j];
        }
        __syncthreads();
        for (int r = t; r < nd; r += nt)
            if (r != c) a[r * w2 + c] = czero<double>();
        __syncthreads();
    }
    if (singular) {
        if (t == 0) atomicAdd(bad, 1);
        return;
    }
    for (int e = t; e < (int)nn; e += nt) {
        int c = e / nd, r = e % nd;  // column-major output
        Minv[gs * nn + e] = ccast<T>(a[r * w2 + nd + c]);
    }
}

template <class T>
void coarse_self_inverse(const Geom& g, int nd, const cx<T>* M, cx<T>* Minv, int* bad, hipStream_t s) {
    size_t lds = sizeof(cx<double>) * nd * 2 * nd;
    k_coarse_selfinv<T><<<2 * g.vh, 256, lds, s>>>(g, nd, M, Minv, bad);
}

// ---------------------------------------------------------------------------
// layout conversion of coarse vectors and blocks
// ---------------------------------------------------------------------------
template <class T>
__global__ void k_coarse_import(Geom g, int nd, int n, const double* __restrict__ canon, cx<T>* __restrict__ out) {
    long e = blockIdx.x * (long)blockDim.x + threadIdx.x;
    long vol = 2L * g.vh;
    if (e >= vol * nd) return;
    long s = e / nd;
    int c = (int)(e % nd);
    int x[4];
    canon_coords(g.d, s, x);
    size_t gs = lay_global(g, x);
    const cx<double>* src = reinterpret_cast<const cx<double>*>(canon);
    for (int v = 0; v < n; v++) out[(size_t)v * vol * nd + gs * nd + c] = ccast<T>(src[(size_t)v * vol * nd + s * nd + c]);
}

template <class T>
__global__ void k_coarse_export(Geom g, int nd, int n, const cx<T>* __restrict__ in, double* __restrict__ canon) {
    long e = blockIdx.x * (long)blockDim.x + threadIdx.x;
    long vol = 2L * g.vh;
    if (e >= vol * nd) return;
    long s = e / nd;
    int c = (int)(e % nd);
    int x[4];
    canon_coords(g.d, s, x);
    size_t gs = lay_global(g, x);
    cx<double>* dst = reinterpret_cast<cx<double>*>(canon);
    for (int v = 0; v < n; v++) dst[(size_t)v * vol * nd + s * nd + c] = ccast<double>(in[(size_t)v * vol * nd + gs * nd + c]);
}

// blocks: layout [site][nslot][nd][nd] column-major -> canonical [site][nslot][nd][nd] row-major
template <class T>
__global__ void k_coarse_export_blocks(Geom g, int nd, int nslot, const cx<T>* __restrict__ in, double* __restrict__ canon) {
    long e = blockIdx.x * (long)blockDim.x + threadIdx.x;
    long vol = 2L * g.vh;
    long nn = (long)nd * nd;
    if (e >= vol * nslot * nn) return;
    long s = e / (nslot * nn);
    long rem = e % (nslot * nn);
    int slot = (int)(rem / nn);
    int q = (int)(rem % nn);
    int r = q / nd, c = q % nd;
    int x[4];
    canon_coords(g.d, s, x);
    size_t gs = lay_global(g, x);
    cx<double>* dst = reinterpret_cast<cx<double>*>(canon);
    dst[e] = ccast<double>(in[(gs * nslot + slot) * nn + (size_t)c * nd + r]);
}

template <class T>
__global__ void k_coarse_shift(Geom g, int nd, double dm, cx<T>* M) {
    long e = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (e >= 2L * g.vh * nd) return;
    long s = e / nd;
    int r = (int)(e % nd);
    M[(s * 9) * nd * nd + (size_t)r * nd + r].re += T(dm);
}

template <class T>
void coarse_import_vector(const Geom& g, int nd, int n, const double* canon, cx<T>* out, hipStream_t s) {
    long tot = 2L * g.vh * nd;
    k_coarse_import<T><<<nblk_of(tot, 256), 256, 0, s>>>(g, nd, n, canon, out);
}
template <class T>
void coarse_export_vector(const Geom& g, int nd, int n, const cx<T>* in, double* canon, hipStream_t s) {
    long tot = 2L * g.vh * nd;
    k_coarse_export<T><<<nblk_of(tot, 256), 256, 0, s>>>(g, nd, n, in, canon);
}
template <class T>
void coarse_export_blocks(const Geom& g, int nd, int nslot, const cx<T>* in, double* canon, hipStream_t s) {
    long tot = 2L * g.vh * nslot * nd * nd;
    k_coarse_export_blocks<T><<<nblk_of(tot, 256), 256, 0, s>>>(g, nd, nslot, in, canon);
}
template <class T>
void coarse_shift_diag(const Geom& g, int nd, double dm, cx<T>* M, hipStream_t s) {
    long tot = 2L * g.vh * nd;
    k_coarse_shift<T><<<nblk_of(tot, 256), 256, 0, s>>>(g, nd, dm, M);
}

// ---------------------------------------------------------------------------
// Coarse SAP half sweep (the algebra of the fine kernel on dense site blocks):
//   z_e <- Minv_e (b_e - H z)                 (z_e + t0, t0 = A_ee^{-1} r_e)
//   rho  = b_o - M0_o z_o - H z               (with the new z_e: r_o - H_int t0)
//   MR on M0_o - H_int Minv_e H_int from e_o = 0
//   z_e -= Minv_e H_int e_o,  z_o += e_o
// One workgroup per (block, group of KR right-hand sides).
//
// Bound: with 4 MR steps a 2^4 block of nd = 40 applies 504 blocks of nd x nd per
// half sweep (6.5 MB in FP32), in 17 dependent phases; nothing of it fits on chip,
// so the blocks stream from L2 / MALL and a phase is as fast as the loads the
// workgroup keeps in flight.  One row per thread (320 threads, 8-byte loads,
// a serial walk over a site's columns) kept too few: 2.0 TB/s with one
// workgroup per CU.  Here a phase is one product with many columns at once:
// LC = nd / RPL lanes read a block column as 16-byte words (RPL rows per
// lane), `parts` such lane groups share the panel of one site (group p takes
// the columns p, p + parts, ..., so neighbouring groups read neighbouring
// columns), every lane loads U columns before it uses the first, and the
// partial rows meet in LDS.  Vectors are staged in LDS as [site][row][KR], one
// aligned read per column for all KR.  The hops of the residual are staged for
// all directions at once (in rounds of `H` where LDS is short); the new z_e is
// stored before the odd residual reads it, which makes H z + H_int t0 one pass.
// Rounding: a lane adds one long chain, so the order counts.  The site's own block is
// by far the largest term and comes after the hops; first, every hop was rounded
// at its size, and the FP32 error of a sweep against FP64 was 2.25e-7 (2^4, nd 40)
// instead of 9.8e-8 (1.30e-7 with a sum per block).  FOLD: with one or two
// lane groups the chain is so long that a batch of columns is summed by itself (2x3^3,
// nd 64: 2.11e-7 without, 1.07e-7 with; 1.57e-7 with a sum per block).  16-bit storage
// has errors of 2^-11 and takes no fold.
// Per half sweep, before -> now (4 MR steps): 64x32^3 level 1 (16x8^3, nd 40,
// FP32, 4 RHS) 812 -> 287 us, 5.8 TB/s; 48x24^3 level 1 (2x3^3 blocks from
// tables, FP32, 4 RHS) 824 -> 349 us, 6.8 TB/s; 32x16^3 level 1 (FP16 storage,
// 1 RHS, 16 workgroups) 253 -> 90 us.
// ---------------------------------------------------------------------------
static constexpr int CS_NT = 1024;
static constexpr int CS_PARTS = 12;   // lane groups that share a site's columns, at most
static constexpr size_t CS_LDS = 150 * 1024;   // of the CU's 160 KB

// columns that a lane has in flight at once
__host__ __device__ constexpr int coarse_sap_cols(size_t t, int rows_rhs) { return t == 8 || rows_rhs > 8 ? 3 : 4; }

// rows of a block column in one load; KR vector entries at one row
template <class S, int RPL> struct alignas(sizeof(cx<S>) * RPL) RowPack { cx<S> v[RPL]; };
template <class T, int KR> struct alignas(sizeof(cx<T>) * KR > 16 ? 16 : sizeof(cx<T>) * KR) RhsPack { cx<T> v[KR]; };

// BIG: blocks of many sites with few unknowns, whose neighbour table does not
// fit in LDS beside the fields: neighbours are found again where they are read, and
// the staged hops take no fields of their own.  Three fields and 48 bytes per site
// then hold every block of 2048 rows (1024 sites of 2 unknowns in FP64: 144 KB)
template <class T, class S, int KR, int RPL, int NV, bool BIG, bool FOLD>
__global__ void __launch_bounds__(CS_NT) k_coarse_sap(CoarseOp<T, S> op, const int* __restrict__ blocks, SapTab tab, int bv,
                                                      const cx<T>* __restrict__ b, cx<T>* __restrict__ z, int mr_steps,
                                                      long ld, int nr, Mask mk, int parts, int H) {
    using RP = RowPack<S, RPL>;
    constexpr int XQ = FOLD && KR * sizeof(cx<T>) > 16 ? 16 / sizeof(cx<T>) : KR;
    using XP = RhsPack<T, XQ>;
    const int q0 = blockIdx.y * KR;
    unsigned on = 0;
#pragma unroll
    for (int q = 0; q < KR; q++)
        if (q0 + q < nr && mk.on(q0 + q)) on |= 1u << q;
    if (!on) return;
    b += (size_t)q0 * ld;
    z += (size_t)q0 * ld;
    extern __shared__ __align__(16) char smem_raw[];
    const Geom g = op.g;
    const int nd = op.nd, nt = blockDim.x, t = threadIdx.x;
    const int F = bv * nd * KR;                          // entries of one block field
    cx<T>* so = reinterpret_cast<cx<T>*>(smem_raw);      // odd-site field
    cx<T>* se = so + F;                                  // even-site field
    // staged hop inputs [H][F] (BIG: H = 2, in the two fields, which are free meanwhile)
    cx<T>* sg = BIG ? so : se + F;
    cx<T>* pr = sg + (size_t)H * F;                      // partial rows [parts][F]
    cx<T>* zero = pr + (size_t)parts * F;                // KR zeros (columns past a group's last)
    double* red = reinterpret_cast<double*>(zero + 2 * KR);   // [waves][KR][3]
    int* sidx = reinterpret_cast<int*>(red + 3 * KR * (nt >> 6));   // [2][bv] layout index of a site
    int* cnt = sidx + 2 * bv;                            // [2][bv] inner hops of a site
    unsigned short* lst = reinterpret_cast<unsigned short*>(cnt + 2 * bv);   // [2][bv][8] slot | place << 4
    int* nbg = reinterpret_cast<int*>(lst + 16 * bv);    // [2][8][bv] layout index of its neighbours (not BIG)
    const int blk = blocks[blockIdx.x];
    if (t < KR) zero[t] = czero<T>();
    auto neighbour = [&](int p, int l, int k) {
        int x[4];
        cb_coords(g, p, sidx[p * bv + l], x);
        return nb_index_sel(g, x, k);
    };
    for (int e = t; e < 2 * bv; e += nt) {
        const int p = e / bv, l = e - p * bv;
        sidx[e] = tab.bv ? tab.sites[((size_t)blk * 2 + p) * bv + l] : (blk << g.lbvh) + l;
    }
    __syncthreads();
    for (int e = t; e < 16 * bv; e += nt) {
        const int l = e % bv, k = (e / bv) & 7, p = e / (8 * bv);
        const int j = neighbour(p, l, k);
        if (!BIG) nbg[e] = j;
        int place;
        if (tab.bv) {
            const size_t gy = (size_t)(1 - p) * g.vh + j;
            place = (tab.of[gy] == blk) ? tab.loc[gy] : -1;
        } else {
            place = ((j >> g.lbvh) == blk) ? j - (blk << g.lbvh) : -1;
        }
        lst[(p * bv + l) * 8 + k] = place < 0 ? 0 : (1 + k) | (place << 4);   // slot 0: leaves the block
    }
    __syncthreads();
    for (int e = t; e < 2 * bv; e += nt) {
        int n = 0;
        for (int k = 0; k < 8; k++) {
            const unsigned short w = lst[e * 8 + k];
            if (w) lst[e * 8 + n++] = w;
        }
        cnt[e] = n;
    }
    // the thread's share of a block field: entries t, t + nt, ... (RHS t % KR)
    int vg[NV];              // vector offset of the entry within one parity of one RHS
    const int myq = t % KR;
    const bool myon = (on >> myq) & 1u;
    auto field = [&](int p, int u) {   // whole-vector offset of entry u at parity p
        const int v = t + u * nt, l = v / (nd * KR);
        return (size_t)myq * ld + ((size_t)p * g.vh + sidx[p * bv + l]) * nd + vg[u];
    };
#pragma unroll
    for (int u = 0; u < NV; u++) vg[u] = ((t + u * nt) / KR) % nd;
    __syncthreads();
    const size_t nn = (size_t)nd * nd;
    const int LC = nd / RPL, NG = nt / LC;
    const int grp = t / LC, r0 = (t - grp * LC) * RPL;
    constexpr int U = coarse_sap_cols(sizeof(T), RPL * KR);
    // partial rows of a product, for the lane groups' (site, part) tasks:
    // entry e < count(l) of site l reads the block at base(l) + slot nn and the vector at offset xo
    auto product = [&](auto&& base, auto&& count, auto&& entry) {
        for (int task = grp; task < bv * parts && grp < NG; task += NG) {
            const int l = task / parts, part = task - l * parts;
            const cx<S>* A = base(l) + r0;
            const int n = count(l);
            cx<T> acc[RPL][KR];
#pragma unroll
            for (int r = 0; r < RPL; r++)
#pragma unroll
                for (int q = 0; q < KR; q++) acc[r][q] = czero<T>();
            // the group's columns part, part + parts, ... of every entry, U at a
            // time; the next U are loaded while the current ones multiply
            const int nc = (nd - part + parts - 1) / parts;
            int e = 0, i0 = 0;
            auto fetch = [&](RP (&a)[U], int& xo) -> int {
                if (e >= n) return 0;
                int slot, x0;
                entry(l, e, slot, x0);
                const int c = part + i0 * parts, m = min(U, nc - i0);
                const cx<S>* pa = A + (slot * (int)nn + c * nd);
                xo = x0 + c * KR;
#pragma unroll
                for (int u = 0; u < U; u++) a[u] = *reinterpret_cast<const RP*>(pa + (u < m ? u * (parts * nd) : 0));
                i0 += U;
                if (i0 >= nc) { i0 = 0; e++; }
                return m;
            };
            auto use = [&](const RP (&a)[U], int xo, int m) {
                if constexpr (FOLD) {
                    // the batch by itself, XQ right-hand sides at a time
#pragma unroll
                    for (int q1 = 0; q1 < KR; q1 += XQ) {
                        cx<T> sum[RPL][XQ];
#pragma unroll
                        for (int r = 0; r < RPL; r++)
#pragma unroll
                            for (int q = 0; q < XQ; q++) sum[r][q] = czero<T>();
#pragma unroll
                        for (int u = 0; u < U; u++) {
                            const XP x = *reinterpret_cast<const XP*>(so + (u < m ? xo + u * (parts * KR) + q1 : (int)(zero - so)));
#pragma unroll
                            for (int r = 0; r < RPL; r++) {
                                const cx<T> ar = ccast<T>(a[u].v[r]);
#pragma unroll
                                for (int q = 0; q < XQ; q++) cmac(sum[r][q], ar, x.v[q]);
                            }
                        }
#pragma unroll
                        for (int r = 0; r < RPL; r++)
#pragma unroll
                            for (int q = 0; q < XQ; q++) acc[r][q1 + q] += sum[r][q];
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < U; u++) {
                        const XP x = *reinterpret_cast<const XP*>(so + (u < m ? xo + u * (parts * KR) : (int)(zero - so)));
#pragma unroll
                        for (int r = 0; r < RPL; r++) {
                            const cx<T> ar = ccast<T>(a[u].v[r]);
#pragma unroll
                            for (int q = 0; q < KR; q++) cmac(acc[r][q], ar, x.v[q]);
                        }
                    }
                }
            };
            RP a0[U], a1[U];
            int x0 = 0, x1 = 0, m0 = fetch(a0, x0);
            while (m0) {
                const int m1 = fetch(a1, x1);
                use(a0, x0, m0);
                if (!m1) break;
                m0 = fetch(a0, x0);
                use(a1, x1, m1);
            }
            cx<T>* o = pr + (size_t)part * F + (size_t)(l * nd + r0) * KR;
#pragma unroll
            for (int r = 0; r < RPL; r++)
#pragma unroll
                for (int q = 0; q < KR; q++) o[r * KR + q] = acc[r][q];
        }
    };
    // the thread's entries of the sum of the parts (in order)
    auto gather = [&](cx<T> (&s)[NV]) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < NV; u++) {
            const int v = t + u * nt;
            if (v < F) {
#pragma unroll
                for (int p = 0; p < CS_PARTS; p++)
                    if (p < parts) s[u] += pr[p * F + v];
            }
        }
    };
    auto clear = [&](cx<T> (&s)[NV]) {
#pragma unroll
        for (int u = 0; u < NV; u++) s[u] = czero<T>();
    };
    auto put = [&](cx<T>* f, const cx<T> (&s)[NV], T sgn) {   // f = sgn s, visible to the workgroup
#pragma unroll
        for (int u = 0; u < NV; u++)
            if (t + u * nt < F) f[t + u * nt] = sgn * s[u];
        __syncthreads();
    };
    // s += sum over the slots [s0, 9) of the sites of parity p applied to z, from the last
    // to the first (slot 0: the site itself)
    auto outer = [&](int p, int s0, cx<T> (&s)[NV]) {
        for (int end = 9, sa; end > s0; end = sa) {
            sa = max(s0, end - H);
            const int ns = end - sa;
            // SU entries per thread are loaded before the first is stored
            constexpr int SU = 4;
            for (int e0 = t; e0 < ns * F; e0 += SU * nt) {
                cx<T> v[SU];
                int to[SU];
#pragma unroll
                for (int u = 0; u < SU; u++) {
                    const int e = e0 + u * nt;
                    v[u] = czero<T>();
                    to[u] = -1;
                    if (e >= ns * F) continue;
                    int m = e / nd;
                    const int c = e - m * nd, q = m / (ns * bv);
                    m -= q * (ns * bv);
                    const int sl = sa + m / bv, l = m % bv;
                    to[u] = (m * nd + c) * KR + q;
                    if ((on >> q) & 1u) {
                        const int j = !sl ? sidx[p * bv + l] : BIG ? neighbour(p, l, sl - 1) : nbg[(p * 8 + sl - 1) * bv + l];
                        v[u] = z[(size_t)q * ld + ((size_t)(sl ? 1 - p : p) * g.vh + j) * nd + c];
                    }
                }
#pragma unroll
                for (int u = 0; u < SU; u++)
                    if (to[u] >= 0) sg[to[u]] = v[u];
            }
            __syncthreads();
            product([&](int l) { return op.M + (((size_t)p * g.vh + sidx[p * bv + l]) * 9 + sa) * nn; },
                    [&](int) { return ns; },
                    [&](int l, int e, int& slot, int& x0) {
                        slot = ns - 1 - e;
                        x0 = (int)(sg - so) + (slot * bv + l) * nd * KR;
                    });
            gather(s);
            __syncthreads();   // the staged inputs and the partial rows are free again
        }
    };
    // s += sum of the inner hops of parity p applied to the field f, then M0 f0 where there is f0
    auto inner = [&](int p, const cx<T>* f0, const cx<T>* f, cx<T> (&s)[NV]) {
        const int o0 = f0 ? (int)(f0 - so) : 0, o1 = (int)(f - so), self = f0 ? 1 : 0;
        product([&](int l) { return op.M + ((size_t)p * g.vh + sidx[p * bv + l]) * 9 * nn; },
                [&](int l) { return self + cnt[p * bv + l]; },
                [&](int l, int e, int& slot, int& x0) {
                    if (e == cnt[p * bv + l]) {
                        slot = 0;
                        x0 = o0 + l * nd * KR;
                    } else {
                        const int w = lst[(p * bv + l) * 8 + e];
                        slot = w & 15;
                        x0 = o1 + (w >> 4) * nd * KR;
                    }
                });
        gather(s);
    };
    // s = Minv_e f
    auto minv = [&](const cx<T>* f, cx<T> (&s)[NV]) {
        const int o = (int)(f - so);
        product([&](int l) { return op.Minv + (size_t)sidx[l] * nn; }, [&](int) { return 1; },
                [&](int l, int, int& slot, int& x0) {
                    slot = 0;
                    x0 = o + l * nd * KR;
                });
        clear(s);
        gather(s);
    };
    cx<T> rho[NV], eo[NV], sv[NV];
    // z_e + t0_e = Minv (b_e - H z)
    clear(sv);
    outer(0, 1, sv);
#pragma unroll
    for (int u = 0; u < NV; u++)
        if (t + u * nt < F) sv[u] = (myon ? b[field(0, u)] : czero<T>()) - sv[u];
    put(se, sv, T(1));
    minv(se, sv);
    // stored at once: no other workgroup reads these z, and the odd residual of
    // this one wants z + t0 at the inner hops
#pragma unroll
    for (int u = 0; u < NV; u++)
        if (myon && t + u * nt < F) z[field(0, u)] = sv[u];
    __syncthreads();
    // rho = b_o - M0 z_o - H z - H_int t0
    clear(rho);
    outer(1, 0, rho);
#pragma unroll
    for (int u = 0; u < NV; u++) {
        if (t + u * nt < F) rho[u] = (myon ? b[field(1, u)] : czero<T>()) - rho[u];
        eo[u] = czero<T>();
    }
    put(so, rho, T(1));
    const int lane = t & 63, w = t >> 6, nw = nt >> 6;
    for (int it = 0; it < mr_steps; it++) {
        clear(sv);
        inner(0, nullptr, so, sv);
        put(se, sv, T(1));
        minv(se, sv);
        put(se, sv, T(-1));   // -Minv H rho: the odd pass adds all its terms
        clear(sv);
        inner(1, so, se, sv);
        double d[3] = {0, 0, 0};
#pragma unroll
        for (int u = 0; u < NV; u++)
            if (t + u * nt < F) {
                const cx<T> p = cmulc(sv[u], rho[u]);
                d[0] += p.re;
                d[1] += p.im;
                d[2] += norm2(sv[u]);
            }
        // the lanes of one RHS are KR apart
#pragma unroll
        for (int o = 32; o >= KR; o >>= 1)
#pragma unroll
            for (int c = 0; c < 3; c++) d[c] += __shfl_xor(d[c], o, 64);
        if (lane < KR)
#pragma unroll
            for (int c = 0; c < 3; c++) red[(w * KR + lane) * 3 + c] = d[c];
        __syncthreads();
        double a0 = 0, a1 = 0, a2 = 0;
        for (int v = 0; v < nw; v++) {
            const double* rv = red + (v * KR + myq) * 3;
            a0 += rv[0];
            a1 += rv[1];
            a2 += rv[2];
        }
        if (a2 > 0) {
            const cx<T> alpha = {T(a0 / a2), T(a1 / a2)};
#pragma unroll
            for (int u = 0; u < NV; u++) {
                eo[u] += alpha * rho[u];
                rho[u] -= alpha * sv[u];
            }
        }
        if (it + 1 < mr_steps) put(so, rho, T(1));
    }
    put(so, eo, T(1));
    clear(sv);
    inner(0, nullptr, so, sv);
    put(se, sv, T(1));
    minv(se, sv);
    if (!myon) return;
#pragma unroll
    for (int u = 0; u < NV; u++)
        if (t + u * nt < F) {
            z[field(0, u)] -= sv[u];
            z[field(1, u)] += eo[u];
        }
}

// How a block of bv even and bv odd sites is worked on by one workgroup for a
// group of kr right-hand sides; ok = false where its fields don't fit in LDS
// or registers.
struct SapShape {
    bool ok, big;
    int nt, nv, parts, hops;
    long units;   // block fields that LDS has left for partial rows and staged hops
    size_t lds;
};
template <class T>
static SapShape coarse_sap_shape(int bv, int nd, int kr, int rpl, bool big = false) {
    SapShape s{};
    s.big = big;
    const int lc = nd / rpl, f = bv * nd * kr;
    const size_t unit = sizeof(cx<T>) * f;
    const size_t fixed = sizeof(cx<T>) * 2 * kr + sizeof(double) * 3 * kr * (CS_NT / 64) + (size_t)(big ? 48 : 112) * bv;
    s.units = (long)((CS_LDS - fixed) / unit) - 2;
    if (s.units < (big ? 1 : 2)) return s;
    // Parts: a phase takes the rounds of the lane groups, each the batches of columns
    // that a group loads one after another (a column adds a twentieth of a batch); a
    // round of staged hops, a partial row to add and the size of the workgroup count
    // little.  The weights are a fit to 186 timed shapes (2^4, 2x4^3, 2x3^3, 4^2x2^2,
    // 4^4; 4 to 60 unknowns; every storage; one and eight right-hand sides; all parts):
    // 2 % above the best parts in the mean, 22 % at most.  The fewest rounds alone
    // were 11 % above in the mean and up to 2.1 times: LDS left for one staged hop, or
    // batches half empty.  Few unknowns take two parts wherever these are one round:
    // a single part adds a site's last columns one after another at full size (FP32,
    // N = 2, 4^2x2^2: error 7.59e-8 against 7.14e-8; time the same within 4 %)
    const int u = coarse_sap_cols(sizeof(T), rpl * kr);
    double best = 0;
    for (int p = 1; p <= CS_PARTS && p < s.units + big && p <= nd; p++) {
        const int work = std::max(std::min(bv * p * lc, CS_NT), (f + 2) / 3);
        const int nt = std::min(CS_NT, (work + 63) / 64 * 64), groups = std::max(1, nt / lc);
        // the nine slots of the residual in one round, or in two, three, five
        const long left = s.units - p;
        const int hops = big ? 2 : left >= 9 ? 9 : left >= 5 ? 5 : left >= 3 ? 3 : left >= 2 ? 2 : 1;
        const int columns = (nd + p - 1) / p;
        const int rounds = (bv * p + groups - 1) / groups, staged = (9 + hops - 1) / hops + (8 + hops - 1) / hops;
        const double cost = rounds * ((columns + u - 1) / u + 0.05 * columns) + 0.1 * staged +
                            0.05 * p * ((f + nt - 1) / nt) + 0.05 * nt / 256;
        if (p > 1 && cost >= best && !(p == 2 && nd < 12 && bv * p * lc <= CS_NT)) continue;
        best = cost;
        s.parts = p;
        s.hops = hops;
        s.nt = nt;
    }
    s.nv = (f + s.nt - 1) / s.nt;
    s.lds = unit * (2 + s.parts + (big ? 0 : s.hops)) + fixed;
    s.ok = s.nv <= 3 && lc <= CS_NT;
    return s;
}

template <class T, class S, int KR, int RPL, int NV, bool BIG, bool FOLD>
static void coarse_sap_go(const CoarseOp<T, S>& op, const int* blocks, int nblocks, SapTab tab, int bv, const cx<T>* b,
                          cx<T>* z, int mr_steps, hipStream_t s, int nr, long ld, Mask mk, const SapShape& sh) {
    static std::mutex mu;
    static size_t configured = 65536;
    {
        std::lock_guard<std::mutex> lock(mu);
        // a refusal leaves its error for the launch below to report
        if (sh.lds > configured && hipFuncSetAttribute((const void*)k_coarse_sap<T, S, KR, RPL, NV, BIG, FOLD>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh.lds) == hipSuccess)
            configured = sh.lds;
    }
    dim3 grid(nblocks, (nr + KR - 1) / KR);
    k_coarse_sap<T, S, KR, RPL, NV, BIG, FOLD><<<grid, sh.nt, sh.lds, s>>>(op, blocks, tab, bv, b, z, mr_steps, ld, nr, mk, sh.parts,
                                                               sh.hops);
}

template <class T, class S, int RPL>
static void coarse_sap_pick(const CoarseOp<T, S>& op, const int* blocks, int nblocks, SapTab tab, const cx<T>* b, cx<T>* z,
                            int mr_steps, hipStream_t s, int nr, long ld, Mask mk) {
    const int bv = tab.bv ? tab.bv : op.g.bvh;
    auto go = [&](auto kr, auto nv, auto big, const SapShape& sh) {
        constexpr int KR = decltype(kr)::value, NV = decltype(nv)::value;
        constexpr bool BIG = decltype(big)::value;
        // fewer unknowns gain nothing by it (2x3^3, N = 2: 1.00 of the error with a sum per
        // block without, 1.03 with)
        if constexpr (sizeof(S) > 2)
            if (sh.parts <= 2 && op.nd >= 12)
                return coarse_sap_go<T, S, KR, RPL, NV, BIG, true>(op, blocks, nblocks, tab, bv, b, z, mr_steps, s, nr, ld, mk, sh);
        coarse_sap_go<T, S, KR, RPL, NV, BIG, false>(op, blocks, nblocks, tab, bv, b, z, mr_steps, s, nr, ld, mk, sh);
    };
    auto launch = [&](auto kr, const SapShape& sh) {
        if (sh.nv == 1) go(kr, std::integral_constant<int, 1>{}, std::false_type{}, sh);
        else if (sh.nv == 2) go(kr, std::integral_constant<int, 2>{}, std::false_type{}, sh);
        else go(kr, std::integral_constant<int, 3>{}, std::false_type{}, sh);
    };
    // A group shares a block's loads but is a longer chain in its workgroup: the
    // narrowest group whose workgroups have a CU each (256), or where even the widest
    // has more, that one.  Timed for 8 to 256 blocks per colour, 12 to 60 unknowns,
    // every storage, two to eight RHS.  With a CU for each the wider group takes 1.1
    // (FP64) to 1.5 times as long: 64 blocks of 2^4, N = 20, FP32, four RHS 118 us
    // single, 133 in pairs, 196 in fours.  With two rounds the narrower takes up to
    // twice as long: the same with eight RHS 230 us single, 137 in pairs.  (With few
    // unknowns two workgroups share a CU and the narrower group would win a round
    // longer: 128 blocks, N = 8, FP32, four RHS 55 us single, 61 in pairs.)
    auto groups = [&](int kr) { return nblocks * ((nr + kr - 1) / kr); };
    const SapShape s1 = coarse_sap_shape<T>(bv, op.nd, 1, RPL);
    if (groups(1) > 256) {
        if constexpr (sizeof(S) != 2 || RPL == 4) {
            const SapShape s2 = coarse_sap_shape<T>(bv, op.nd, 2, RPL);
            if constexpr (sizeof(T) == 4) {
                const SapShape s4 = coarse_sap_shape<T>(bv, op.nd, 4, RPL);
                if (nr > 2 && s4.ok && s4.units >= 6 && (groups(2) > 256 || !s2.ok))
                    return launch(std::integral_constant<int, 4>{}, s4);
            }
            if (nr > 1 && s2.ok) return launch(std::integral_constant<int, 2>{}, s2);
        }
    }
    if (s1.ok) return launch(std::integral_constant<int, 1>{}, s1);
    const SapShape sb = coarse_sap_shape<T>(bv, op.nd, 1, RPL, true);
    if (!sb.ok) throw std::invalid_argument("coarse SAP block too large for one workgroup");
    go(std::integral_constant<int, 1>{}, std::integral_constant<int, 3>{}, std::true_type{}, sb);
}

template <class T, class S>
void coarse_sap_half(const CoarseOp<T, S>& op, const int* blocks, int nblocks, const cx<T>* b, cx<T>* z, int mr_steps,
                     hipStream_t s, int nr, long ld, Mask mk, SapTab tab) {
    if (nblocks <= 0) return;
    // rows per lane: 16 bytes of a column (nd is even; FP16 columns of an odd N
    // start on 8-byte boundaries only)
    if constexpr (sizeof(S) == 8) coarse_sap_pick<T, S, 1>(op, blocks, nblocks, tab, b, z, mr_steps, s, nr, ld, mk);
    else if constexpr (sizeof(S) == 4) coarse_sap_pick<T, S, 2>(op, blocks, nblocks, tab, b, z, mr_steps, s, nr, ld, mk);
    else if (op.nd % 4 == 0) coarse_sap_pick<T, S, 4>(op, blocks, nblocks, tab, b, z, mr_steps, s, nr, ld, mk);
    else coarse_sap_pick<T, S, 2>(op, blocks, nblocks, tab, b, z, mr_steps, s, nr, ld, mk);
}

// ---------------------------------------------------------------------------
// transfer between two coarse levels.  P columns: [N][vol_f][ndf] (layout
// order of the finer level); the coarser level has 2N unknowns per site.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void agg_site_c(const AggMap& m, const int xc[4], int s, int x[4]) {
    int l3 = s % m.a[3]; s /= m.a[3];
    int l2 = s % m.a[2]; s /= m.a[2];
    int l1 = s % m.a[1];
    int l0 = s / m.a[1];
    x[0] = xc[0] * m.a[0] + l0;
    x[1] = xc[1] * m.a[1] + l1;
    x[2] = xc[2] * m.a[2] + l2;
    x[3] = xc[3] * m.a[3] + l3;
}

// out_r[h N + k] = sum over half h of the aggregate's rows of conj(P_k) in_r, for a
// group of KR right-hand sides.  Workgroup: coarser site (and a share of the test
// vectors, grid.z); a wave takes every fourth test vector with all its loads in
// flight, one per 64 rows, so a row of P is read once for the group and a sum
// over the aggregate is one wave sum.  Four waves on each test vector in turn
// waited for memory once per vector and RHS: 64x32^3 level 1 -> 2, N = 20, FP32,
// four RHS 264 -> 56 us; 32x16^3, FP16 storage, one RHS 65 -> 13.5 us.
static constexpr int CR_EPT = 16;   // rows per lane: an aggregate has at most 1024
template <class T, class S, int KR>
__global__ void __launch_bounds__(256) k_coarse_restrict(AggMap m, int ndf, int N, const cx<S>* __restrict__ P,
                                                         const cx<T>* __restrict__ in, cx<T>* __restrict__ out, long ldi,
                                                         long ldo, int nr, Mask mk) {
    const int q0 = blockIdx.y * KR;
    unsigned on = 0;
#pragma unroll
    for (int r = 0; r < KR; r++)
        if (q0 + r < nr && mk.on(q0 + r)) on |= 1u << r;
    if (!on) return;
    extern __shared__ __align__(16) char smem_raw[];
    cx<T>* v = reinterpret_cast<cx<T>*>(smem_raw);   // [KR][ne]
    const int gc = blockIdx.x;
    const int pc = gc >= m.c.vh, ic = gc - pc * m.c.vh;
    int xc[4];
    cb_coords(m.c, pc, ic, xc);
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const size_t volf = 2L * m.f.vh;
    const int h0 = ndf / 2, ne = m.asz * ndf;
    size_t off[CR_EPT];
    unsigned upper = 0;   // bit u: the lane's row u lies in half 1
#pragma unroll
    for (int u = 0; u < CR_EPT; u++) {
        off[u] = 0;
        if (64 * u >= ne) continue;
        const int e = min(lane + 64 * u, ne - 1);
        const int s = e / ndf, d = e - s * ndf;
        int x[4];
        agg_site_c(m, xc, s, x);
        off[u] = lay_global(m.f, x) * ndf + d;
        if (d >= h0) upper |= 1u << u;
    }
    // wave w stages the right-hand sides w, w + 4, ...
    for (int r = w; r < KR; r += 4)
#pragma unroll
        for (int u = 0; u < CR_EPT; u++) {
            const int e = lane + 64 * u;
            if (e < ne) v[r * ne + e] = ((on >> r) & 1u) ? in[(size_t)(q0 + r) * ldi + off[u]] : czero<T>();
        }
    __syncthreads();
    for (int k = blockIdx.z * 4 + w; k < N; k += 4 * gridDim.z) {
        const cx<S>* Pk = P + (size_t)k * volf * ndf;
        cx<S> p[CR_EPT];
#pragma unroll
        for (int u = 0; u < CR_EPT; u++)
            if (64 * u < ne) p[u] = Pk[off[u]];
        cx<double> a0[KR], a1[KR];
#pragma unroll
        for (int r = 0; r < KR; r++) a0[r] = a1[r] = czero<double>();
#pragma unroll
        for (int u = 0; u < CR_EPT; u++) {
            const int e = lane + 64 * u;
            if (e >= ne) continue;
            const cx<T> pu = ccast<T>(p[u]);
#pragma unroll
            for (int r = 0; r < KR; r++) {
                const cx<double> pr = ccast<double>(cmulc(pu, v[r * ne + e]));
                if ((upper >> u) & 1u) a1[r] += pr;
                else a0[r] += pr;
            }
        }
#pragma unroll
        for (int r = 0; r < KR; r++) {
            const cx<double> s0 = {wave_sum(a0[r].re), wave_sum(a0[r].im)}, s1 = {wave_sum(a1[r].re), wave_sum(a1[r].im)};
            if (lane == 0 && ((on >> r) & 1u)) {
                cx<T>* o = out + (size_t)(q0 + r) * ldo + (size_t)gc * 2 * N + k;
                o[0] = ccast<T>(s0);
                o[N] = ccast<T>(s1);
            }
        }
    }
}

template <class T, class S>
__global__ void k_coarse_prolong(AggMap m, int ndf, int N, const cx<S>* __restrict__ P, const cx<T>* __restrict__ in,
                                 cx<T>* __restrict__ out, long ldi, long ldo, Mask mk) {
    long e = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const long volf = 2L * m.f.vh;
    if (e >= volf * ndf || !mk.on(blockIdx.y)) return;
    in += blockIdx.y * ldi;
    out += blockIdx.y * ldo;
    long gf = e / ndf;
    int d = (int)(e % ndf);
    int p = gf >= m.f.vh, i = (int)(gf - p * m.f.vh);
    int x[4], xc[4];
    cb_coords(m.f, p, i, x);
    for (int mu = 0; mu < 4; mu++) xc[mu] = x[mu] / m.a[mu];
    size_t gc = lay_global(m.c, xc);
    const int h = d / (ndf / 2);
    cx<T> s = czero<T>();
    for (int k = 0; k < N; k++) s += ccast<T>(P[((size_t)k * volf + gf) * ndf + d]) * in[gc * 2 * N + h * N + k];
    out[gf * ndf + d] = s;
}

template <class T, class S>
void coarse_restrict(const AggMap& m, int ndf, int N, const cx<S>* P, const cx<T>* in, cx<T>* out, hipStream_t s,
                     int nr, long ldi, long ldo, Mask mk) {
    // the test vectors are split until about 512 workgroups run
    const int ks = std::max(1, std::min((N + 3) / 4, 512 / std::max(1, 2 * m.c.vh)));
    auto go = [&](auto kr) {
        constexpr int KR = decltype(kr)::value;
        dim3 grid(2 * m.c.vh, (nr + KR - 1) / KR, ks);
        const size_t lds = sizeof(cx<T>) * KR * m.asz * ndf;
        k_coarse_restrict<T, S, KR><<<grid, 256, lds, s>>>(m, ndf, N, P, in, out, ldi, ldo, nr, mk);
    };
    // (at most 32 KB of staged rows: 1024 rows of four FP32 or two FP64 vectors)
    if constexpr (sizeof(T) == 4)
        if (nr >= 3) return go(std::integral_constant<int, 4>{});
    if (nr >= 2) go(std::integral_constant<int, 2>{});
    else go(std::integral_constant<int, 1>{});
}
template <class T, class S>
void coarse_prolong(const AggMap& m, int ndf, int N, const cx<S>* P, const cx<T>* in, cx<T>* out, hipStream_t s,
                    int nr, long ldi, long ldo, Mask mk) {
    long tot = 2L * m.f.vh * ndf;
    dim3 grid(nblk_of(tot, 256), nr);
    k_coarse_prolong<T, S><<<grid, 256, 0, s>>>(m, ndf, N, P, in, out, ldi, ldo, mk);
}

// modified Gram-Schmidt per (coarser site, half): rows = aggregate sites x ndf/2
template <class T>
__global__ void k_coarse_gs(AggMap m, int ndf, int N, const cx<T>* __restrict__ tv, cx<T>* __restrict__ P, int* bad) {
    __shared__ double red[2 * 16];
    const int gc = blockIdx.x, h = blockIdx.y;
    const int pc = gc >= m.c.vh, ic = gc - pc * m.c.vh;
    int xc[4];
    cb_coords(m.c, pc, ic, xc);
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, nw = (blockDim.x + 63) >> 6;
    const int h0 = ndf / 2;
    const int rows = m.asz * h0;
    const bool act = t < rows;
    const long volf = 2L * m.f.vh;
    size_t off = 0;
    if (act) {
        int s = t / h0, d = h * h0 + t % h0;
        int x[4];
        agg_site_c(m, xc, s, x);
        size_t gf = lay_global(m.f, x);
        off = gf * ndf + d;
    }
    for (int k = 0; k < N; k++) {
        cx<double> q = act ? ccast<double>(tv[(size_t)k * volf * ndf + off]) : czero<double>();
        for (int j = 0; j < k; j++) {
            cx<double> pj = act ? ccast<double>(P[(size_t)j * volf * ndf + off]) : czero<double>();
            cx<double> d = cmulc(pj, q);
            d.re = wave_sum(d.re);
            d.im = wave_sum(d.im);
            __syncthreads();
            if (lane == 0) { red[2 * w] = d.re; red[2 * w + 1] = d.im; }
            __syncthreads();
            d = czero<double>();
            for (int ww = 0; ww < nw; ww++) { d.re += red[2 * ww]; d.im += red[2 * ww + 1]; }
            q -= d * pj;
        }
        double n2 = wave_sum(norm2(q));
        __syncthreads();
        if (lane == 0) red[2 * w] = n2;
        __syncthreads();
        n2 = 0;
        for (int ww = 0; ww < nw; ww++) n2 += red[2 * ww];
        double inv = 0;
        if (n2 > 0) inv = 1.0 / sqrt(n2);
        else if (t == 0) atomicAdd(bad, 1);
        if (act) P[(size_t)k * volf * ndf + off] = ccast<T>(inv * q);
    }
}

template <class T>
void coarse_gram_schmidt(const AggMap& m, int ndf, int N, const cx<T>* tv, cx<T>* P, int* bad, hipStream_t s) {
    int nt = ((m.asz * (ndf / 2) + 63) / 64) * 64;
    dim3 grid(2 * m.c.vh, 2);
    k_coarse_gs<T><<<grid, nt, 0, s>>>(m, ndf, N, tv, P, bad);
}

// next coarser operator from a coarse one: workgroup (coarser site, column b)
template <class T>
__global__ void k_coarse_assemble(CoarseOp<T> op, AggMap m, int N, const cx<T>* __restrict__ P, cx<T>* __restrict__ Mc) {
    extern __shared__ char smem_raw[];
    const int ndf = op.nd;
    const int h0 = ndf / 2;
    const size_t nnf = (size_t)ndf * ndf;
    cx<double>* red = reinterpret_cast<cx<double>*>(smem_raw);   // [nw][2N]
    const int gc = blockIdx.x, bcol = blockIdx.y;
    const int ndc = 2 * N, hb = bcol / N, kb = bcol % N;
    const int pc = gc >= m.c.vh, ic = gc - pc * m.c.vh;
    int xc[4];
    cb_coords(m.c, pc, ic, xc);
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, nw = (blockDim.x + 63) >> 6;
    const bool act = t < m.asz * ndf;
    const long volf = 2L * m.f.vh;
    int s = act ? t / ndf : 0, r = act ? t % ndf : 0;
    int x[4];
    agg_site_c(m, xc, s, x);
    const int p = site_parity(x);
    const size_t gf = (size_t)p * m.f.vh + cb_index(m.f, x);
    // column b of P restricted to half hb, at site y
    auto pcol = [&](size_t gy, int c) -> cx<T> {
        return (c / h0 == hb) ? P[((size_t)kb * volf + gy) * ndf + c] : czero<T>();
    };
    for (int slot = 0; slot < 9; slot++) {
        cx<T> wv = czero<T>();
        if (act) {
            if (slot == 0) {
                for (int c = 0; c < ndf; c++) wv += op.M[(gf * 9) * nnf + (size_t)c * ndf + r] * pcol(gf, c);
                for (int k = 0; k < 8; k++) {
                    int y[4];
                    nb_coords(op.g, x, k, y);
                    if (y[0] / m.a[0] != xc[0] || y[1] / m.a[1] != xc[1] || y[2] / m.a[2] != xc[2] || y[3] / m.a[3] != xc[3]) continue;
                    size_t gy = (size_t)(1 - p) * m.f.vh + cb_index(m.f, y);
                    for (int c = 0; c < ndf; c++) wv += op.M[(gf * 9 + 1 + k) * nnf + (size_t)c * ndf + r] * pcol(gy, c);
                }
            } else {
                int k = slot - 1;
                int y[4];
                nb_coords(op.g, x, k, y);
                if (y[0] / m.a[0] != xc[0] || y[1] / m.a[1] != xc[1] || y[2] / m.a[2] != xc[2] || y[3] / m.a[3] != xc[3]) {
                    size_t gy = (size_t)(1 - p) * m.f.vh + cb_index(m.f, y);
                    for (int c = 0; c < ndf; c++) wv += op.M[(gf * 9 + 1 + k) * nnf + (size_t)c * ndf + r] * pcol(gy, c);
                }
            }
        }
        for (int a = 0; a < ndc; a++) {
            const int ha = a / N, ka = a % N;
            cx<double> d = czero<double>();
            if (act && r / h0 == ha) d = cmulc(ccast<double>(P[((size_t)ka * volf + gf) * ndf + r]), ccast<double>(wv));
            d.re = wave_sum(d.re);
            d.im = wave_sum(d.im);
            if (lane == 0) red[w * ndc + a] = d;
        }
        __syncthreads();
        for (int a = t; a < ndc; a += blockDim.x) {
            cx<double> sum = czero<double>();
            for (int ww = 0; ww < nw; ww++) sum += red[ww * ndc + a];
            Mc[(((size_t)gc * 9 + slot) * ndc + bcol) * ndc + a] = ccast<T>(sum);
        }
        __syncthreads();
    }
}

template <class T>
void coarse_assemble(const CoarseOp<T>& op, const AggMap& m, int N, const cx<T>* P, cx<T>* Mc, hipStream_t s) {
    int nt = ((m.asz * op.nd + 63) / 64) * 64;
    size_t lds = sizeof(cx<double>) * 2 * N * (nt / 64);
    dim3 grid(2 * m.c.vh, 2 * N);
    k_coarse_assemble<T><<<grid, nt, lds, s>>>(op, m, N, P, Mc);
}

// counter-based normal numbers (Philox4x32-10 + Box-Muller), element index site*nd + c
__device__ __forceinline__ void philox_c(uint32_t c[4], uint32_t k0, uint32_t k1) {
    for (int r = 0; r < 10; r++) {
        uint64_t p0 = (uint64_t)0xD2511F53u * c[0];
        uint64_t p1 = (uint64_t)0xCD9E8D57u * c[2];
        uint32_t n0 = (uint32_t)(p1 >> 32) ^ c[1] ^ k0, n2 = (uint32_t)(p0 >> 32) ^ c[3] ^ k1;
        c[1] = (uint32_t)p1; c[3] = (uint32_t)p0; c[0] = n0; c[2] = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

template <class T>
__global__ void k_coarse_random(Geom g, int nd, int n, unsigned long long seed, int sid, cx<T>* out) {
    long e = blockIdx.x * (long)blockDim.x + threadIdx.x;
    long vol = 2L * g.vh;
    if (e >= vol * nd) return;
    long s = e / nd;
    int c = (int)(e % nd);
    int x[4];
    canon_coords(g.d, s, x);
    size_t gs = lay_global(g, x);
    for (int v = 0; v < n; v++) {
        unsigned long long el = (unsigned long long)e;
        uint32_t ctr[4] = {(uint32_t)el, (uint32_t)(el >> 32), (uint32_t)v, (uint32_t)sid};
        philox_c(ctr, (uint32_t)seed, (uint32_t)(seed >> 32));
        double u1 = (ctr[0] + 0.5) * (1.0 / 4294967296.0);
        double u2 = (ctr[1] + 0.5) * (1.0 / 4294967296.0);
        double rr = sqrt(-2.0 * log(u1));
        out[(size_t)v * vol * nd + gs * nd + c] = cx<T>{T(rr * cos(2.0 * M_PI * u2)), T(rr * sin(2.0 * M_PI * u2))};
    }
}

template <class T>
void coarse_random(const Geom& g, int nd, int n, unsigned long long seed, int sid, cx<T>* out, hipStream_t s) {
    long tot = 2L * g.vh * nd;
    k_coarse_random<T><<<nblk_of(tot, 256), 256, 0, s>>>(g, nd, n, seed, sid, out);
}

// operator kernels for compute type T and storage type S
#define DD_COARSE_OP_INST(T, S)                                                                                      \
    template int coarse_gmres_coop_max_grid<T, S>();                                                                 \
    template hipError_t coarse_gmres_coop<T, S>(const CoarseOp<T, S>&, cx<T>*, long, long, cx<T>*, GmDev*, int, int, \
                                                cx<double>*, unsigned*, int*, int, hipStream_t);                      \
    template void coarse_apply<T, S>(const CoarseOp<T, S>&, int, int, const cx<T>*, int, const cx<T>*, bool, cx<T>*,   \
                                     hipStream_t, Mask, int, long, InScale);                                        \
    template bool coarse_uses_mfma<T, S>(const CoarseOp<T, S>&, int);                                                \
    template void coarse_apply_folded<T, S>(const CoarseOp<T, S>&, const cx<T>*, int, const cx<T>*, cx<T>*,           \
                                            hipStream_t, Mask, int, long, InScale);                                 \
    template void coarse_sap_half<T, S>(const CoarseOp<T, S>&, const int*, int, const cx<T>*, cx<T>*, int, hipStream_t, \
                                        int, long, Mask, SapTab);                                                   \
    template void coarse_restrict<T, S>(const AggMap&, int, int, const cx<S>*, const cx<T>*, cx<T>*, hipStream_t, int, \
                                        long, long, Mask);                                                          \
    template void coarse_prolong<T, S>(const AggMap&, int, int, const cx<S>*, const cx<T>*, cx<T>*, hipStream_t, int,  \
                                       long, long, Mask);

#define DD_COARSE_INST(T)                                                                                                \
    DD_COARSE_OP_INST(T, T)                                                                                          \
    template void coarse_self_inverse<T>(const Geom&, int, const cx<T>*, cx<T>*, int*, hipStream_t);                  \
    template void coarse_fold_inverse<T>(const Geom&, int, const cx<T>*, const cx<T>*, cx<T>*, hipStream_t);          \
    template void coarse_import_vector<T>(const Geom&, int, int, const double*, cx<T>*, hipStream_t);                \
    template void coarse_export_vector<T>(const Geom&, int, int, const cx<T>*, double*, hipStream_t);                \
    template void coarse_export_blocks<T>(const Geom&, int, int, const cx<T>*, double*, hipStream_t);                \
    template void coarse_shift_diag<T>(const Geom&, int, double, cx<T>*, hipStream_t);                                \
    template void coarse_gram_schmidt<T>(const AggMap&, int, int, const cx<T>*, cx<T>*, int*, hipStream_t);          \
    template void coarse_assemble<T>(const CoarseOp<T>&, const AggMap&, int, const cx<T>*, cx<T>*, hipStream_t);     \
    template void coarse_random<T>(const Geom&, int, int, unsigned long long, int, cx<T>*, hipStream_t);

DD_COARSE_INST(double)
DD_COARSE_INST(float)
DD_COARSE_OP_INST(float, _Float16)

}  // namespace dd
