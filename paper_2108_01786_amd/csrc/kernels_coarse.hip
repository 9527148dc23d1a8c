// Two-grid iteration for the second-kind systems.
//
// Every operator here is, after the sign of the surface rows (Ctx::gmres),
// B = d I + K with d = +-1/2 and K a smooth kernel times quadrature weights.
// A subset of the nodes, every c_k-th of boundary k with weights c_k w, is
// again a trapezoid grid, and its small system B_H e_H = r_H (r at those
// nodes) gives the correction e = (r - K_hH e_H) / d at every node: the
// Nystroem interpolation, K_hH the kernel from the coarse sources to all
// targets.  What is left, r - B e = K_hH e_H - K e, is the difference of two
// quadratures of one smooth integrand, and a smooth function itself: with a
// smooth right-hand side one correction leaves 1e-10 to 1e-15 of it, with
// any other the first leaves the smooth part of the quadrature's error and
// the second takes that to rounding.  The transposed system is the same with
// the weights on the other side (e_H / w is the smooth density).
//
// The grid rule.  A trapezoid sum of m nodes over an integrand analytic in a
// strip of half-width delta (in alpha) errs by e^{-m delta}.  delta is
// limited by the distance of another boundary (or a far part of the same
// one), about |zeta_q - zeta_p| / |zeta_q'|, and by the parameterisation: near
// a critical point alpha_0 of zeta, at about |zeta' / zeta''| = 1 / (2 |L|) with
// L = zeta'' / (2 zeta'), alpha and 2 alpha_0 - alpha have the same zeta, so the
// self kernel's nearest pole is about 1 / |L| away (on an ellipse of semi-axes
// q > b exactly 2 atanh(b / q)).
// strip_block takes the least of both over sampled nodes of every boundary; the
// host keeps m >= ln(1 / eps) / delta nodes of it (Ctx::choose_coarse).
#include <algorithm>

#include "entries.h"
#include "internal.h"

namespace wwbi {

namespace {

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

// Fine node and weight factor of every coarse node.
__global__ void k_coarse_map(Coarse C, int *map, double *fac) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= C.n) return;
    int k = 0;
    while (k + 1 < C.nb && i >= C.off[k + 1]) ++k;
    map[i] = C.first[k] + (i - C.off[k]) * C.c[k];
    fac[i] = (double)C.c[k];
}

// Entry of K for target t and source s (its weight already scaled): the full
// entry less the identity part on the diagonal.
template <int MODE>
__device__ __forceinline__ double k_entry(const Nodes &N, const Tgt &t, const Src &s, bool corr,
                                          const double *hrow) {
    const bool diag = t.idx == s.idx;
    if (MODE == kCoarseGt)
        return diag ? s.w * t.lim : gt_val64(N, t, s);
    if (MODE == kCoarseWall) return t_val64(N, t, s, hrow);
    if (diag) return s.w * t.lim - ((corr && t.k >= 2) ? s.w : 0.0);
    return a_val64(N, t, s, corr);
}

// The identity part at node p, before the sign of the surface rows.
template <int MODE>
__device__ __forceinline__ double identity_part(int k) {
    if (MODE == kCoarseWall) return -0.5;
    if (MODE == kCoarseGt) return k == 0 ? 0.5 : -0.5;
    return k == 0 ? -0.5 : 0.5;
}

// The coarse matrix, one entry per thread (rows in the unsigned form: the
// solver negates the first rows itself).
template <int MODE>
__global__ __launch_bounds__(256) void k_assemble_coarse(Nodes N, const double *hrow,
                                                         const int *map, const double *fac, int n,
                                                         int corr, double *out, long ld) {
    const int j = blockIdx.x * 64 + (threadIdx.x & 63);
    const int i = blockIdx.y * 4 + (threadIdx.x >> 6);
    if (i >= n || j >= ld) return;
    double v = 0.0;
    if (j < n) {
        const int ti = MODE == kCoarseAT ? j : i, si = MODE == kCoarseAT ? i : j;
        const Tgt t = load_tgt(N, map[ti]);
        Src s = load_src(N, map[si]);
        s.w *= fac[si];
        v = k_entry<MODE>(N, t, s, corr != 0, hrow);
        if (i == j) v += identity_part<MODE>(t.k);
    }
    out[(long)i * ld + j] = v;
}

// K_hH of A for many right-hand sides: rows of all n0 nodes, the coarse nodes'
// columns, a column per lane and kInterpRows rows per wave.
constexpr int kInterpRows = 16;

__global__ __launch_bounds__(256) void k_assemble_interp(Nodes N, const int *map,
                                                         const double *fac, int rows, int n,
                                                         int corr, double *out, long ld) {
    const int j = blockIdx.x * 64 + (threadIdx.x & 63);
    const int i0 = (blockIdx.y * 4 + (threadIdx.x >> 6)) * kInterpRows;
    if (j >= ld) return;
    Src s = load_src(N, map[j < n ? j : 0]);
    s.w *= fac[j < n ? j : 0];
    for (int i = i0; i < min(rows, i0 + kInterpRows); ++i) {
        const Tgt t = load_tgt(N, i);
        const double v = k_entry<kCoarseA>(N, t, s, corr != 0, nullptr);
        out[(long)i * ld + j] = j < n ? v : 0.0;
    }
}

// K_hH e_H: one output node per thread (rows r0 .. r0 + nr), the coarse
// nodes of chunk blockIdx.y staged in LDS; slice blockIdx.y of `part`.  For
// the transpose the outputs are sources and the coarse nodes targets.
constexpr int kCoarseStage = 32;

template <int MODE>
__global__ __launch_bounds__(256) void k_coarse_product(Nodes N, const double *hrow,
                                                        const int *map, const double *fac, int n,
                                                        int r0, int nr, int chunk, int corr,
                                                        const double *e, double *part) {
    constexpr bool T = MODE == kCoarseAT;
    __shared__ Src ss[T ? 1 : kCoarseStage];
    __shared__ Tgt ts[T ? kCoarseStage : 1];
    __shared__ double se[kCoarseStage];
    const int r = blockIdx.x * 256 + threadIdx.x;
    const bool live = r < nr;
    const int me = r0 + (live ? r : 0);
    Tgt t;
    Src s;
    if (T) s = load_src(N, me);
    else t = load_tgt(N, me);
    const int jb = blockIdx.y * chunk, je = min(n, jb + chunk);
    double acc = 0.0;
    for (int jj = jb; jj < je; jj += kCoarseStage) {
        const int j = jj + threadIdx.x;
        if ((int)threadIdx.x < kCoarseStage && j < je) {
            if (T) {
                ts[threadIdx.x] = load_tgt(N, map[j]);
                se[threadIdx.x] = e[j];
            } else {
                ss[threadIdx.x] = load_src(N, map[j]);
                se[threadIdx.x] = fac[j] * e[j];
            }
        }
        __syncthreads();
        const int m = min(kCoarseStage, je - jj);
        for (int i = 0; i < m; ++i)
            acc += k_entry<MODE>(N, T ? ts[i] : t, T ? s : ss[i], corr != 0, hrow) * se[i];
        __syncthreads();
    }
    if (live) part[(long)blockIdx.y * nr + r] = acc;
}

// x (+)= (r - S K_hH e_H) / d on every node: the slices summed in order, the
// sums of rows [0, flip) negated.
__global__ __launch_bounds__(64 * kSliceWaves) void k_coarse_finish(int nr, const double *part,
                                                                    int ns, int flip,
                                                                    double inv_d, const double *r,
                                                                    double *x, int add) {
    __shared__ double red[kSliceWaves][64];
    const int i = blockIdx.x * 64 + (threadIdx.x & 63);
    double s = sum_slices_waves<kSliceWaves>(part, ns, nr, i, i < nr, red);
    if (threadIdx.x >= 64 || i >= nr) return;
    if (i < flip) s = -s;
    const double e = (r[i] - s) * inv_d;
    x[i] = add ? x[i] + e : e;
}

// x = b / d (the correction of a right-hand side without smooth part)
__global__ void k_scale_copy(int n, const double *b, double a, double *x) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = a * b[i];
}

// Per system out[0..63]: partial sums of b^2, out[64..127]: of
// (b_{i+1} - b_i)^2, to tell a sampled smooth function (far below b^2) from noise (about 2 b^2)
__global__ __launch_bounds__(256) void k_roughness(const double *b, long bs, int n,
                                                   double *out) {
    __shared__ double sh[8];
    b += blockIdx.y * bs;
    out += blockIdx.y * 128;
    double s = 0.0, d = 0.0;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
        const double v = b[i], w = i + 1 < n ? b[i + 1] - v : 0.0;
        s += v * v;
        d += w * w;
    }
    for (int o = 32; o > 0; o >>= 1) {
        s += __shfl_xor(s, o, 64);
        d += __shfl_xor(d, o, 64);
    }
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { sh[wv] = s; sh[4 + wv] = d; }
    __syncthreads();
    if (threadIdx.x == 0) {
        out[blockIdx.x] = ((sh[0] + sh[1]) + sh[2]) + sh[3];
        out[64 + blockIdx.x] = ((sh[4] + sh[5]) + sh[6]) + sh[7];
    }
}

int product_chunk(int nr, int n) {
    // about 1500 blocks, chunks of a multiple of the stage
    const int ob = cdiv(nr, 256);
    int c = cdiv(n, std::max(1, cdiv(1500, ob)));
    return std::max(1, cdiv(c, kCoarseStage)) * kCoarseStage;
}

}  // namespace

void launch_coarse_map(const Coarse &C, int *map, double *fac, hipStream_t st) {
    hipLaunchKernelGGL(k_coarse_map, dim3(cdiv(C.n, 256)), dim3(256), 0, st, C, map, fac);
}

void launch_assemble_coarse(const Nodes &N, const double *hrow, int mode, const int *map,
                            const double *fac, int n, int corr, double *out, long ld,
                            hipStream_t st) {
    const dim3 grid(cdiv(ld, 64), cdiv(n, 4));
    switch (mode) {
    case kCoarseA: hipLaunchKernelGGL(k_assemble_coarse<kCoarseA>, grid, dim3(256), 0, st, N, hrow, map, fac, n, corr, out, ld); break;
    case kCoarseAT: hipLaunchKernelGGL(k_assemble_coarse<kCoarseAT>, grid, dim3(256), 0, st, N, hrow, map, fac, n, corr, out, ld); break;
    case kCoarseGt: hipLaunchKernelGGL(k_assemble_coarse<kCoarseGt>, grid, dim3(256), 0, st, N, hrow, map, fac, n, corr, out, ld); break;
    default: hipLaunchKernelGGL(k_assemble_coarse<kCoarseWall>, grid, dim3(256), 0, st, N, hrow, map, fac, n, corr, out, ld); break;
    }
}

void launch_assemble_interp(const Nodes &N, const int *map, const double *fac, int n, int corr,
                            double *out, long ld, hipStream_t st) {
    hipLaunchKernelGGL(k_assemble_interp, dim3(cdiv(ld, 64), cdiv(N.n, 4 * kInterpRows)),
                       dim3(256), 0, st, N, map, fac, N.n, n, corr, out, ld);
}

int coarse_slices(int nr, int n) { return cdiv(n, product_chunk(nr, n)); }

void launch_coarse_correct(const Nodes &N, const double *hrow, int mode, const int *map,
                           const double *fac, int n, int corr, const double *e, int r0, int nr,
                           int flip, double inv_d, const double *r, double *x, bool add,
                           double *part, hipStream_t st) {
    const int chunk = product_chunk(nr, n), ns = cdiv(n, chunk);
    const dim3 grid(cdiv(nr, 256), ns);
    switch (mode) {
    case kCoarseA: hipLaunchKernelGGL(k_coarse_product<kCoarseA>, grid, dim3(256), 0, st, N, hrow, map, fac, n, r0, nr, chunk, corr, e, part); break;
    case kCoarseAT: hipLaunchKernelGGL(k_coarse_product<kCoarseAT>, grid, dim3(256), 0, st, N, hrow, map, fac, n, r0, nr, chunk, corr, e, part); break;
    case kCoarseGt: hipLaunchKernelGGL(k_coarse_product<kCoarseGt>, grid, dim3(256), 0, st, N, hrow, map, fac, n, r0, nr, chunk, corr, e, part); break;
    default: hipLaunchKernelGGL(k_coarse_product<kCoarseWall>, grid, dim3(256), 0, st, N, hrow, map, fac, n, r0, nr, chunk, corr, e, part); break;
    }
    hipLaunchKernelGGL(k_coarse_finish, dim3(cdiv(nr, 64)), dim3(64 * kSliceWaves), 0, st, nr,
                       part, ns, flip, inv_d, r, x, add ? 1 : 0);
}

void launch_scale_copy(int n, const double *b, double a, double *x, hipStream_t st) {
    hipLaunchKernelGGL(k_scale_copy, dim3(cdiv(n, 256)), dim3(256), 0, st, n, b, a, x);
}

void launch_roughness(const double *b, long bs, int n, int nsys, double *out, hipStream_t st) {
    hipLaunchKernelGGL(k_roughness, dim3(64, nsys), dim3(256), 0, st, b, bs, n, out);
}

}  // namespace wwbi
