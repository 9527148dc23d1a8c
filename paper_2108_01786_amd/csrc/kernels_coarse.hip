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

// Where the pairs of a tile allow it (tile_kind: all but the tiles around the
// diagonal and where boundaries come close), the far form of an entry serves:
// the E quotient without the near, band and diagonal tests, 20 instructions a
// pair.  Products with every pair by its full entry took 29 us at 10240 x 640
// nodes, 23 at 4608 x 448, 43 at 5002 x 1792 and 208 at 40960 x 1792; now 19,
// 13, 24 and 89.  The small ones are bound by the latency of a block: its own
// node, the staged ones, the tests, 16 to 64 pairs.

// Far entries of A, a column per lane, target after target: f(i) loads row i's
// target, put(i, v) takes the value.
template <int KIND, bool LO, class Row, class Put>
__device__ __forceinline__ void far_rows(int rows, const Src &s, double fa, double fb, double ec,
                                         Row row, Put put) {
    for (int i = 0; i < rows; ++i) put(i, a_fast64<KIND, LO>(row(i), s, fa, fb, ec));
}

// Rows [0, rows) of K (targets row(i), node indices [pa, pb]) against the
// wave's columns: lane l holds coarse source j0 + l of n.
template <class Row, class Put>
__device__ __forceinline__ void interp_tile(const Nodes &N, const int *map, const double *fac,
                                            int n, int j0, int corr, int pa, int pb, int rows,
                                            Row row, Put put) {
    const int j = min(j0 + (int)(threadIdx.x & 63), n - 1);
    Src s = load_src(N, map[j]);
    s.w *= fac[j];
    const int qa = map[min(j0, n - 1)], qb = map[min(j0 + 63, n - 1)];
    const int kind = tile_kind<64>(N, pa, pb, qa, qb);
    if (kind == kTileFull) {
        for (int i = 0; i < rows; ++i)
            put(i, k_entry<kCoarseA>(N, row(i), s, corr != 0, nullptr));
        return;
    }
    const int kp = N.bid[pa], kq = N.bid[qa];
    const double fa = 0.5 * s.w * s.dx, fb = 0.5 * s.w * s.dy;
    const double ec = (corr && kp == kq && kp >= 2) ? s.w : 0.0;
    const bool lo = kind == kTileLo;
    if ((kp == 0) == (kq == 0)) {
        if (lo) far_rows<kFastIm, true>(rows, s, fa, fb, ec, row, put);
        else far_rows<kFastIm, false>(rows, s, fa, fb, ec, row, put);
    } else if (kp == 0) {
        if (lo) far_rows<kFastReNeg, true>(rows, s, fa, fb, 0.0, row, put);
        else far_rows<kFastReNeg, false>(rows, s, fa, fb, 0.0, row, put);
    } else {
        if (lo) far_rows<kFastRePos, true>(rows, s, fa, fb, 0.0, row, put);
        else far_rows<kFastRePos, false>(rows, s, fa, fb, 0.0, row, put);
    }
}

// The coarse matrix, kCoarseRows rows of 64 columns a wave (rows in the
// unsigned form: the solver negates the first rows itself).
constexpr int kCoarseRows = 4;

template <int MODE>
__global__ __launch_bounds__(256) void k_assemble_coarse(Nodes N, const double *hrow,
                                                         const int *map, const double *fac, int n,
                                                         int corr, double *out, long ld) {
    const int j0 = blockIdx.x * 64, j = j0 + (threadIdx.x & 63);
    const int i0 = (blockIdx.y * 4 + (threadIdx.x >> 6)) * kCoarseRows;
    const int rows = min(kCoarseRows, n - i0);
    if (rows <= 0) return;
    auto put = [&](int i, double v) {
        if (i0 + i == j) v += identity_part<MODE>(N.bid[map[j]]);
        if (j < ld) out[(long)(i0 + i) * ld + j] = j < n ? v : 0.0;
    };
    if (MODE == kCoarseA) {
        interp_tile(N, map, fac, n, j0, corr, map[i0], map[i0 + rows - 1], rows,
                    [&](int i) { return load_tgt(N, map[i0 + i]); }, put);
        return;
    }
    const int jc = min(j, n - 1);
    for (int i = 0; i < rows; ++i) {
        const int ti = MODE == kCoarseAT ? jc : i0 + i, si = MODE == kCoarseAT ? i0 + i : jc;
        const Tgt t = load_tgt(N, map[ti]);
        Src s = load_src(N, map[si]);
        s.w *= fac[si];
        put(i, k_entry<MODE>(N, t, s, corr != 0, hrow));
    }
}

// K_hH of A for many right-hand sides: rows of all n0 nodes, the coarse nodes'
// columns, a column per lane and kInterpRows rows per wave.
constexpr int kInterpRows = 16;

__global__ __launch_bounds__(256) void k_assemble_interp(Nodes N, const int *map,
                                                         const double *fac, int nodes, int n,
                                                         int corr, double *out, long ld) {
    const int j0 = blockIdx.x * 64, j = j0 + (threadIdx.x & 63);
    const int i0 = (blockIdx.y * 4 + (threadIdx.x >> 6)) * kInterpRows;
    const int rows = min(kInterpRows, nodes - i0);
    if (rows <= 0) return;
    interp_tile(N, map, fac, n, j0, corr, i0, i0 + rows - 1, rows,
                [&](int i) { return load_tgt(N, i0 + i); },
                [&](int i, double v) {
                    if (j < ld) out[(long)(i0 + i) * ld + j] = j < n ? v : 0.0;
                });
}

// K_hH e_H: one output node per thread (rows r0 .. r0 + nr), the coarse
// nodes of chunk blockIdx.y staged in LDS; slice blockIdx.y of `part`.  For
// the transpose the outputs are sources and the coarse nodes targets.  The
// same-boundary pairs within kNearBand steps, whose entry is a transcendental
// formula, are the last `bands` slices: a lane visits its own few there, where in the
// other slices a wave would take that formula for every coarse node that any
// of its 64 lanes has near.
constexpr int kCoarseStage = 64;
constexpr int kCoarseTile = 16;          // coarse nodes per tile_kind test
constexpr int kTileLanes = 64 / (kCoarseStage / kCoarseTile);

// A staged coarse node for the far form: E and, for A, its source data times
// e (a = w dx e / 2, b = w dy e / 2), else a = its weight times e.
struct FarNode {
    double ex, ey, exl, eyl, a, b;
};

// Sums over m staged nodes for one output node (E = ox, oy, oxl, oyl): for A
// of the entries themselves into p; else of e pr / |D|^2 into p and e pi /
// |D|^2 into q, D = E_source - E_target.
template <int MODE, int KIND, bool LO>
__device__ __forceinline__ void far_sums(const FarNode *f, int m, double ox, double oy,
                                         double oxl, double oyl, double &p, double &q) {
    for (int i = 0; i < m; ++i) {
        const FarNode &c = f[i];
        double dr = c.ex - ox, di = c.ey - oy;
        if (LO) {
            dr += c.exl - oxl;
            di += c.eyl - oyl;
        }
        if (MODE == kCoarseAT) {
            dr = -dr;
            di = -di;
        }
        const double nr = c.ex + ox, ni = c.ey + oy;
        const double inv = recip64_from32(dr * dr + di * di);
        const double pr = nr * dr + ni * di, pi = ni * dr - nr * di;
        if (MODE != kCoarseA) {
            const double g = c.a * inv;
            p += g * pr;
            q += g * pi;
        } else if (KIND == kFastIm) {
            p += (c.a * pr - c.b * pi) * inv;
        } else if (KIND == kFastReNeg) {
            p -= (c.a * pi + c.b * pr) * inv;
        } else {
            p += (c.a * pi + c.b * pr) * inv;
        }
    }
}

template <int MODE>
__global__ __launch_bounds__(256) void k_coarse_product(Nodes N, Coarse C, const double *hrow,
                                                        const int *map, const double *fac, int r0,
                                                        int nr, int chunk, int bands, int corr,
                                                        const double *e, double *part) {
    constexpr bool T = MODE == kCoarseAT;
    __shared__ Src ss[T ? 1 : kCoarseStage];
    __shared__ Tgt ts[T ? kCoarseStage : 1];
    __shared__ double se[kCoarseStage];
    __shared__ FarNode sf[kCoarseStage];
    const int n = C.n, lane = threadIdx.x & 63;
    const int r = blockIdx.x * 256 + threadIdx.x;
    const bool live = r < nr;
    const int me = r0 + (live ? r : nr - 1);
    Tgt t;
    Src s;
    if (T) s = load_src(N, me);
    else t = load_tgt(N, me);
    const int loc = T ? s.loc : t.loc, M = T ? s.M : t.M, kme = T ? s.k : t.k;
    double acc = 0.0;
    const int band = (int)blockIdx.y - ((int)gridDim.y - bands);
    if (band >= 0) {
        // the band: coarse nodes [lo, hi] of this boundary, cyclically
        const int k = kme - N.bid[C.first[0]], c = C.c[k], mc = M / c;
        int lo = (loc - kNearBand + 64 * c) / c - 64;
        if (lo * c < loc - kNearBand) ++lo;
        int hi = (loc + kNearBand) / c;
        if (hi - lo + 1 >= mc) {
            lo = 0;
            hi = mc - 1;
        }
        for (int l = lo + band; l <= hi; l += bands) {
            const int jl = l < 0 ? l + mc : l >= mc ? l - mc : l, j = C.off[k] + jl;
            const int node = C.first[k] + jl * c;
            if (T) {
                t = load_tgt(N, node);
                if (in_band(t, s, kNearBand)) acc += k_entry<MODE>(N, t, s, corr != 0, hrow) * e[j];
            } else {
                s = load_src(N, node);
                if (in_band(t, s, kNearBand))
                    acc += k_entry<MODE>(N, t, s, corr != 0, hrow) * ((double)c * e[j]);
            }
        }
        if (live) part[(long)blockIdx.y * nr + r] = acc;
        return;
    }
    // the wave's output nodes
    const int oa = r0 + min(blockIdx.x * 256 + wave_base(), nr - 1);
    const int ob = min(oa + 63, r0 + nr - 1), ko = N.bid[oa];
    const double ox = T ? s.ex : t.ex, oy = T ? s.ey : t.ey;
    const double oxl = T ? s.exl : t.exl, oyl = T ? s.eyl : t.eyl;
    const int jb = blockIdx.y * chunk, je = min(n, jb + chunk);
    for (int jj = jb; jj < je; jj += kCoarseStage) {
        const int j = jj + threadIdx.x, js = min(je, jj + kCoarseStage);
        if (j < js) {
            if (T) {
                const Tgt c = load_tgt(N, map[j]);
                ts[threadIdx.x] = c;
                se[threadIdx.x] = e[j];
                sf[threadIdx.x] = FarNode{c.ex, c.ey, c.exl, c.eyl, e[j], 0.0};
            } else {
                const Src c = load_src(N, map[j]);
                const double we = fac[j] * e[j];
                ss[threadIdx.x] = c;
                se[threadIdx.x] = we;
                const double h = MODE == kCoarseA ? 0.5 * c.w * we : c.w * we;
                sf[threadIdx.x] = FarNode{c.ex, c.ey, c.exl, c.eyl,
                                          MODE == kCoarseA ? h * c.dx : h, h * c.dy};
            }
        }
        // lanes kTileLanes i ..: how to take tile i, and its boundary
        const int ta = min(jj + lane / kTileLanes * kCoarseTile, js - 1);
        const int ca = map[ta], cb = map[min(ta + kCoarseTile, js) - 1], kcs = N.bid[ca];
        const int kinds = T ? tile_kind<kTileLanes>(N, ca, cb, oa, ob)
                            : tile_kind<kTileLanes>(N, oa, ob, ca, cb);
        __syncthreads();
        for (int i0 = 0; i0 < js - jj; i0 += kCoarseTile) {
            const int m = min(kCoarseTile, js - jj - i0);
            const int kind = __builtin_amdgcn_readlane(kinds, i0 / kCoarseTile * kTileLanes);
            if (kind == kTileFull) {
                for (int i = i0; i < i0 + m; ++i) {
                    const Tgt &ti = T ? ts[i] : t;
                    const Src &si = T ? s : ss[i];
                    if (!in_band(ti, si, kNearBand))
                        acc += k_entry<MODE>(N, ti, si, corr != 0, hrow) * se[i];
                }
                continue;
            }
            const FarNode *f = sf + i0;
            const bool lo = kind == kTileLo;
            const int kc = __builtin_amdgcn_readlane(kcs, i0 / kCoarseTile * kTileLanes);
            const int kt = T ? kc : ko, ks = T ? ko : kc;
            const bool im = (kt == 0) == (ks == 0);
            double p = 0.0, q = 0.0;
            if (MODE != kCoarseA || im) {
                if (lo) far_sums<MODE, kFastIm, true>(f, m, ox, oy, oxl, oyl, p, q);
                else far_sums<MODE, kFastIm, false>(f, m, ox, oy, oxl, oyl, p, q);
            } else if (kt == 0) {
                if (lo) far_sums<MODE, kFastReNeg, true>(f, m, ox, oy, oxl, oyl, p, q);
                else far_sums<MODE, kFastReNeg, false>(f, m, ox, oy, oxl, oyl, p, q);
            } else {
                if (lo) far_sums<MODE, kFastRePos, true>(f, m, ox, oy, oxl, oyl, p, q);
                else far_sums<MODE, kFastRePos, false>(f, m, ox, oy, oxl, oyl, p, q);
            }
            if (MODE == kCoarseA) {
                acc += p;
            } else if (T) {
                const double fa = 0.5 * s.w * s.dx, fb = 0.5 * s.w * s.dy;
                acc += im ? fa * p - fb * q : kt == 0 ? -(fa * q + fb * p) : fa * q + fb * p;
            } else {
                // R's real part on pairs of the surface and a wall, its
                // imaginary part on the others
                const double re = 0.5 * (t.dx * q + t.dy * p);
                acc += im ? -0.5 * (t.dx * p - t.dy * q) : kt == 0 ? -re : re;
            }
            if (MODE <= kCoarseAT && corr && kt == ks && kt >= 2) {
                double es = 0.0;
                for (int i = i0; i < i0 + m; ++i) es += T ? s.w * se[i] : ss[i].w * se[i];
                acc -= es;
            }
        }
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

__global__ __launch_bounds__(256) void k_norms(const double *r, const double *b, int n,
                                               double *out) {
    __shared__ double sh[4];
    const double *v = blockIdx.y ? b : r;
    double s = 0.0;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) s += v[i] * v[i];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) out[blockIdx.y * 64 + blockIdx.x] = ((sh[0] + sh[1]) + sh[2]) + sh[3];
}

// Coarse nodes per slice: about 2048 blocks, a multiple of the tile (at most
// kSmallCoarseMax / kCoarseTile = 128 slices, and up to 9 for the band).
int product_chunk(int nr, int n) {
    const int c = cdiv(n, std::max(1, cdiv(2048, cdiv(nr, 256))));
    return std::max(1, cdiv(c, kCoarseTile)) * kCoarseTile;
}

}  // namespace

void launch_coarse_map(const Coarse &C, int *map, double *fac, hipStream_t st) {
    hipLaunchKernelGGL(k_coarse_map, dim3(cdiv(C.n, 256)), dim3(256), 0, st, C, map, fac);
}

void launch_assemble_coarse(const Nodes &N, const double *hrow, int mode, const int *map,
                            const double *fac, int n, int corr, double *out, long ld,
                            hipStream_t st) {
    const dim3 grid(cdiv(ld, 64), cdiv(n, 4 * kCoarseRows));
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

void launch_coarse_correct(const Nodes &N, const Coarse &C, const double *hrow, int mode,
                           const int *map, const double *fac, int corr, const double *e, int r0,
                           int nr, int flip, double inv_d, const double *r, double *x, bool add,
                           double *part, hipStream_t st) {
    // at most four of the band's nodes per lane and slice
    int least = C.c[0];
    for (int k = 1; k < C.nb; ++k) least = std::min(least, C.c[k]);
    const int bands = cdiv(2 * kNearBand / least + 1, 4);
    const int chunk = product_chunk(nr, C.n), ns = cdiv(C.n, chunk) + bands;
    const dim3 grid(cdiv(nr, 256), ns);
    switch (mode) {
    case kCoarseA: hipLaunchKernelGGL(k_coarse_product<kCoarseA>, grid, dim3(256), 0, st, N, C, hrow, map, fac, r0, nr, chunk, bands, corr, e, part); break;
    case kCoarseAT: hipLaunchKernelGGL(k_coarse_product<kCoarseAT>, grid, dim3(256), 0, st, N, C, hrow, map, fac, r0, nr, chunk, bands, corr, e, part); break;
    case kCoarseGt: hipLaunchKernelGGL(k_coarse_product<kCoarseGt>, grid, dim3(256), 0, st, N, C, hrow, map, fac, r0, nr, chunk, bands, corr, e, part); break;
    default: hipLaunchKernelGGL(k_coarse_product<kCoarseWall>, grid, dim3(256), 0, st, N, C, hrow, map, fac, r0, nr, chunk, bands, corr, e, part); break;
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

void launch_norms(const double *r, const double *b, int n, double *out, hipStream_t st) {
    hipLaunchKernelGGL(k_norms, dim3(64, b ? 2 : 1), dim3(256), 0, st, r, b, n, out);
}

}  // namespace wwbi
