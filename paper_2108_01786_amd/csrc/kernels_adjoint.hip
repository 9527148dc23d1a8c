// Derivative contractions of the adjoint of the velocity-potential solve.
//
// Forward map (walls fixed, surface samples z, d = z', e = z'' free):
//   A(z, d, e) omega = b,  b_0 = phi~            (Sec. 3.2-3.3)
//   gamma = (-D omega_0, D omega_1, ...)
//   s U = u_mv(z, d) + H gamma_0 / 2 + T(z, d, e) gamma     (Sec. 3.4)
// With c = Ubar / s and lambda = A^{-T} omegabar, the geometric part of the
// gradient is
//   sum_m c_m [d u_mv + dT gamma]_m - sum_m c_m U_m ds_m - lambda^T dA omega.
// Every kernel entry that involves a surface node contributes through
//   d kappa / d Delta = -(1 + kappa^2)/2,  kappa = cot((z_q - z_p)/2),
// so dS/dz_q = -d_q (1 + kappa^2)/4 = -dS/dz_p, dS/dd_q = kappa/2 for the
// source flavour and dR/dz_q = d_p (1 + kappa^2)/4 = -dR/dz_p, dR/dd_p =
// -kappa/2 for the target flavour.
#include "entries.h"
#include "internal.h"

namespace wwbi {

namespace {

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }
constexpr int kTlmMax = 32;      // directions of one tangent-linear launch
constexpr int kTlmWaves = 4608;  // waves the column pass's source split aims at

struct Cx {
    double re, im;
};
__device__ __forceinline__ Cx cmul(Cx a, Cx b) {
    return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
__device__ __forceinline__ Cx ctimes_i(Cx a) { return {-a.im, a.re}; }
__device__ __forceinline__ Cx cscale(Cx a, double s) { return {a.re * s, a.im * s}; }

// Row pass: targets r on the surface, all sources q != r.
//   out[0] = sum_q omega_q dA_rq/dx_r        out[1] = ... /dy_r
//   out[2] = sum_q gamma_q dT_rq/dx_r        out[3] = ... /dy_r
//   out[4] = sum_q gamma_q dT_rq/ddx_r       out[5] = ... /ddy_r
__device__ __forceinline__ void row_terms(const Tgt &t, const Src &s, double cr, double ci,
                                          double wq, double gq, double (&a)[6]) {
    const Cx kap{cr, ci};
    const Cx Q{1.0 + cr * cr - ci * ci, 2.0 * cr * ci};
    // source flavour, target derivative: dS/dz_r = +d_q Q / 4
    const Cx dS = cscale(cmul({s.dx, s.dy}, Q), 0.25 * s.w * wq);
    const Cx dSy = ctimes_i(dS);
    if (s.k == 0) { a[0] += dS.im; a[1] += dSy.im; }   // Im block (surface row, surface col)
    else { a[0] += dS.re; a[1] += dSy.re; }            // Re block (surface row, wall col)
    // target flavour: dR/dz_r = -d_r Q / 4, dR/dd_r = -kappa / 2
    const double gw = s.w * gq;
    const Cx dR = cscale(cmul({t.dx, t.dy}, Q), -0.25 * gw);
    const Cx dRy = ctimes_i(dR);
    const Cx dD = cscale(kap, -0.5 * gw);
    const Cx dDy = ctimes_i(dD);
    if (s.k == 0) { a[2] += dR.re; a[3] += dRy.re; a[4] += dD.re; a[5] += dDy.re; }
    else { a[2] += dR.im; a[3] += dRy.im; a[4] += dD.im; a[5] += dDy.im; }
}

// Column pass: sources r on the surface, all targets p != r.
//   out[0..3] = sum_p lambda_p dA_pr/d(x_r, y_r, dx_r, dy_r)
//   out[4..5] = sum_{p on surface} c_p dT_pr/d(x_r, y_r)
__device__ __forceinline__ void col_terms(const Tgt &t, const Src &s, double cr, double ci,
                                          double lp, double cp, double (&a)[6]) {
    const Cx kap{cr, ci};
    const Cx Q{1.0 + cr * cr - ci * ci, 2.0 * cr * ci};
    // source flavour, source derivative: dS/dz_r = -d_r Q / 4, dS/dd_r = kappa / 2
    const double lw = s.w * lp;
    const Cx dS = cscale(cmul({s.dx, s.dy}, Q), -0.25 * lw);
    const Cx dSy = ctimes_i(dS);
    const Cx dK = cscale(kap, 0.5 * lw);
    const Cx dKy = ctimes_i(dK);
    if (t.k == 0) {   // surface row: Im S
        a[0] += dS.im; a[1] += dSy.im; a[2] += dK.im; a[3] += dKy.im;
        // target flavour, source derivative: dR/dz_r = d_p Q / 4 (surface source: Re)
        const Cx dR = cscale(cmul({t.dx, t.dy}, Q), 0.25 * s.w * cp);
        a[4] += dR.re;
        a[5] += ctimes_i(dR).re;
    } else {          // wall row: -Re S
        a[0] -= dS.re; a[1] -= dSy.re; a[2] -= dK.re; a[3] -= dKy.re;
    }
}

__device__ __forceinline__ void store6(double *part, long st, long off, const double (&a)[6]) {
#pragma unroll
    for (int k = 0; k < 6; ++k) part[k * st + off] = a[k];
}

// Far part of both passes: every pair except the surface pairs within nb
// grid steps of r (diagonal included), with kappa from E alone.  A block takes
// 64 nodes r, a lane each, and a chunk of the other index, staged in LDS and
// shared by its waves: slice blockIdx.y of `part` (component stride st).  What
// a pair contributes is linear in a few sums over 1 + kappa^2 and kappa, so
// the loops form those (35 operations a pair instead of 75) and the factors of
// node r follow once.  With a node per thread of 256, a wave went through 256
// pairs on its own and the launch had half a wave per SIMD: 95 us for the rows
// and 86 for the columns at 2048 x 4608 nodes; now 19 and 18.
constexpr int kAdjWaves = 4;
constexpr int kAdjStage = 64 * kAdjWaves;

// A staged node: E, complex weight a (of 1 + kappa^2) and real weight g.
struct AdjNode {
    double ex, ey, exl, eyl, ar, ai, g;
    int loc;
};

// Sums over nodes [i0, i1): A = sum a (1 + kappa^2), Q = sum g (1 + kappa^2),
// K = sum g kappa; kappa of (source, target) = (node, own) or, with OWN_SRC,
// (own, node).  CHECK: nodes within nb steps of the own are left out.
struct AdjSums {
    Cx A, Q, K;
};
template <bool OWN_SRC, bool CHECK>
__device__ __forceinline__ void adj_sums(const AdjNode *f, int i0, int i1, double ox, double oy,
                                         double oxl, double oyl, int loc, int M, int nb,
                                         AdjSums &o) {
    for (int i = i0; i < i1; ++i) {
        const AdjNode &c = f[i];
        double dr = (c.ex - ox) + (c.exl - oxl), di = (c.ey - oy) + (c.eyl - oyl);
        if (OWN_SRC) {
            dr = -dr;
            di = -di;
        }
        const double nr = c.ex + ox, ni = c.ey + oy;
        const double inv = recip64(dr * dr + di * di);
        double cr = -(ni * dr - nr * di) * inv, ci = (nr * dr + ni * di) * inv;
        double ar = c.ar, ai = c.ai, g = c.g;
        if (CHECK && cyc_dist(c.loc, loc, M) <= nb) cr = ci = ar = ai = g = 0.0;
        const double qr = 1.0 + cr * cr - ci * ci, qi = 2.0 * cr * ci;
        o.A.re += ar * qr - ai * qi;
        o.A.im += ar * qi + ai * qr;
        o.Q.re += g * qr;
        o.Q.im += g * qi;
        o.K.re += g * cr;
        o.K.im += g * ci;
    }
}

// The chunk's sums over the surface's nodes (S) and the walls' (W) for the
// wave's share of every stage.
template <bool OWN_SRC, class Load>
__device__ __forceinline__ void adj_chunk(const Nodes &N, AdjNode *f, int r0, int n0, int b0,
                                          int e0, int nb, double ox, double oy, double oxl,
                                          double oyl, Load load, AdjSums &S, AdjSums &W) {
    const int wv = threadIdx.x >> 6, r = r0 + (threadIdx.x & 63);
    for (int b = b0; b < e0; b += kAdjStage) {
        const int m = min(kAdjStage, e0 - b);
        if (b > b0) __syncthreads();
        if ((int)threadIdx.x < m) f[threadIdx.x] = load(b + threadIdx.x);
        __syncthreads();
        const int share = (m + kAdjWaves - 1) / kAdjWaves;
        const int i0 = min(m, share * wv), i1 = min(m, i0 + share);
        const int ms = min(max(n0 - b, i0), i1);       // surface nodes come first
        if (ms > i0) {
            const int ra = r0, rb = min(r0 + 63, n0 - 1);
            if (ranges_apart(N, ra, rb, b + i0, b + ms - 1, nb))
                adj_sums<OWN_SRC, false>(f, i0, ms, ox, oy, oxl, oyl, r, n0, nb, S);
            else
                adj_sums<OWN_SRC, true>(f, i0, ms, ox, oy, oxl, oyl, r, n0, nb, S);
        }
        adj_sums<OWN_SRC, false>(f, ms, i1, ox, oy, oxl, oyl, r, n0, nb, W);
    }
}

// The waves' six values of a node added in wave order into the slice.
__device__ __forceinline__ void adj_store(double (*red)[6][64], const double (&a)[6], int r0,
                                          int n0, double *part, long st, long slice) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < 6; ++k) red[wv][k][lane] = a[k];
    __syncthreads();
    for (int k = wv; k < 6; k += kAdjWaves) {
        double v = red[0][k][lane];
        for (int w = 1; w < kAdjWaves; ++w) v += red[w][k][lane];
        if (r0 + lane < n0) part[k * st + slice * n0 + r0 + lane] = v;
    }
}

__global__ __launch_bounds__(kAdjStage) void k_adj_rows(Nodes N, int n0, int n, int chunk, int nb,
                                                        const double *__restrict__ omega,
                                                        const double *__restrict__ gamma,
                                                        double *__restrict__ part, long st) {
    __shared__ AdjNode f[kAdjStage];
    __shared__ double red[kAdjWaves][6][64];
    const int r0 = blockIdx.x * 64, r = min(r0 + (int)(threadIdx.x & 63), n0 - 1);
    const int qb = blockIdx.y * chunk, qe = min(n, qb + chunk);
    AdjSums S{}, W{};
    // dS/dz_r = d_q Q / 4 with the weight w omega, the R terms with w gamma
    adj_chunk<false>(N, f, r0, n0, qb, qe, nb, N.ex[r], N.ey[r], N.exl[r], N.eyl[r],
                     [&](int q) {
                         const double w = N.w[q], a = 0.25 * w * omega[q];
                         return AdjNode{N.ex[q], N.ey[q], N.exl[q], N.eyl[q],
                                        a * N.dx[q], a * N.dy[q], w * gamma[q], N.loc[q]};
                     },
                     S, W);
    const Cx d{N.dx[r], N.dy[r]};
    // dR/dz_r = -d_r Q / 4, dR/dd_r = -kappa / 2; a surface source takes Im S
    // and Re R, a wall source Re S and Im R
    const Cx R0 = cscale(cmul(d, S.Q), -0.25), R1 = cscale(cmul(d, W.Q), -0.25);
    const double a[6] = {S.A.im + W.A.re,        S.A.re - W.A.im,
                         R0.re + R1.im,          -R0.im + R1.re,
                         -0.5 * (S.K.re + W.K.im), 0.5 * (S.K.im - W.K.re)};
    adj_store(red, a, r0, n0, part, st, blockIdx.y);
}

__global__ __launch_bounds__(kAdjStage) void k_adj_cols(Nodes N, int n0, int n, int chunk, int nb,
                                                        const double *__restrict__ lam,
                                                        const double *__restrict__ cvec,
                                                        double *__restrict__ part, long st) {
    __shared__ AdjNode f[kAdjStage];
    __shared__ double red[kAdjWaves][6][64];
    const int r0 = blockIdx.x * 64, r = min(r0 + (int)(threadIdx.x & 63), n0 - 1);
    const int pb = blockIdx.y * chunk, pe = min(n, pb + chunk);
    AdjSums S{}, W{};
    // the S terms with the weight lambda, dR/dz_r = d_p Q / 4 with c (surface
    // targets only)
    adj_chunk<true>(N, f, r0, n0, pb, pe, nb, N.ex[r], N.ey[r], N.exl[r], N.eyl[r],
                    [&](int p) {
                        const double c = p < n0 ? 0.25 * cvec[p] : 0.0;
                        return AdjNode{N.ex[p], N.ey[p], N.exl[p], N.eyl[p],
                                       c * N.dx[p], c * N.dy[p], lam[p], N.loc[p]};
                    },
                    S, W);
    const double w = N.w[r];
    const Cx d{N.dx[r], N.dy[r]};
    // dS/dz_r = -d_r Q / 4, dS/dd_r = kappa / 2; a surface row takes Im S, a
    // wall row -Re S
    const Cx S0 = cscale(cmul(d, S.Q), -0.25 * w), S1 = cscale(cmul(d, W.Q), -0.25 * w);
    const double a[6] = {S0.im - S1.re,
                         S0.re + S1.im,
                         0.5 * w * (S.K.im - W.K.re),
                         0.5 * w * (S.K.re + W.K.im),
                         w * S.A.re,
                         -w * S.A.im};
    adj_store(red, a, r0, n0, part, st, blockIdx.y);
}

// Near part of both passes: the surface partners of r within nb grid steps
// (the whole surface when it has at most 2 nb + 1 nodes), diagonal excluded,
// with the exact-difference kappa; written as slice `slice`.
// kAdjNearLanes lanes share a node and add their sums in a fixed butterfly order.
constexpr int kAdjNearLanes = 8;

template <bool COLS>
__global__ __launch_bounds__(256) void k_adj_near(Nodes N, int n0, int nb,
                                                  const double *__restrict__ v1,
                                                  const double *__restrict__ v2,
                                                  double *__restrict__ part, long st, int slice) {
    const int g = threadIdx.x % kAdjNearLanes;
    const int r = blockIdx.x * (256 / kAdjNearLanes) + threadIdx.x / kAdjNearLanes;
    const int rr = min(r, n0 - 1);
    const bool whole = 2 * nb + 1 >= n0;
    const int d0 = whole ? -rr : -nb, d1 = whole ? n0 - 1 - rr : nb;
    double a[6] = {0, 0, 0, 0, 0, 0};
    const Tgt tr = load_tgt(N, rr);
    const Src sr = load_src(N, rr);
    for (int d = d0 + g; d <= d1; d += kAdjNearLanes) {
        if (d == 0) continue;
        int l = rr + d;
        if (l < 0) l += n0;
        if (l >= n0) l -= n0;
        double cr, ci;
        if (!COLS) {
            const Src s = load_src(N, l);
            kappa64(N, tr, s, cr, ci);
            row_terms(tr, s, cr, ci, v1[l], v2[l], a);
        } else {
            const Tgt t = load_tgt(N, l);
            kappa64(N, t, sr, cr, ci);
            col_terms(t, sr, cr, ci, v1[l], v2[l], a);
        }
    }
#pragma unroll
    for (int k = 0; k < 6; ++k)
#pragma unroll
        for (int o = kAdjNearLanes / 2; o > 0; o >>= 1) a[k] += __shfl_xor(a[k], o, 64);
    if (g == 0 && r < n0) store6(part, st, (long)slice * n0 + r, a);
}

// The ns slices of component blockIdx.y summed into its first.
__global__ __launch_bounds__(64 * kSliceWaves) void k_adj_sum(int n0, int ns, double *part,
                                                              long st) {
    __shared__ double red[kSliceWaves][64];
    const int r = blockIdx.x * 64 + (threadIdx.x & 63);
    double *p = part + blockIdx.y * st;
    const double v = sum_slices_waves<kSliceWaves>(p, ns, n0, r, r < n0, red);
    if (threadIdx.x < 64 && r < n0) p[r] = v;
}

// Derivatives of u_mv = -(V1 + sum a / 2) y' + sum_j a_j Re{cot((z - z_j)/2) z' / 2}
// with respect to x, y, x', y' of one surface node.
__device__ __forceinline__ void umv_derivs(const Flow &F, double x, double y, double dx, double dy,
                                           double &ux, double &uy, double &udx, double &udy) {
    double asum = 0.0;
    for (int j = 0; j < F.nobs; ++j) asum += F.a[j];
    ux = 0.0;
    uy = 0.0;
    udx = 0.0;
    udy = -(F.V1 + 0.5 * asum);
    for (int j = 0; j < F.nobs; ++j) {
        double cr, ci;
        cot_half64(x - F.zx[j], y - F.zy[j], cr, ci);
        const Cx kap{cr, ci};
        const Cx Q{1.0 + cr * cr - ci * ci, 2.0 * cr * ci};
        const Cx dz = cscale(cmul({dx, dy}, Q), -0.25 * F.a[j]);   // d/dz of a kappa z'/2
        ux += dz.re;
        uy += ctimes_i(dz).re;
        udx += 0.5 * F.a[j] * kap.re;
        udy += 0.5 * F.a[j] * ctimes_i(kap).re;
    }
}

// The diagonal limit L = e / (2 d) (d = z', e = z'') of a surface node and its
// complex derivatives dL/dd = -L / d and dL/de = 1 / (2 d); A_rr = -1/2 + w Im L
// and T_rr = w Re L.
__device__ __forceinline__ void diag_limit_derivs(double dx, double dy, double ex, double ey,
                                                  Cx &dLdd, Cx &dLde) {
    const double d2 = dx * dx + dy * dy;
    const Cx inv_d{dx / d2, -dy / d2};                 // 1/d
    const Cx L{(ex * dx + ey * dy) / (2.0 * d2), (ey * dx - ex * dy) / (2.0 * d2)};
    dLdd = cscale(cmul(L, inv_d), -1.0);
    dLde = cscale(inv_d, 0.5);
}

// Combine every term on the surface nodes.
__global__ void k_adj_finalize(Nodes N, Flow F, int n0, const double *__restrict__ Ubar,
                               const double *__restrict__ U, const double *__restrict__ omega,
                               const double *__restrict__ gamma, const double *__restrict__ lam,
                               const double *__restrict__ prow,
                               const double *__restrict__ pcol, long st, double *g_phi,
                               double *g_x, double *g_y, double *g_dx, double *g_dy, double *g_ddx,
                               double *g_ddy) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n0) return;
    double R[6], Cc[6];
    for (int k = 0; k < 6; ++k) {
        R[k] = prow[k * st + r];
        Cc[k] = pcol[k * st + r];
    }
    const double x = N.x[r], y = N.y[r], dx = N.dx[r], dy = N.dy[r];
    const double ex = N.ddx[r], ey = N.ddy[r];
    const double s = N.s[r], w = N.w[r];
    const double c = Ubar[r] / s;
    const double lr = lam[r], wr = omega[r], gr = gamma[r];
    double ux, uy, udx, udy;
    umv_derivs(F, x, y, dx, dy, ux, uy, udx, udy);
    // diagonal limits L = e/(2d): A_rr = -1/2 + w Im L, T_rr = w Re L
    Cx dLdd, dLde;
    diag_limit_derivs(dx, dy, ex, ey, dLdd, dLde);
    const Cx dLdd_y = ctimes_i(dLdd);
    const Cx dLde_y = ctimes_i(dLde);
    const double la = -lr * wr * w, tc = c * gr * w;   // weights of Im (A) and Re (T) parts
    g_phi[r] = lr;
    g_x[r] = c * ux + c * R[2] + gr * Cc[4] - lr * R[0] - wr * Cc[0];
    g_y[r] = c * uy + c * R[3] + gr * Cc[5] - lr * R[1] - wr * Cc[1];
    g_dx[r] = c * udx - c * U[r] * dx / s + c * R[4] - wr * Cc[2] + la * dLdd.im + tc * dLdd.re;
    g_dy[r] = c * udy - c * U[r] * dy / s + c * R[5] - wr * Cc[3] + la * dLdd_y.im + tc * dLdd_y.re;
    g_ddx[r] = la * dLde.im + tc * dLde.re;
    g_ddy[r] = la * dLde_y.im + tc * dLde_y.re;
}

// ---------------------------------------------------------------------------
// Tangent-linear model (forward mode) of the same chain, for up to kTlmMax
// directions at once.  A direction moves the surface's node data (x, y, x',
// y', x'', y'') and phi~; dirs holds 7 x nd x M_0 values, component c of
// direction i at (c * nd + i) * M_0.  With d omega = A^{-1} (d phi~ e_0 -
// dA omega) and dU = (d u_mv + dT gamma + T d gamma + H d gamma_0 / 2 - U ds) / s,
// the terms of dA omega and dT gamma that move with the target node are the
// adjoint's row sums (k_adj_rows) times the direction at that node; the terms
// that move with the source node come from k_tlm_cols (matrix cores).
// ---------------------------------------------------------------------------

// Weights of the column part: W[(q * 6 + c) * kTlmMax + i] is direction i's
// change of source q's x, y, x', y' times omega_q (c = 0..3) and of its x, y
// times gamma_q (c = 4, 5); zero for i >= nd.
__global__ void k_tlm_weights(int n0, int nd, const double *__restrict__ dirs,
                              const double *__restrict__ omega, const double *__restrict__ gamma,
                              double *__restrict__ W) {
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (long)n0 * 6 * kTlmMax) return;
    const int i = (int)(e % kTlmMax), c = (int)((e / kTlmMax) % 6), q = (int)(e / (6 * kTlmMax));
    double v = 0.0;
    if (i < nd) {
        const int cc = c < 4 ? c : c - 4;
        v = dirs[((long)cc * nd + i) * n0 + q] * (c < 4 ? omega[q] : gamma[q]);
    }
    W[e] = v;
}

// Column part on the matrix cores: for targets p and directions i,
//   colA_i[p] = sum_{q != p on the surface} sum_c dA_pq/dc_q W_c(q, i)   (c = x, y, x', y')
//   colT_i[p] = sum_{q != p on the surface} sum_c dT_pq/dc_q W_{4+c}(q, i) (c = x, y; p on the surface)
// a contraction over (q, c) of the derivative coefficients with the weights.
// A wave owns 16 targets and all directions (two 16-wide tiles when nd > 16)
// over one chunk of sources (blockIdx.y), 4 sources per step: lane l takes
// the pair (p0 + l % 16, q0 + l / 16), which is exactly the A operand it
// supplies to v_mfma_f64_16x16x4f64 (row l % 16, k slot l / 16), forms kappa
// once (kappa64: near pairs from the exact difference) and one coefficient
// per component c, and the B operand is W_c(q0 + l / 16, 16 t + l % 16).
// With S = (w/2) z'_q kappa and R = -(1/2) z'_p kappa:
//   dS/dz_q = -(w/4) z'_q (1 + kappa^2), dS/dz'_q = (w/2) kappa (surface rows
//   take Im S, wall rows -Re S), dR/dz_q = (w/4) z'_p (1 + kappa^2) (Re R).
// Result element r of lane l is target p0 + l / 16 + 4 r, direction l % 16.
__global__ __launch_bounds__(256) void k_tlm_cols(Nodes N, int n0, int n, int nd, int chunk,
                                                  const double *__restrict__ W,
                                                  double *__restrict__ pA,
                                                  double *__restrict__ pT) {
    typedef double v4d __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int p0 = (blockIdx.x * 4 + wv) * 16;
    if (p0 >= n) return;                        // whole waves; no barriers below
    const int il = lane & 15, kq = lane >> 4;
    const int p = p0 + il;
    const bool live = p < n;
    const Tgt t = load_tgt(N, live ? p : n - 1);
    const bool surf = t.k == 0;
    const bool tpart = p0 < n0;                 // the tile holds surface targets
    const bool two = nd > 16;
    const int qb = blockIdx.y * chunk, qe = min(n0, qb + chunk);
    v4d a0 = {0.0, 0.0, 0.0, 0.0}, a1 = a0, t0 = a0, t1 = a0;
    // the step's source and weights, loaded one step ahead
    auto weights = [&](int qc, double (&wo)[12]) __attribute__((always_inline)) {
        const double *w = W + (long)qc * 6 * kTlmMax + il;
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            wo[2 * c] = w[c * kTlmMax];
            wo[2 * c + 1] = w[c * kTlmMax + 16];
        }
    };
    Src s = load_src(N, min(qb + kq, n0 - 1));
    double wc[12];
    weights(min(qb + kq, n0 - 1), wc);
    for (int qs = qb; qs < qe; qs += 4) {
        const int q = qs + kq;
        const int qn = min(qs + 4 + kq, n0 - 1);
        const Src sn = load_src(N, qn);
        double wn[12];
        weights(qn, wn);
        double ca[4] = {0.0, 0.0, 0.0, 0.0}, ct[2] = {0.0, 0.0};
        if (live && q < qe && q != p) {
            double cr, ci;
            kappa64(N, t, s, cr, ci);
            const Cx Q{1.0 + cr * cr - ci * ci, 2.0 * cr * ci};
            const Cx dz = cscale(cmul({s.dx, s.dy}, Q), -0.25 * s.w);
            const Cx dd = cscale({cr, ci}, 0.5 * s.w);
            if (surf) {
                ca[0] = dz.im; ca[1] = dz.re; ca[2] = dd.im; ca[3] = dd.re;
                const Cx dr = cscale(cmul({t.dx, t.dy}, Q), 0.25 * s.w);
                ct[0] = dr.re; ct[1] = -dr.im;
            } else {
                ca[0] = -dz.re; ca[1] = dz.im; ca[2] = -dd.re; ca[3] = dd.im;
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            a0 = __builtin_amdgcn_mfma_f64_16x16x4f64(ca[c], wc[2 * c], a0, 0, 0, 0);
            if (two) a1 = __builtin_amdgcn_mfma_f64_16x16x4f64(ca[c], wc[2 * c + 1], a1, 0, 0, 0);
        }
        if (tpart) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                t0 = __builtin_amdgcn_mfma_f64_16x16x4f64(ct[c], wc[8 + 2 * c], t0, 0, 0, 0);
                if (two)
                    t1 = __builtin_amdgcn_mfma_f64_16x16x4f64(ct[c], wc[9 + 2 * c], t1, 0, 0, 0);
            }
        }
        s = sn;
#pragma unroll
        for (int e = 0; e < 12; ++e) wc[e] = wn[e];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = p0 + kq + 4 * r;
        const long sa = (long)blockIdx.y * nd;
        if (row < n) {
            if (il < nd) pA[(sa + il) * n + row] = a0[r];
            if (two && il + 16 < nd) pA[(sa + il + 16) * n + row] = a1[r];
        }
        if (tpart && row < n0) {
            if (il < nd) pT[(sa + il) * n0 + row] = t0[r];
            if (two && il + 16 < nd) pT[(sa + il + 16) * n0 + row] = t1[r];
        }
    }
}

// Right-hand sides of the nd tangent systems (rhs, system i at i * ldb, the
// surface rows negated as the solves take them) and the surface terms of dU (um, direction i at i * n0):
//   rhs_i = [p on the surface] (dphi~_i - row terms of dA omega) - colA_i,
//   um_i = d u_mv + row terms of dT gamma + colT_i - U ds,
// the row terms being the adjoint's row sums times the direction at the node
// plus the diagonal limits' derivatives.
__global__ void k_tlm_rhs(Nodes N, Flow F, int n0, int n, int nd, const double *__restrict__ dirs,
                          const double *__restrict__ omega, const double *__restrict__ gamma,
                          const double *__restrict__ U, const double *__restrict__ prow, long st,
                          const double *__restrict__ pA, const double *__restrict__ pT, int nsc,
                          double *rhs, long ldb, double *um) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    const int i = blockIdx.y;
    if (r >= n) return;
    double colA = 0.0;
    for (int b = 0; b < nsc; ++b) colA += pA[((long)b * nd + i) * n + r];
    if (r >= n0) {
        rhs[i * ldb + r] = -colA;
        return;
    }
    double R[6];
    for (int k = 0; k < 6; ++k) R[k] = prow[k * st + r];
    double colT = 0.0;
    for (int b = 0; b < nsc; ++b) colT += pT[((long)b * nd + i) * n0 + r];
    double d[7];
    for (int c = 0; c < 7; ++c) d[c] = dirs[((long)c * nd + i) * n0 + r];
    const double x = N.x[r], y = N.y[r], dx = N.dx[r], dy = N.dy[r];
    const double s = N.s[r], w = N.w[r];
    Cx dLdd, dLde;
    diag_limit_derivs(dx, dy, N.ddx[r], N.ddy[r], dLdd, dLde);
    const Cx a = cmul(dLdd, {d[2], d[3]}), b2 = cmul(dLde, {d[4], d[5]});
    const Cx dL{a.re + b2.re, a.im + b2.im};
    double ux, uy, udx, udy;
    umv_derivs(F, x, y, dx, dy, ux, uy, udx, udy);
    const double dArow = R[0] * d[0] + R[1] * d[1] + w * omega[r] * dL.im;
    rhs[i * ldb + r] = -(d[6] - dArow - colA);
    const double dumv = ux * d[0] + uy * d[1] + udx * d[2] + udy * d[3];
    const double dTrow = R[2] * d[0] + R[3] * d[1] + R[4] * d[2] + R[5] * d[3] + w * gamma[r] * dL.re;
    const double ds = (dx * d[2] + dy * d[3]) / s;
    um[(long)i * n0 + r] = dumv + dTrow + colT - U[r] * ds;
}

// dU_i = (um_i + H d gamma_0,i / 2 + T d gamma_i) / s for every direction
// (blockIdx.y), all three terms at stride n0.
__global__ void k_tlm_finalize(int n0, const double *__restrict__ s, const double *__restrict__ um,
                               const double *__restrict__ hg, const double *__restrict__ tg,
                               double *__restrict__ dU) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n0) return;
    const long o = (long)blockIdx.y * n0 + r;
    dU[o] = (um[o] + 0.5 * hg[o] + tg[o]) / s[r];
}

// c = Ubar / s on the surface
__global__ void k_adj_c(int n0, const double *Ubar, const double *s, double *c) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r < n0) c[r] = Ubar[r] / s[r];
}

}  // namespace

// Nodes per far slice: about 1024 blocks, a multiple of 64.
static int adj_chunk_nodes(int n, int n0) {
    const int c = cdiv(n, std::max(1, cdiv(1024, cdiv(n0, 64))));
    return cdiv(c, 64) * 64;
}

// partial slices per component: far chunks plus the near slice
int adjoint_nsplit(int n, int n0) { return cdiv(n, adj_chunk_nodes(n, n0)) + 1; }

// slices of the tangent-linear column pass over the M_0 surface sources:
// about kTlmWaves waves for n targets in tiles of 16, chunks of a multiple of
// 4 sources
static int tlm_chunk(int n, int n0) {
    const int ks = std::max(1, std::min(16, cdiv(kTlmWaves, cdiv(n, 16))));
    return cdiv(cdiv(n0, ks), 4) * 4;
}
int tlm_nsplit(int n, int n0) { return cdiv(n0, tlm_chunk(n, n0)); }
size_t tlm_weights_size(int n0) { return (size_t)n0 * 6 * kTlmMax; }

void launch_tlm_cols(const Nodes &N, int n0, int n, int nd, const double *dirs,
                     const double *omega, const double *gamma, double *W, double *pA, double *pT,
                     hipStream_t st) {
    const long nw = (long)tlm_weights_size(n0);
    hipLaunchKernelGGL(k_tlm_weights, dim3(cdiv(nw, 256)), dim3(256), 0, st, n0, nd, dirs, omega,
                       gamma, W);
    const int chunk = tlm_chunk(n, n0);
    hipLaunchKernelGGL(k_tlm_cols, dim3(cdiv(n, 64), cdiv(n0, chunk)), dim3(256), 0, st, N, n0, n,
                       nd, chunk, W, pA, pT);
}

void launch_tlm_rhs(const Nodes &N, const Flow &F, int n0, int n, int nd, const double *dirs,
                    const double *omega, const double *gamma, const double *U,
                    const double *prow, const double *pA, const double *pT, double *rhs, long ldb,
                    double *um, hipStream_t st) {
    hipLaunchKernelGGL(k_tlm_rhs, dim3(cdiv(n, 256), nd), dim3(256), 0, st, N, F, n0, n, nd, dirs,
                       omega, gamma, U, prow, (long)adjoint_nsplit(n, n0) * n0, pA, pT, tlm_nsplit(n, n0), rhs, ldb,
                       um);
}

void launch_tlm_finalize(int n0, int nd, const double *s, const double *um, const double *hg,
                         const double *tg, double *dU, hipStream_t st) {
    hipLaunchKernelGGL(k_tlm_finalize, dim3(cdiv(n0, 256), nd), dim3(256), 0, st, n0, s, um, hg,
                       tg, dU);
}

void launch_adj_c(int n0, const double *Ubar, const double *s, double *c, hipStream_t st) {
    hipLaunchKernelGGL(k_adj_c, dim3(cdiv(n0, 256)), dim3(256), 0, st, n0, Ubar, s, c);
}

void launch_adj_rows(const Nodes &N, const double *hrow, int n0, int n, const double *omega,
                     const double *gamma, double *part, hipStream_t st) {
    (void)hrow;
    const int chunk = adj_chunk_nodes(n, n0), ns = cdiv(n, chunk);
    const long cs = (long)(ns + 1) * n0;
    hipLaunchKernelGGL(k_adj_rows, dim3(cdiv(n0, 64), ns), dim3(kAdjStage), 0, st, N, n0, n, chunk,
                       kNearBand, omega, gamma, part, cs);
    hipLaunchKernelGGL((k_adj_near<false>), dim3(cdiv(n0, 256 / kAdjNearLanes)), dim3(256), 0, st,
                       N, n0, kNearBand, omega, gamma, part, cs, ns);
    hipLaunchKernelGGL(k_adj_sum, dim3(cdiv(n0, 64), 6), dim3(64 * kSliceWaves), 0, st, n0, ns + 1,
                       part, cs);
}

void launch_adj_cols(const Nodes &N, int n0, int n, const double *lam, const double *cvec,
                     double *part, hipStream_t st) {
    const int chunk = adj_chunk_nodes(n, n0), ns = cdiv(n, chunk);
    const long cs = (long)(ns + 1) * n0;
    hipLaunchKernelGGL(k_adj_cols, dim3(cdiv(n0, 64), ns), dim3(kAdjStage), 0, st, N, n0, n, chunk,
                       kNearBand, lam, cvec, part, cs);
    hipLaunchKernelGGL((k_adj_near<true>), dim3(cdiv(n0, 256 / kAdjNearLanes)), dim3(256), 0, st, N,
                       n0, kNearBand, lam, cvec, part, cs, ns);
    hipLaunchKernelGGL(k_adj_sum, dim3(cdiv(n0, 64), 6), dim3(64 * kSliceWaves), 0, st, n0, ns + 1,
                       part, cs);
}

void launch_adj_finalize(const Nodes &N, const Flow &F, int n0, int n, const double *Ubar,
                         const double *U, const double *omega, const double *gamma,
                         const double *lam, const double *prow, const double *pcol, double *g_phi,
                         double *g_x, double *g_y, double *g_dx, double *g_dy, double *g_ddx,
                         double *g_ddy, hipStream_t st) {
    hipLaunchKernelGGL(k_adj_finalize, dim3(cdiv(n0, 64)), dim3(64), 0, st, N, F, n0, Ubar, U,
                       omega, gamma, lam, prow, pcol, (long)adjoint_nsplit(n, n0) * n0, g_phi, g_x,
                       g_y, g_dx, g_dy, g_ddx, g_ddy);
}

}  // namespace wwbi
