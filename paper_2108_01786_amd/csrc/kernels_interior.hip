// Values inside the fluid from boundary values (Sec. 5.1 and the
// Helsing-Ojala appendix): for z in the fluid,
//   f(z) = sum_km lam_km f_km / sum_km lam_km,
//   lam_km = sigma_k / M_k * (1/2) cot((zeta_km - z)/2) zeta'_km,
// the trapezoid sums of contour integrals over the positively oriented
// boundary of the fluid: the free surface against its parameter
// (sigma_0 = -1), the bottom and the clockwise obstacles along theirs.
// A point that coincides with a node takes that node's value.
//
// Also the boundary velocity u - i v = (dphi/ds - i dphi/dn) |zeta'| / zeta'.
#include "ddmath.h"
#include "entries.h"
#include "internal.h"

namespace wwbi {

namespace {

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

constexpr int kHoStage = 256;

// A staged node: E, sigma w zeta' / 2 and the values of NF functions.
template <int NF> struct HoNode {
    double ex, ey, exl, eyl, a, b, f[2 * NF];
};

// Partial sums over chunk blockIdx.y of the nodes, one point per thread:
// part[c][s][p] for c = Re den, Im den, then Re and Im of each function's num;
// hit[s][p] = the first node of the chunk that coincides with the point, or
// -1.  The weights are most of a pair (30 operations of 34): two functions at
// the same points share them (6000 x 6000: 83 us a function alone, 78 for
// two).
template <int NF>
__global__ __launch_bounds__(256) void k_ho_partial(Nodes N, int n, int n0, int P,
                                                    const double *__restrict__ zx,
                                                    const double *__restrict__ zy, HoValues F,
                                                    int chunk, double *__restrict__ part,
                                                    int *__restrict__ hit) {
    __shared__ HoNode<NF> sn[kHoStage];
    const int p = blockIdx.x * 256 + threadIdx.x;
    const bool live = p < P;
    const double x = live ? zx[p] : 0.0, y = live ? zy[p] : 0.0;
    // E_z = e^{i z} as a double-double, like the nodes' E: the difference
    // E_zeta - E_z then keeps its relative accuracy for nearby points
    DD ezr, ezi;
    dd_expi(x, y, ezr, ezi);
    const double er = ezr.hi, ei = ezi.hi, erl = ezr.lo, eil = ezi.lo;
    const double cut = (er * er + ei * ei) * (1.0 / 4096.0);
    double dr = 0.0, di = 0.0, nr[NF], ni[NF];
#pragma unroll
    for (int c = 0; c < NF; ++c) nr[c] = ni[c] = 0.0;
    int h = -1;
    const int qb = blockIdx.y * chunk, qe = min(n, qb + chunk);
    for (int qq = qb; qq < qe; qq += kHoStage) {
        const int q = qq + threadIdx.x;
        if (q < qe) {
            HoNode<NF> v;
            v.ex = N.ex[q];
            v.ey = N.ey[q];
            v.exl = N.exl[q];
            v.eyl = N.eyl[q];
            const double sw = (q < n0 ? -0.5 : 0.5) * N.w[q];
            v.a = sw * N.dx[q];
            v.b = sw * N.dy[q];
#pragma unroll
            for (int c = 0; c < NF; ++c) {
                v.f[2 * c] = F.fr[c][q];
                v.f[2 * c + 1] = F.fi[c][q];
            }
            sn[threadIdx.x] = v;
        }
        __syncthreads();
        const int m = live ? min(kHoStage, qe - qq) : 0;
        for (int i = 0; i < m; ++i) {
            const HoNode<NF> &v = sn[i];
            const double ddr = (v.ex - er) + (v.exl - erl);
            const double ddi = (v.ey - ei) + (v.eyl - eil);
            const double den = ddr * ddr + ddi * ddi;
            double kr, ki;
            if (den < cut) {
                const double u = N.x[qq + i] - x, w = N.y[qq + i] - y;
                // the point is this node (or a period image)
                if (den == 0.0 || (u == 0.0 && w == 0.0)) {
                    if (h < 0) h = qq + i;
                    continue;
                }
                cot_half64(u, w, kr, ki);
            } else {
                // cot((zeta - z)/2) = i (E_zeta + E_z) / (E_zeta - E_z)
                const double sr = v.ex + er, si = v.ey + ei;
                const double inv = recip64(den);
                kr = -(si * ddr - sr * ddi) * inv;
                ki = (sr * ddr + si * ddi) * inv;
            }
            // lam = sigma w (1/2) kappa zeta'
            const double lr = kr * v.a - ki * v.b;
            const double li = kr * v.b + ki * v.a;
            dr += lr;
            di += li;
#pragma unroll
            for (int c = 0; c < NF; ++c) {
                nr[c] += lr * v.f[2 * c] - li * v.f[2 * c + 1];
                ni[c] += lr * v.f[2 * c + 1] + li * v.f[2 * c];
            }
        }
        __syncthreads();
    }
    if (live) {
        const long st = (long)gridDim.y * P;
        const long o = (long)blockIdx.y * P + p;
        part[o] = dr;
        part[st + o] = di;
#pragma unroll
        for (int c = 0; c < NF; ++c) {
            part[(2 + 2 * c) * st + o] = nr[c];
            part[(3 + 2 * c) * st + o] = ni[c];
        }
        hit[o] = h;
    }
}

// f(z) = num / den, or the coinciding node's value; neg_im stores -Im f.  64
// points per block, the slices shared by kSliceWaves waves (a thread per point
// went through them in 35 us at 6000 points and 64 slices).
template <int NF>
__global__ __launch_bounds__(64 * kSliceWaves) void k_ho_finalize(
    int P, int ns, const double *__restrict__ part, const int *__restrict__ hit, HoValues F,
    int neg_im) {
    __shared__ double red[kSliceWaves][64];
    __shared__ int first[kSliceWaves][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + lane;
    const bool live = p < P;
    int h = -1;
    const int k0 = (int)((long)ns * wv / kSliceWaves), k1 = (int)((long)ns * (wv + 1) / kSliceWaves);
    for (int s = k1 - 1; live && s >= k0; --s) {
        const int v = hit[(long)s * P + p];
        h = v >= 0 ? v : h;
    }
    first[wv][lane] = h;
    const long st = (long)ns * P;
    double v[2 + 2 * NF];
#pragma unroll
    for (int c = 0; c < 2 + 2 * NF; ++c) {
        v[c] = sum_slices_waves<kSliceWaves>(part + c * st, ns, P, p, live, red);
        __syncthreads();
    }
    if (wv != 0 || !live) return;
    h = -1;
    for (int w = kSliceWaves - 1; w >= 0; --w) h = first[w][lane] >= 0 ? first[w][lane] : h;
    const double sg = neg_im ? -1.0 : 1.0;
    const double inv = 1.0 / (v[0] * v[0] + v[1] * v[1]);
#pragma unroll
    for (int c = 0; c < NF; ++c) {
        const double nr = v[2 + 2 * c], ni = v[3 + 2 * c];
        F.outr[c][p] = h >= 0 ? F.fr[c][h] : (nr * v[0] + ni * v[1]) * inv;
        F.outi[c][p] = sg * (h >= 0 ? F.fi[c][h] : (ni * v[0] - nr * v[1]) * inv);
    }
}

// u - i v on every node from s dphi/ds and s dphi/dn:
// (dphi/ds - i dphi/dn) |zeta'| / zeta' = (sds - i sdn) / zeta';
// stores (u, v), or (Re, Im) of u - i v when phi_prime is set
__global__ void k_boundary_velocity(int n, const double *dx, const double *dy, const double *sds,
                                    const double *sdn, int phi_prime, double *u, double *v) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const double a = dx[p], b = dy[p];
    const double inv = 1.0 / (a * a + b * b);
    // (sds - i sdn) (a - i b) / |zeta'|^2
    const double re = (sds[p] * a - sdn[p] * b) * inv;
    const double im = (-sds[p] * b - sdn[p] * a) * inv;
    u[p] = re;
    v[p] = phi_prime ? im : -im;
}

// s dphi/dn = s dphi_mv/dn + local + sum of the split partials of T gamma,
// local = H gamma_0 / 2 on the surface and -gamma_k / 2 on wall k
__global__ __launch_bounds__(64 * kSliceWaves) void k_normal_finalize(
    int n, int n0, const double *umv, const double *gamma, const double *hg, const double *part,
    int nsplit, double *out) {
    __shared__ double red[kSliceWaves][64];
    const int p = blockIdx.x * 64 + (threadIdx.x & 63);
    const double acc = sum_slices_waves<kSliceWaves>(part, nsplit, n, p, p < n, red);
    if (threadIdx.x >= 64 || p >= n) return;
    const double loc = p < n0 ? 0.5 * hg[p] : -0.5 * gamma[p];
    out[p] = umv[p] + loc + acc;
}

// Dirichlet data of phi_t - C on the surface (Sec. 5.1, Laplace-Young), negated
// as the solves take the surface rows: -b with b =
// tau kappa - |grad phi|^2 / 2 - g eta, kappa = Im(zeta''/zeta')/s = 2 Im L / s
__global__ void k_pressure_data(int n0, Nodes N, const double *sds, const double *sdn,
                                double tau, double grav, double *b) {
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n0) return;
    const double s = N.s[m];
    const double a = sds[m] / s, c = sdn[m] / s;
    b[m] = -(tau * 2.0 * N.lim[m] / s - 0.5 * (a * a + c * c) - grav * N.y[m]);
}

// Fluid-side boundary values of the auxiliary Cauchy integrals:
// surface Re = the data (given negated), Im = P omega + H(omega_0)/2; wall k Re = KS omega_0 +
// GS omega_w - H(omega_k)/2, Im = psi|_k (mean of omega_k for k >= 2, 0 on
// the bottom).
__global__ void k_phi_aux_values(int n, int n0, const double *data, const double *ps,
                                 const double *rw, const double *hw, const int *bid,
                                 const double *means, double *fr, double *fi) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    if (p < n0) {
        fr[p] = -data[p];
        fi[p] = ps[p] + 0.5 * hw[p];
    } else {
        const int k = bid[p];
        fr[p] = rw[p - n0] - 0.5 * hw[p];
        fi[p] = k >= 2 ? means[k - 2] : 0.0;
    }
}

// p = -(phi_t - C) - |u - i v|^2 / 2 - g y
__global__ void k_pressure_final(int P, const double *phit, const double *wr, const double *wi,
                                 const double *zy, double grav, double *out) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    out[p] = -phit[p] - 0.5 * (wr[p] * wr[p] + wi[p] * wi[p]) - grav * zy[p];
}

}  // namespace

void launch_pressure_data(int n0, const Nodes &N, const double *sds, const double *sdn,
                          double tau, double grav, double *b, hipStream_t st) {
    hipLaunchKernelGGL(k_pressure_data, dim3(cdiv(n0, 256)), dim3(256), 0, st, n0, N, sds, sdn,
                       tau, grav, b);
}

void launch_phi_aux_values(int n, int n0, const double *data, const double *ps,
                           const double *rw, const double *hw, const int *bid,
                           const double *means, double *fr, double *fi, hipStream_t st) {
    hipLaunchKernelGGL(k_phi_aux_values, dim3(cdiv(n, 256)), dim3(256), 0, st, n, n0, data, ps, rw,
                       hw, bid, means, fr, fi);
}

void launch_pressure_final(int P, const double *phit, const double *wr, const double *wi,
                           const double *zy, double grav, double *out, hipStream_t st) {
    hipLaunchKernelGGL(k_pressure_final, dim3(cdiv(P, 256)), dim3(256), 0, st, P, phit, wr, wi, zy,
                       grav, out);
}

static int ho_chunk(int P, int n) {
    int ns = cdiv(2048, cdiv(P, 256));
    ns = ns < 1 ? 1 : (ns > 64 ? 64 : ns);
    int c = cdiv(n, ns);
    c = cdiv(c, 32) * 32;
    return c < 32 ? 32 : c;
}

int ho_slices(int P, int n) { return cdiv(n, ho_chunk(P, n)); }

namespace {
// out[0] = points with a non-finite coordinate, out[1] = points with |y| above
// the node height limit (one block; the counts are exact small integers)
__global__ __launch_bounds__(256) void k_check_points(int P, const double *__restrict__ zx,
                                                      const double *__restrict__ zy,
                                                      double *__restrict__ out) {
    __shared__ double sh[8];
    double bad = 0.0, far = 0.0;
    for (int p = threadIdx.x; p < P; p += blockDim.x) {
        const double x = zx[p], y = zy[p];
        const bool fin = isfinite(x) && isfinite(y);
        bad += fin ? 0.0 : 1.0;
        far += fin && fabs(y) > kMaxAbsY ? 1.0 : 0.0;
    }
    for (int o = 32; o > 0; o >>= 1) {
        bad += __shfl_xor(bad, o, 64);
        far += __shfl_xor(far, o, 64);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sh[2 * w] = bad;
        sh[2 * w + 1] = far;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double b = 0.0, f = 0.0;
        for (int i = 0; i < (int)(blockDim.x >> 6); ++i) {
            b += sh[2 * i];
            f += sh[2 * i + 1];
        }
        out[0] = b;
        out[1] = f;
    }
}
}  // namespace

void launch_check_points(int P, const double *zx, const double *zy, double *out,
                         hipStream_t st) {
    hipLaunchKernelGGL(k_check_points, dim3(1), dim3(256), 0, st, P, zx, zy, out);
}

void launch_helsing_ojala(const Nodes &N, int n, int n0, int P, const double *zx,
                          const double *zy, const HoValues &F, int nf, double *part, int *hit,
                          bool neg_im, hipStream_t st) {
    const int chunk = ho_chunk(P, n);
    const int ns = cdiv(n, chunk);
    const dim3 grid(cdiv(P, 256), ns), fin(cdiv(P, 64));
    if (nf == 2) {
        hipLaunchKernelGGL(k_ho_partial<2>, grid, dim3(256), 0, st, N, n, n0, P, zx, zy, F, chunk,
                           part, hit);
        hipLaunchKernelGGL(k_ho_finalize<2>, fin, dim3(64 * kSliceWaves), 0, st, P, ns, part, hit, F,
                           neg_im ? 1 : 0);
    } else {
        hipLaunchKernelGGL(k_ho_partial<1>, grid, dim3(256), 0, st, N, n, n0, P, zx, zy, F, chunk,
                           part, hit);
        hipLaunchKernelGGL(k_ho_finalize<1>, fin, dim3(64 * kSliceWaves), 0, st, P, ns, part, hit, F,
                           neg_im ? 1 : 0);
    }
}

void launch_boundary_velocity(int n, const double *dx, const double *dy, const double *sds,
                              const double *sdn, bool phi_prime, double *u, double *v,
                              hipStream_t st) {
    hipLaunchKernelGGL(k_boundary_velocity, dim3(cdiv(n, 256)), dim3(256), 0, st, n, dx, dy, sds,
                       sdn, phi_prime ? 1 : 0, u, v);
}

void launch_normal_finalize(int n, int n0, const double *umv, const double *gamma,
                            const double *hg, const double *part, int nsplit, double *out,
                            hipStream_t st) {
    hipLaunchKernelGGL(k_normal_finalize, dim3(cdiv(n, 64)), dim3(64 * kSliceWaves), 0, st, n,
                       n0, umv, gamma, hg, part, nsplit, out);
}

}  // namespace wwbi
