// Far field of the on-the-fly FP64 products through cell moments.
//
// An on-the-fly product evaluates 20 to 30 FP64 operations for each of its
// n^2 pairs: at n = 40960 1.17 ms of pure arithmetic (1.4 pairs a ns, about
// 70% of the FP64 rate), the most of a large solve.  But nearly all pairs are
// far apart, and with E = e^{i zeta} the kernel is a Cauchy kernel,
//     kappa_pq = i (E_q + E_p) / (E_q - E_p) = i (1 + 2 E_p / (E_q - E_p)),
// so the 64 consecutive nodes of a cell (centre c, radius r in the E plane)
// act on a target through the moments of their weights c_q alone,
//     sum_q c_q / (E_q - E_p) = -(1 / z) sum_k m_k t^k,
//     z = E_p - c,  t = r / z,  m_k = sum_q c_q ((E_q - c) / r)^k,
// which converges like |t|^k.  A wave takes 64 targets against a cell with as
// many terms as its nearest target needs (8 to 28) for |t|^K <= 2^-54, the
// rounding of the sum itself: 8 to 28 complex multiply-adds instead of 64
// pairs.  Cells nearer than 1 / 0.263 radii, and those that straddle two
// boundaries, are summed pair by pair in the quotient form, without the
// same-boundary band, which like the near pairs is the caller's (k_near_band,
// k_near_fix).  E's trailing parts enter z and E_q - c, so both keep their
// relative accuracy however close the cell.
//
// The Hilbert regulariser h = (1/2) cot((alpha_q - alpha_p) / 2) of some
// modes is the same kernel on the unit circle; in the frame of the cell's
// node l_c, 1 / (e^{i (alpha_p - alpha_c)} - 1) = -(1/2) - i h(l_p - l_c), a
// table value, and sum_q c_q h_pq = Im(A) / 2 - h(l_p - l_c) Re(A), A = sum
// of the circle's moments times t^k.
//
// At 40960 nodes the product of A takes 146 us for 1165 pair by pair, at 10240
// 35 for 88, and 6 for the moments; near cells are most of the small ones. Its
// errors against extended precision are those of the pairwise sums (rms 0.8 to
// 1.6e-16 at 5002 to 10240 nodes on unit data, before 0.7 to 1.6e-16).
#include <algorithm>

#include "entries.h"
#include "internal.h"

namespace wwbi {

namespace {

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

// A cell's record: the sum of its weights, centre, radius, boundary, first and
// last summed node's index there, M; its moments in E, and on the circle.
constexpr int kMom = 28;
constexpr int kRecHead = 8;
constexpr int kRecE = kRecHead + 2 * kMom, kRecH = kRecE + 2 * kMom;
static_assert(kRecH <= kCellMomentVecs * kCellNodes, "the records' place behind the slices");

// Modes as of the on-the-fly products: weights w x zeta' / 2 (the source
// flavours), or w x (the target flavours), or x alone (outputs are sources).
__host__ __device__ constexpr bool source_flavour(int mode) {
    return mode == 0 || mode == 4 || mode == 6 || mode == 7;
}
__host__ __device__ constexpr bool has_h(int mode) {
    return mode == 2 || mode == 4 || mode == 5 || mode == 7;
}

// Radius of a cell of 64 nodes on the circle, about its node 32.
__device__ __forceinline__ double circle_radius(int M) {
    return M > kCellNodes ? 2.0 * sinpi((double)(kCellNodes / 2) / (double)M) : 2.0;
}

// One block per cell b overlapping the summed nodes [s0, s0 + ns): wave 0 the
// moments in E, wave 1 (modes with h) those on the circle.
template <int MODE, bool COLS>
__global__ __launch_bounds__(has_h(MODE) ? 128 : 64) void k_cell_moments(
    Nodes N, int s0, int ns, const double *__restrict__ x, double *mom, const int *active) {
    if (active && *active == 0) return;
    const int lane = threadIdx.x & 63, b = s0 / kCellNodes + blockIdx.x;
    const bool circle = has_h(MODE) && threadIdx.x >= 64;
    const int q = b * kCellNodes + lane;
    const bool in = q >= s0 && q < s0 + ns;
    const int qc = min(q, N.n - 1);
    const double xq = in ? x[q - s0] : 0.0;
    const double wx = COLS ? xq : N.w[qc] * xq;
    const double *cell = N.cell + 4 * b;
    double *rec = mom + (long)b * kRecH;
    double cr = wx, ci = 0.0, ur, ui;
    if (circle) {
        // e^{i (alpha_q - alpha_c)} - 1 over the radius, the centre at the
        // cell's node 32 (only whole cells are used)
        const int M = N.Mk[qc];
        const double th = (double)(lane - kCellNodes / 2) / (double)M;
        const double sh = sinpi(th), ch = cospi(th), ih = 1.0 / circle_radius(M);
        ur = -2.0 * sh * sh * ih;
        ui = 2.0 * sh * ch * ih;
    } else {
        const double ir = cell[2] > 0.0 ? 1.0 / cell[2] : 0.0;
        ur = ((N.ex[qc] - cell[0]) + N.exl[qc]) * ir;
        ui = ((N.ey[qc] - cell[1]) + N.eyl[qc]) * ir;
        if (!COLS && source_flavour(MODE)) {
            cr = 0.5 * wx * N.dx[qc];
            ci = 0.5 * wx * N.dy[qc];
        }
    }
    double mr = 0.0, mi = 0.0;           // lane k keeps moment k
    for (int k = 0; k < kMom; ++k) {
        const double tr = wave_total(cr), ti = wave_total(ci);
        if (lane == k) { mr = tr; mi = ti; }
        const double a = cr * ur - ci * ui;
        ci = cr * ui + ci * ur;
        cr = a;
    }
    double *m = rec + (circle ? kRecE : kRecHead);
    if (lane < kMom) {
        m[2 * lane] = mr;
        m[2 * lane + 1] = mi;
    }
    if (circle) return;
    const double sum = wave_total(wx);
    if (lane == 0) {
        const int qa = max(b * kCellNodes, s0), qb = min(b * kCellNodes + kCellNodes, s0 + ns) - 1;
        rec[0] = sum;
        rec[1] = cell[0];
        rec[2] = cell[1];
        rec[3] = cell[2];
        // -1: the cell straddles two boundaries
        rec[4] = N.bid[qb] == N.bid[qa] ? (double)N.bid[qa] : -1.0;
        rec[5] = (double)N.loc[qa];
        rec[6] = (double)N.loc[qb];
        rec[7] = (double)N.Mk[qa];
    }
}

// sum_{k < K} m_k t^k
template <int K>
__device__ __forceinline__ void horner(const double *__restrict__ m, double tr, double ti,
                                       double &ar, double &ai) {
    double r = m[2 * K - 2], i = m[2 * K - 1];
#pragma unroll
    for (int k = K - 2; k >= 0; --k) {
        const double a = fma(r, tr, fma(-i, ti, m[2 * k]));
        i = fma(r, ti, fma(i, tr, m[2 * k + 1]));
        r = a;
    }
    ar = r;
    ai = i;
}

// |t|^2 up to which K terms leave less than 2^-54 (28: the far limit)
constexpr double kReach28 = 0.0690, kReach20 = 0.0236, kReach16 = 0.00929, kReach12 = 0.00195,
                 kReach8 = 8.64e-5;

__device__ __forceinline__ void moment_sum(const double *__restrict__ m, double worst2, double tr,
                                           double ti, double &ar, double &ai) {
    if (__all(worst2 <= kReach8)) horner<8>(m, tr, ti, ar, ai);
    else if (__all(worst2 <= kReach12)) horner<12>(m, tr, ti, ar, ai);
    else if (__all(worst2 <= kReach16)) horner<16>(m, tr, ti, ar, ai);
    else if (__all(worst2 <= kReach20)) horner<20>(m, tr, ti, ar, ai);
    else horner<28>(m, tr, ti, ar, ai);
}

// A node of a near cell: E, its weight in the sums over kappa and in those
// over h and 1, its boundary and index there.
struct NearNode {
    double ex, ey, exl, eyl, cr, ci, wx;
    int k, loc;
};

// The weight times kappa for one pair, zero unless `out`; SF: complex weights.
template <bool SF>
__device__ __forceinline__ void pair_term(const NearNode &c, double ox, double oy, double oxl,
                                          double oyl, bool out, double &kr, double &ki) {
    const double dr = (c.ex - ox) + (c.exl - oxl), di = (c.ey - oy) + (c.eyl - oyl);
    const double nr = c.ex + ox, ni = c.ey + oy;
    double inv = recip64(dr * dr + di * di);
    inv = out ? inv : 0.0;
    // kappa = -pi + i pr
    const double pr = nr * dr + ni * di, pi = ni * dr - nr * di;
    if (SF) {
        kr = -(c.cr * pi + c.ci * pr) * inv;
        ki = (c.cr * pr - c.ci * pi) * inv;
    } else {
        const double g = c.cr * inv;
        kr = -g * pi;
        ki = g * pr;
    }
}

constexpr int kCellWaves = 4;
constexpr int kStageCells = 16;          // records in LDS at a time
constexpr int kShare = kCellNodes / kCellWaves;

// One block per 64-node cell of outputs (nodes [o0, o0 + no)) and chunk of
// cells of summed nodes [s0, s0 + ns), its waves taking the cells in turn:
// slice blockIdx.y of part.
template <int MODE, bool COLS>
__global__ __launch_bounds__(64 * kCellWaves, 4) void k_cell_far(
    Nodes N, const double *hrow, int o0, int no, int s0, int ns, int corr, int chunk,
    const double *__restrict__ x, const double *__restrict__ mom, double *__restrict__ part,
    const int *active) {
    if (active && *active == 0) return;
    constexpr bool SF = !COLS && source_flavour(MODE), H = has_h(MODE);
    constexpr int nb = kNearBand, REC = H ? kRecH : kRecE;
    constexpr int kStageLoads = (kStageCells * REC + 64 * kCellWaves - 1) / (64 * kCellWaves);
    __shared__ double recs[kStageCells * REC];
    __shared__ double red[kCellWaves][64];
    __shared__ int near[kStageCells];
    __shared__ NearNode nodes[kCellWaves * kCellNodes];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int p = (o0 / kCellNodes + blockIdx.x) * kCellNodes + lane;
    const bool live = p >= o0 && p < o0 + no;
    const int me = min(max(p, o0), o0 + no - 1);
    Tgt t;       // the output node: a target, or (COLS) a source
    Src s;
    if (COLS) s = load_src(N, me);
    else t = load_tgt(N, me);
    const int mk = COLS ? s.k : t.k, ml = COLS ? s.loc : t.loc, mM = COLS ? s.M : t.M;
    const double ox = COLS ? s.ex : t.ex, oy = COLS ? s.ey : t.ey;
    const double oxl = COLS ? s.exl : t.exl, oyl = COLS ? s.eyl : t.eyl;
    // sums over the far cells of the surface (0) and of the walls (1): of the
    // weights (c) and of the weights over E_q - E_p (f)
    double c0r = 0.0, c0i = 0.0, f0r = 0.0, f0i = 0.0;
    double c1r = 0.0, c1i = 0.0, f1r = 0.0, f1i = 0.0;
    // sums of the weights times kappa, h and 1
    double k0r = 0.0, k0i = 0.0, k1r = 0.0, k1i = 0.0, hs = 0.0, es = 0.0, acc = 0.0;
    const int cfirst = s0 / kCellNodes, clast = (s0 + ns - 1) / kCellNodes;
    const int cb = cfirst + blockIdx.y * chunk, ce = min(clast + 1, cb + chunk);
    for (int b0 = cb; b0 < ce; b0 += kStageCells) {
        const int bn = min(kStageCells, ce - b0);
        if (b0 > cb) __syncthreads();      // the records and flags have been read
        // all of a thread's loads in flight before the first is stored
        double in[kStageLoads];
#pragma unroll
        for (int u = 0; u < kStageLoads; ++u) {
            const int i = u * 64 * kCellWaves + threadIdx.x;
            in[u] = i < bn * REC ? mom[(long)(b0 + i / REC) * kRecH + i % REC] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kStageLoads; ++u) {
            const int i = u * 64 * kCellWaves + threadIdx.x;
            if (i < kStageCells * REC) recs[i] = in[u];
        }
        __syncthreads();
        for (int i = wv; i < bn; i += kCellWaves) {
            const double *rec = recs + i * REC;
            const int b = b0 + i, kb = __builtin_amdgcn_readfirstlane((int)rec[4]);
            const int la = (int)rec[5], lb = (int)rec[6];
            const double zr = (ox - rec[1]) + oxl, zi = (oy - rec[2]) + oyl, r = rec[3];
            const double inv = recip64(zr * zr + zi * zi);
            double t2 = r * r * inv;
            bool reach = t2 <= kReach28;
            const bool own = mk == kb;
            const bool with_h = H && own && (MODE == 7 || (MODE == 5 ? kb != 0 : kb == 0));
            // apart by index too: no pair of a far cell is in the band
            const int gap = max(la - ml, ml - lb), span = max(lb - ml, ml - la);
            const bool apart = !own || (gap > nb && mM - span > nb);
            // (with h, full cells only: the centre is then one of its nodes)
            const bool whole = kb >= 0 && (!H || lb - la == kCellNodes - 1);
            double h = 0.0, rh = 0.0;
            if (with_h && whole) {
                // h(l_p - l_c), from the boundary's row
                int d = ml - (la + kCellNodes / 2);
                d += d < 0 ? mM : 0;
                h = hrow[me - ml + d];
                rh = circle_radius(mM);
                const double th2 = rh * rh * (0.25 + h * h);
                reach = reach && th2 <= kReach28;
                t2 = max(t2, th2);
            }
            const int all_apart = __all(apart);
            if (lane == 0) near[i] = 0;
            if (whole && __all(!live || (apart && reach))) {
                const double *m = rec + kRecHead;
                const double w2 = live ? t2 : 0.0;
                const double vr = zr * inv, vi = -zi * inv;      // 1 / z
                double ar, ai;
                moment_sum(m, w2, r * vr, r * vi, ar, ai);
                const double fr = vr * ar - vi * ai, fi = vr * ai + vi * ar;
                if (kb == 0) {
                    f0r -= fr;
                    f0i -= fi;
                    c0r += m[0];
                    c0i += m[1];
                } else {
                    f1r -= fr;
                    f1i -= fi;
                    c1r += m[0];
                    c1i += m[1];
                }
                if (MODE == 0 && own) es += rec[0];
                if (H && __any(with_h)) {
                    moment_sum(rec + kRecE, with_h ? w2 : 0.0, -0.5 * rh, -h * rh, ar, ai);
                    hs += with_h ? 0.5 * ai - h * ar : 0.0;
                }
            } else if (lane == 0) {
                // 1: pair by pair, 2: also none of the pairs is in the band
                near[i] = kb >= 0 && all_apart ? 2 : 1;
            }
        }
        __syncthreads();
        // The near cells, pair by pair, four cells at a time staged by the
        // block: wave w takes kShare nodes of each.
        const int kind = lane < bn ? near[lane] : 0;
        unsigned long long todo = __ballot(kind != 0);
        while (todo) {
            // this batch: the cells of the next four bits, wave w stages its own
            int cells[kCellWaves], kinds = 0, cnt = 0;
#pragma unroll
            for (int u = 0; u < kCellWaves; ++u) {
                cells[u] = todo ? __builtin_ctzll(todo) : -1;
                if (todo) {
                    kinds |= (__builtin_amdgcn_readlane(kind, cells[u]) == 2) << u;
                    ++cnt;
                    todo &= todo - 1;
                }
            }
            int mine = cells[0];
#pragma unroll
            for (int u = 1; u < kCellWaves; ++u) mine = wv == u ? cells[u] : mine;
            if (mine >= 0) {
                const int a = (b0 + mine) * kCellNodes + lane;
                const int q = min(max(a, s0), s0 + ns - 1);
                const double xq = a == q ? x[q - s0] : 0.0;
                NearNode v;
                v.ex = N.ex[q];
                v.ey = N.ey[q];
                v.exl = N.exl[q];
                v.eyl = N.eyl[q];
                v.wx = COLS ? xq : N.w[q] * xq;
                v.cr = SF ? 0.5 * v.wx * N.dx[q] : v.wx;
                v.ci = SF ? 0.5 * v.wx * N.dy[q] : 0.0;
                v.k = N.bid[q];
                v.loc = N.loc[q];
                nodes[wv * kCellNodes + lane] = v;
            }
            __syncthreads();
            for (int u = 0; u < cnt; ++u) {
                const NearNode *f = nodes + u * kCellNodes + kShare * wv;
                int cu = cells[0];
#pragma unroll
                for (int v = 1; v < kCellWaves; ++v) cu = u == v ? cells[v] : cu;
                const int kb = __builtin_amdgcn_readfirstlane((int)recs[cu * REC + 4]);
                const bool h_any = H && (kb < 0 || MODE == 7 || (MODE == 5 ? kb != 0 : kb == 0)) &&
                                   __any(kb < 0 || mk == kb);
                double pr0 = 0.0, pi0 = 0.0, pr1 = 0.0, pi1 = 0.0;
                if (((kinds >> u) & 1) && !h_any) {
                    // one boundary, no pair in the band, no h
                    double w = 0.0;
#pragma unroll 2
                    for (int j = 0; j < kShare; ++j) {
                        double kr, ki;
                        pair_term<SF>(f[j], ox, oy, oxl, oyl, true, kr, ki);
                        pr0 += kr;
                        pi0 += ki;
                        if (MODE == 0) w += f[j].wx;
                    }
                    if (MODE == 0 && mk == kb) es += w;
                    if (kb != 0) {
                        pr1 = pr0;
                        pi1 = pi0;
                        pr0 = pi0 = 0.0;
                    }
                } else {
#pragma unroll 2
                    for (int j = 0; j < kShare; ++j) {
                        const NearNode &c = f[j];
                        const bool own = c.k == mk;
                        const bool out = !own || cyc_dist(ml, c.loc, mM) > nb;
                        double kr, ki;
                        pair_term<SF>(c, ox, oy, oxl, oyl, out, kr, ki);
                        pr0 += c.k == 0 ? kr : 0.0;
                        pi0 += c.k == 0 ? ki : 0.0;
                        pr1 += c.k == 0 ? 0.0 : kr;
                        pi1 += c.k == 0 ? 0.0 : ki;
                        if (MODE == 0) es += own && out ? c.wx : 0.0;
                        if (H) {
                            const bool wh = own && out &&
                                            (MODE == 7 || (MODE == 5 ? c.k != 0 : c.k == 0));
                            hs += wh ? c.wx * hrow_lookup(hrow + (me - ml), c.loc, ml, mM) : 0.0;
                        }
                    }
                }
                k0r += pr0;
                k0i += pi0;
                k1r += pr1;
                k1i += pi1;
            }
            __syncthreads();
        }
    }
    // the far cells' sums of kappa, i (C + 2 E_p F)
    k0r -= c0i + 2.0 * (ox * f0i + oy * f0r);
    k0i += c0r + 2.0 * (ox * f0r - oy * f0i);
    k1r -= c1i + 2.0 * (ox * f1i + oy * f1r);
    k1i += c1r + 2.0 * (ox * f1r - oy * f1i);
    if (COLS) {
        // kappa of the pair is minus that of the swapped pair; times w zeta' / 2
        const double a = -0.5 * s.w * s.dx, c = -0.5 * s.w * s.dy;
        const double s0r = a * k0r - c * k0i, s0i = a * k0i + c * k0r;
        const double s1r = a * k1r - c * k1i, s1i = a * k1i + c * k1r;
        acc += mk == 0 ? s0i - s1r : s0r + s1i;
        if (corr && mk >= 2) acc -= s.w * es;
    } else if (SF) {
        if (MODE == 0) {
            acc += mk == 0 ? k0i + k1r : -k0r + k1i;
            if (corr && mk >= 2) acc -= es;
        } else if (MODE == 4) {
            acc += k1i - (k0r - hs);
        } else if (MODE == 6) {
            acc += k0i + k1i;
        } else {
            acc += (k0r + k1r) - hs;
        }
    } else {
        const double r0 = -0.5 * (t.dx * k0r - t.dy * k0i), i0 = -0.5 * (t.dx * k0i + t.dy * k0r);
        const double r1 = -0.5 * (t.dx * k1r - t.dy * k1i), i1 = -0.5 * (t.dx * k1i + t.dy * k1r);
        if (MODE == 5) acc += i0 - (r1 + hs);
        else if (MODE == 8) acc += mk == 0 ? i0 - r1 : r0 + i1;
        else acc += r0 + hs + i1;
    }
    red[wv][lane] = acc;
    __syncthreads();
    if (wv == 0 && live) {
        double v = red[0][lane];
        for (int w = 1; w < kCellWaves; ++w) v += red[w][lane];
        part[(long)blockIdx.y * no + (p - o0)] = v;
    }
}

int out_cells(int o0, int no) { return (o0 + no - 1) / kCellNodes - o0 / kCellNodes + 1; }

// Cells of summed nodes per slice: up to about 4096 blocks, at most 128 slices.
int cell_chunk(int no, int ns) {
    const int oc = cdiv(no, kCellNodes) + 1, sc = cdiv(ns, kCellNodes) + 1;
    const int slices = std::max(1, std::min(128, 4096 / oc));
    return cdiv(cdiv(sc, slices), kCellWaves) * kCellWaves;
}

template <int MODE, bool COLS>
void launch_mode(const Nodes &N, const double *hrow, int o0, int no, int s0, int ns, int corr,
                 const double *x, double *part, double *mom, const int *active, hipStream_t st) {
    const int chunk = cell_chunk(no, ns);
    hipLaunchKernelGGL((k_cell_moments<MODE, COLS>), dim3(out_cells(s0, ns)),
                       dim3(has_h(MODE) ? 128 : 64), 0, st, N, s0, ns, x, mom, active);
    hipLaunchKernelGGL((k_cell_far<MODE, COLS>), dim3(out_cells(o0, no), cell_slices(no, ns)),
                       dim3(64 * kCellWaves), 0, st, N, hrow, o0, no, s0, ns, corr, chunk, x, mom,
                       part, active);
}

}  // namespace

int cell_slices(int no, int ns) {
    // the summed range may overlap one more cell than ns / 64
    return cdiv(cdiv(ns, kCellNodes) + 1, cell_chunk(no, ns));
}

void launch_cell_far(const Nodes &N, const double *hrow, int mode, bool cols, int o0, int no,
                     int s0, int ns, int corr, const double *x, double *part, double *mom,
                     const int *active, hipStream_t st) {
#define WWBI_CELL_MODE(M)                                                                        \
    case M: launch_mode<M, false>(N, hrow, o0, no, s0, ns, corr, x, part, mom, active, st); break;
    if (cols) {
        launch_mode<0, true>(N, hrow, o0, no, s0, ns, corr, x, part, mom, active, st);
        return;
    }
    switch (mode) {
        WWBI_CELL_MODE(0)
        WWBI_CELL_MODE(2)
        WWBI_CELL_MODE(3)
        WWBI_CELL_MODE(4)
        WWBI_CELL_MODE(5)
        WWBI_CELL_MODE(6)
        WWBI_CELL_MODE(7)
        WWBI_CELL_MODE(8)
    }
#undef WWBI_CELL_MODE
}

}  // namespace wwbi
