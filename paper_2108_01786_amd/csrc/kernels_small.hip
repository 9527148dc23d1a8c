// Restarted GMRES of a small system in one launch.
//
// Below about a thousand unknowns an Arnoldi step of the multi-kernel loop is
// all latency: four launches of 3 to 7 us each for a product that reads a few
// megabytes.  Here the whole solve is one kernel.  The matrix is spread over
// the registers of a few dozen blocks (RW rows per wave, lane l holding
// columns l, l + 64, ...), every block keeps the whole Krylov basis in its
// LDS and repeats the Gram-Schmidt, Givens and norm arithmetic on it, so the
// blocks exchange nothing but the product's rows, once per step.  All blocks
// take the same operations in the same order on the same data: they agree
// bit for bit on every coefficient and on where a cycle ends.
//
// The exchange.  A row's value travels as two 8-byte words, each holding 32
// bits of the value and a 32-bit tag, written and read with relaxed
// agent-scope atomics; a reader polls the words themselves until both carry
// the step's tag, so no barrier, counter or fence is needed.  Measured alone,
// one exchange of n values between 8 to 64 blocks takes 1.3 us (n = 512) to
// 1.9 us (n = 1024).  Words alternate between two buffers: a block writes
// step s + 2 only after it has read all of step s + 1, which every block
// writes after reading all of step s.  Tags are new for every launch (the
// caller's counter), so nothing has to be cleared.
//
// A poll gives up after a limit on the constant-rate clock or when another
// block has given up; the result is then marked as aborted and the caller
// solves by the multi-kernel loop.  That can only happen when the blocks of
// one launch are kept from running together for that long, by other work
// filling the device.  In the first exchange the limit is kStartTicks, longer
// than most kernels that the blocks may have to wait for: those that wait hold a
// CU each, and launches of 128 of them (2048 unknowns) on three streams could
// each hold part of the device and wait for the rest (not seen in 48 solves on
// four streams).  The first to give up would let the others run.  Once all blocks
// have met they stay resident, and the later limit only ends a launch whose queue
// was set aside.
#include "entries.h"
#include "internal.h"

namespace wwbi {

namespace {

constexpr int kTS = 512;                   // threads per block
constexpr int kWS = kTS / 64;
constexpr int kSmallSteps = 32;            // at most this many steps per cycle
constexpr int kLdsBytes = 145 * 1024;      // for the basis (160 KB less the static part)
constexpr long kStartTicks = 2000000;      // 20 ms at 100 MHz
constexpr long kSpinTicks = 20000000;      // 0.2 s
constexpr int kResident = 256;             // blocks, one to a CU

typedef unsigned long long u64;

__device__ __forceinline__ void put_word(u64 *p, u64 v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 get_word(const u64 *p) {
    return __hip_atomic_load(const_cast<u64 *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int W> struct Width { static constexpr int value = W; };

template <int CPL, int RW>
__global__ __launch_bounds__(kTS, 2) void k_small_gmres(SmallArgs a) {
    extern __shared__ double basis[];      // slot i: v_i, NP doubles (zero past n)
    constexpr int NP = 64 * CPL;
    constexpr int NE = (NP + kTS - 1) / kTS;
    // the shapes of many systems side by side, each block with many rows
    constexpr bool kMany = RW >= 8;
    __shared__ double h1[kSmallSteps + 2], h2[kSmallSteps + 2];
    __shared__ double R[kSmallSteps * (kSmallSteps + 1) / 2];
    constexpr int kQ = kSmallSteps + 1;    // Q[k * kQ + i]: the rotations' product, entry (i, k)
    __shared__ double Q[kQ * kQ];
    __shared__ double g[kSmallSteps + 1], yv[kSmallSteps];
    __shared__ int stop;                   // 1: the cycle ends, 2: a poll gave up
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int sys = blockIdx.y, n = a.n;
    const double *b = a.b + (long)sys * a.bs;
    double *x = a.x + (long)sys * a.xs;
    u64 *xch = a.xch + (long)sys * a.xchs;
    const int row0 = (blockIdx.x * kWS + wv) * RW;

    // this wave's rows of S A
    double m[RW][CPL];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int row = row0 + r;
        const double *ar = a.A + (long)(row < n ? row : 0) * a.ld;
        const double sg = row < a.flip ? -1.0 : 1.0;
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
            const int c = lane + 64 * k;
            m[r][k] = (row < n && c < n) ? sg * ar[c] : 0.0;
        }
    }
    if (t == 0) stop = 0;
    unsigned tag = a.tag;                  // of the next exchange

    // w = S A v for the vector in LDS slot `from`, received whole into we
    // (element t + kTS e of thread t); false when a poll gave up
    auto product = [&](const double *v, double (&we)[NE], auto meanwhile)
                       __attribute__((always_inline)) {
        double acc[RW];
#pragma unroll
        for (int r = 0; r < RW; ++r) acc[r] = 0.0;
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
            const double vk = v[lane + 64 * k];
#pragma unroll
            for (int r = 0; r < RW; ++r) acc[r] += m[r][k] * vk;
        }
        u64 *blo = xch + (long)(tag & 1u) * 2 * NP, *bhi = blo + NP;   // low and high halves
        const u64 tg = (u64)tag << 32;
#pragma unroll
        for (int r = 0; r < RW; ++r) acc[r] = wave_sum63(acc[r]);
        // lanes 2 r and 2 r + 1 write row r's words, all in one store (a store
        // each by the lane that holds the sums took 25 of 137 us of a solve
        // with 2 rows, n = 580)
        double mine = 0.0;
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const double s = lane_value(acc[r], 63);
            if (lane >> 1 == r) mine = s;
        }
        if (lane < 2 * RW && row0 + (lane >> 1) < n) {
            const u64 u = (u64)__double_as_longlong(mine);
            put_word((lane & 1 ? bhi : blo) + row0 + (lane >> 1),
                     tg | (lane & 1 ? u >> 32 : u & 0xffffffffu));
        }
        meanwhile();
        const long t0 = wall_clock64(), limit = tag == a.tag ? a.wait : kSpinTicks;
        int quit = 0;
        u64 lo[NE], hi[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e) lo[e] = hi[e] = tg;     // elements past n need no word
        for (int spin = 1;; ++spin) {
            bool all = true;
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                const int i = t + kTS * e;
                if (i < n) {
                    lo[e] = get_word(blo + i);
                    hi[e] = get_word(bhi + i);
                }
            }
#pragma unroll
            for (int e = 0; e < NE; ++e)
                all = all && (unsigned)(lo[e] >> 32) == tag && (unsigned)(hi[e] >> 32) == tag;
            if (all) break;
            if ((spin & 63) == 0 &&
                (wall_clock64() - t0 > limit ||
                 __hip_atomic_load(a.abort_tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                     a.tag)) {
                quit = 1;
                break;
            }
        }
#pragma unroll
        for (int e = 0; e < NE; ++e)
            we[e] = t + kTS * e < n
                        ? __longlong_as_double((long long)((lo[e] & 0xffffffffu) | (hi[e] << 32)))
                        : 0.0;
        if (quit) {
            stop = 2;
            __hip_atomic_store(a.abort_tag, a.tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            a.out[sys].aborted = 1;        // whatever block 0 reports
        }
        ++tag;
    };
    // h[i] = <slot i, slot q> for i <= last, wave wv taking i = wv, wv + kWS, ...
    auto dots = [&](int q, int last, double *h) __attribute__((always_inline)) {
        double wl[CPL];
        const double *wq = basis + (long)q * NP + lane;
#pragma unroll
        for (int k = 0; k < CPL; ++k) wl[k] = wq[64 * k];
        int i = wv;
        for (; i + kWS <= last; i += 2 * kWS) {
            const double *v0 = basis + (long)i * NP + lane;
            double s0 = 0.0, s1 = 0.0, u0 = 0.0, u1 = 0.0;
#pragma unroll
            for (int k = 0; k + 1 < CPL; k += 2) {
                s0 += v0[64 * k] * wl[k];
                s1 += v0[kWS * NP + 64 * k] * wl[k];
                u0 += v0[64 * k + 64] * wl[k + 1];
                u1 += v0[kWS * NP + 64 * k + 64] * wl[k + 1];
            }
            s0 = wave_sum63(s0 + u0);
            s1 = wave_sum63(s1 + u1);
            if (lane == 63) {
                h[i] = s0;
                h[i + kWS] = s1;
            }
        }
        if (i <= last) {
            const double *v0 = basis + (long)i * NP + lane;
            double s0 = 0.0, u0 = 0.0;
#pragma unroll
            for (int k = 0; k + 1 < CPL; k += 2) {
                s0 += v0[64 * k] * wl[k];
                u0 += v0[64 * k + 64] * wl[k + 1];
            }
            s0 = wave_sum63(s0 + u0);
            if (lane == 63) h[i] = s0;
        }
    };
    // we -= sum_{i < k} h_i v_i on the thread's elements, in groups of eight,
    // four, two and one so that each group's reads are in flight together
    auto project = [&](int k, const double *h, double (&we)[NE]) __attribute__((always_inline)) {
        const double *v[NE];
        double s0[NE], s1[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            // threads past the padded length repeat an element they drop
            v[e] = basis + (t + kTS * e < NP ? t + kTS * e : 0);
            s0[e] = s1[e] = 0.0;
        }
        int q = 0;
        auto group = [&](auto width) __attribute__((always_inline)) {
            constexpr int W = decltype(width)::value;
            double u[NE][W], hq[W];
#pragma unroll
            for (int c = 0; c < W; ++c) {
                hq[c] = h[q + c];
#pragma unroll
                for (int e = 0; e < NE; ++e) u[e][c] = v[e][(long)(q + c) * NP];
            }
#pragma unroll
            for (int c = 0; c < W; ++c)
#pragma unroll
                for (int e = 0; e < NE; ++e) {
                    if (c & 1) s1[e] += hq[c] * u[e][c];
                    else s0[e] += hq[c] * u[e][c];
                }
            q += W;
        };
        if constexpr (NE <= 2 && !kMany) {
            while (q + 8 <= k) group(Width<8>{});
            if (k & 4) group(Width<4>{});
        } else {
            while (q + 4 <= k) group(Width<4>{});       // eight would spill
        }
        if (k & 2) group(Width<2>{});
        if (k & 1) group(Width<1>{});
#pragma unroll
        for (int e = 0; e < NE; ++e) we[e] -= s0[e] + s1[e];
    };
    auto store_slot = [&](int q, const double (&we)[NE], double sc) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int i = t + kTS * e;
            if (i < NP) basis[(long)q * NP + i] = we[e] * sc;
        }
    };
    // sqrt(sum of squares of slot q): every wave for itself
    auto slot_norm = [&](int q) __attribute__((always_inline)) {
        const double *wq = basis + (long)q * NP;
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < CPL; ++k) s += wq[lane + 64 * k] * wq[lane + 64 * k];
        return sqrt(wave_total(s));
    };

    double tol_abs = 0.0;
    // Column j of the Hessenberg matrix, its rotation and the residual
    // estimate, by wave 0; sets stop when the cycle ends with step j.
    auto rotate = [&](int j, int len, double nrm) __attribute__((always_inline)) {
        if (wv != 0) return;
        // The Hessenberg column through the previous rotations, whose
        // product is kept as a matrix: lane i forms entry i from
        // independent reads, where applying them one by one is a chain.
        const double hj = lane <= j ? h1[lane] + h2[lane] : 0.0;
        double r0 = 0.0, r1 = 0.0;
        const double *Qi = Q + (lane <= j ? lane : 0);
        int k = 0;
        for (; k + 1 <= j; k += 2) {
            r0 += lane_value(hj, k) * Qi[k * kQ];
            r1 += lane_value(hj, k + 1) * Qi[(k + 1) * kQ];
        }
        if (k <= j) r0 += lane_value(hj, k) * Qi[k * kQ];
        r0 += r1;
        double *col = R + j * (j + 1) / 2;
        const double c = lane_value(r0, j);
        const double r = sqrt(c * c + nrm * nrm);
        const double ir = r > 0.0 ? 1.0 / r : 0.0;
        const double cj = r > 0.0 ? c * ir : 1.0, sj = nrm * ir;
        if (lane <= j) {
            col[lane] = lane < j ? r0 : r;
            // rows j and j + 1 of the product, (Q_j, e_{j+1}) rotated
            const double qj = Q[lane * kQ + j];
            Q[lane * kQ + j] = cj * qj;
            Q[lane * kQ + j + 1] = -sj * qj;
        }
        if (lane < j) Q[(j + 1) * kQ + lane] = 0.0;
        if (lane == j + 1) {
            Q[lane * kQ + j] = sj;
            Q[lane * kQ + j + 1] = cj;
        }
        if (lane == 0) {
            const double gj = g[j];
            g[j] = cj * gj;
            g[j + 1] = -sj * gj;
            if (fabs(sj * gj) <= tol_abs || !(nrm > 0.0) || j + 1 >= len) stop = 1;
        }
    };

    double xe[NE], re[NE];                 // solution and residual, thread t's elements
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const int i = t + kTS * e;
        xe[e] = 0.0;
        re[e] = i < n ? b[a.map ? a.map[i] : i] * (a.scale ? a.scale[i] : 1.0) : 0.0;
    }
    store_slot(0, re, 1.0);
    __syncthreads();
    const double bnorm = slot_norm(0);
    tol_abs = a.tol * bnorm;
    double beta = bnorm, prev = HUGE_VAL;
    bool aborted = a.give_up != 0;
    // the residual of the solution in xe (through slot 0): re, its norm beta
    auto residual = [&]() __attribute__((always_inline)) {
        __syncthreads();
        store_slot(0, xe, 1.0);
        __syncthreads();
        double we[NE];
        product(basis, we, [] {});
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int i = t + kTS * e;
            re[e] = i < n ? b[a.map ? a.map[i] : i] * (a.scale ? a.scale[i] : 1.0) - we[e] : 0.0;
        }
        __syncthreads();
        if (stop == 2) { aborted = true; return; }
        store_slot(0, re, 1.0);
        __syncthreads();
        beta = slot_norm(0);
    };
    if (a.x0 && !aborted) {
        const double *x0 = a.x0 + (long)sys * a.xs;
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int i = t + kTS * e;
            xe[e] = i < n ? x0[i] : 0.0;
        }
        residual();
    }
    int its = 0, cycles = 0, status = WWBI_NOT_CONVERGED, nhist = 0;
    const bool writer = blockIdx.x == 0 && t == 0;
    SmallRes *out = a.out + sys;
    while (!aborted) {
        // re = the true residual of xe, beta its norm, slot 0 = re
        if (writer && nhist < WWBI_HIST_MAX) out->hist[nhist] = bnorm > 0 ? beta / bnorm : 0.0;
        ++nhist;
        // first: a NaN is above no tolerance
        if (!isfinite(beta) || !isfinite(bnorm)) { status = WWBI_STAGNATED; break; }
        if (!(beta > tol_abs)) { status = WWBI_OK; break; }
        if (its >= a.max_iter || cycles >= a.max_cycles) { status = WWBI_NOT_CONVERGED; break; }
        if (cycles > 0) {
            const float left = __log10f((float)(beta / tol_abs)), gain = __log10f((float)(prev / beta));
            if (!(beta <= 0.99 * prev) || left > (a.spare + a.rate * left) * gain) {
                status = WWBI_STAGNATED;
                break;
            }
        }
        prev = beta;
        __syncthreads();                   // slot 0 has been read by every wave
        store_slot(0, re, 1.0 / beta);
        if (t == 0) {
            g[0] = beta;
            Q[0] = 1.0;
        }
        __syncthreads();
        const int len = min(a.steps, a.max_iter - its);
        // The rotation of step j runs while the rows of step j + 1 travel; the
        // step that ends a cycle is therefore known one product late (but for
        // the last the basis has room for), and that product is dropped.
        // (With many systems a product costs more than the wait.)
        int k = 0;                         // steps done
        double nrm = 0.0;
        for (int j = 0;; ++j) {
            double we[NE];
            product(basis + (long)j * NP, we, [&] {
                if (!kMany && j > 0) rotate(j - 1, len, nrm);
            });
            store_slot(j + 1, we, 1.0);
            __syncthreads();
            if (stop == 2) { aborted = true; break; }
            if (stop) break;
            dots(j + 1, j, h1);
            __syncthreads();
            project(j + 1, h1, we);
            store_slot(j + 1, we, 1.0);
            __syncthreads();
            dots(j + 1, j + 1, h2);        // h2[j + 1] = ||w'||^2
            __syncthreads();
            // ||w''||^2 = ||w'||^2 - ||h2||^2: h2 is at rounding level.  Lane i
            // of every wave holds h2_i (j < 64).
            const double hl = lane <= j ? h2[lane] : 0.0;
            const double ww = h2[j + 1];
            const double q = ww - wave_total(hl * hl);
            nrm = q > 0.0 ? sqrt(q) : 0.0;
            if (kMany) rotate(j, len, nrm);
            project(j + 1, h2, we);
            store_slot(j + 1, we, nrm > 0.0 ? 1.0 / nrm : 0.0);
            k = j + 1;
            __syncthreads();
            if (kMany && stop) break;
            if (!kMany && k >= len) {
                rotate(j, len, nrm);
                __syncthreads();
                break;
            }
        }
        if (aborted) break;
        its += k;
        cycles += 1;
        // y = R^{-1} g, one wave: lane i carries g_i (k <= 64)
        if (wv == 0) {
            double gi = lane < k ? g[lane] : 0.0;
            for (int l = k - 1; l >= 0; --l) {
                const double *col = R + l * (l + 1) / 2;
                const double yl = col[l] != 0.0 ? lane_value(gi, l) / col[l] : 0.0;
                if (lane == 0) yv[l] = yl;
                if (lane < l) gi -= col[lane] * yl;
            }
        }
        __syncthreads();
        if (t == 0) stop = 0;              // every thread has read it; a barrier follows
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int i = t + kTS * e;
            if (i < NP) {
                double s = xe[e];
                for (int q = 0; q < k; ++q) s += yv[q] * basis[(long)q * NP + i];
                xe[e] = s;
            }
        }
        if (!a.verify) { status = WWBI_OK; beta = fabs(g[k]); break; }
        residual();
    }
    if (aborted) status = kSmallAborted;
    // each block writes its share of the solution
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const int i = t + kTS * e;
        if (!aborted && i < n && i / (kWS * RW) == (int)blockIdx.x) x[i] = xe[e];
    }
    if (writer) {
        out->status = status;
        out->its = its;
        out->cycles = cycles;
        out->nhist = nhist < WWBI_HIST_MAX ? nhist : WWBI_HIST_MAX;
        out->bnorm = bnorm;
        out->resid = beta;
    }
}

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

// Columns per lane: in steps of two, above 16 of four.
inline int columns(int n) {
    const int c = (cdiv(n, 64) + 1) / 2 * 2;
    return c <= 16 ? c : (c + 3) / 4 * 4;
}
inline int cycle_steps(int cpl) {
    const int slots = kLdsBytes / (64 * cpl * 8);
    return slots - 1 < kSmallSteps ? slots - 1 : kSmallSteps;
}

template <int CPL, int RW>
int launch_cpl(SmallArgs a, int nsys, hipStream_t st) {
    const int most = cycle_steps(CPL);
    a.steps = a.steps < most ? a.steps : most;
    const size_t lds = (size_t)(a.steps + 1) * 64 * CPL * 8;
    static_assert(RW <= 64 && CPL * 8 * 64 * 2 <= kLdsBytes, "shape");
    const hipError_t e = hipFuncSetAttribute(
        reinterpret_cast<const void *>(&k_small_gmres<CPL, RW>),
        hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    if (e != hipSuccess) return WWBI_EHIP;
    hipLaunchKernelGGL((k_small_gmres<CPL, RW>), dim3(cdiv(a.n, kWS * RW), nsys), dim3(kTS), lds,
                       st, a);
    return WWBI_OK;
}

}  // namespace

// Words of one system's exchange buffers (two parities, two words per value).
long small_exchange_words() { return 2L * 2 * kSmallCoarseMax; }

int small_cycle_steps(int n) { return cycle_steps(columns(n)); }

namespace {

// A block's basis fills the LDS of its CU.  Where many systems would not
// all be resident, more rows per wave run more of them at once (32 of 512
// unknowns: 8 blocks each, one round of 256 blocks instead of four).
bool many_rows(int n, int nsys) {
    return nsys > 1 && columns(n) <= 10 && (long)nsys * cdiv(n, 2 * kWS) > kResident;
}

}  // namespace

int small_rounds(int n, int nsys) {
    const int rows = !many_rows(n, nsys) ? 2 : columns(n) == 10 ? 10 : 8;
    return cdiv((long)nsys * cdiv(n, rows * kWS), kResident);
}

int launch_small_gmres(SmallArgs a, int nsys, hipStream_t st) {
    const int cpl = columns(a.n);
    // a system's blocks may wait for those of the systems before it
    a.wait = kStartTicks * small_rounds(a.n, nsys);
    if (many_rows(a.n, nsys)) {
        switch (cpl) {
        case 2: return launch_cpl<2, 8>(a, nsys, st);
        case 4: return launch_cpl<4, 8>(a, nsys, st);
        case 6: return launch_cpl<6, 8>(a, nsys, st);
        case 8: return launch_cpl<8, 8>(a, nsys, st);
        default: return launch_cpl<10, 10>(a, nsys, st);
        }
    }
    // Else two rows per wave, for a short product: at most 64 blocks a system
    // up to 1024 unknowns, so that the solves of four queues are resident
    // together.  Solves of 384, 448, 580 and 864 unknowns to rounding take 64,
    // 108, 112 and 150 us; with 3 rows 66, 111, 120 and 154, with 4 a little
    // more, with 1 (448) 128.
    switch (cpl) {
    case 2: return launch_cpl<2, 2>(a, nsys, st);
    case 4: return launch_cpl<4, 2>(a, nsys, st);
    case 6: return launch_cpl<6, 2>(a, nsys, st);
    case 8: return launch_cpl<8, 2>(a, nsys, st);
    case 10: return launch_cpl<10, 2>(a, nsys, st);
    case 12: return launch_cpl<12, 2>(a, nsys, st);
    case 14: return launch_cpl<14, 2>(a, nsys, st);
    case 16: return launch_cpl<16, 2>(a, nsys, st);
    case 20: return launch_cpl<20, 2>(a, nsys, st);
    case 24: return launch_cpl<24, 2>(a, nsys, st);
    case 28: return launch_cpl<28, 2>(a, nsys, st);
    case 32: return launch_cpl<32, 2>(a, nsys, st);
    default: return WWBI_EINVAL_SIZE;
    }
}

}  // namespace wwbi
