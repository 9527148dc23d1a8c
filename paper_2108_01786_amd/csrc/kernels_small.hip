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
// A poll gives up after kSpinTicks of the constant-rate clock or when another
// block has given up; the result is then marked as aborted and the caller
// solves by the multi-kernel loop.  That can only happen when the blocks of
// one launch are kept from running together for that long, by other work
// filling the device.
#include "entries.h"
#include "internal.h"

namespace wwbi {

namespace {

constexpr int kTS = 512;                   // threads per block
constexpr int kWS = kTS / 64;
constexpr int kSmallSteps = 48;            // at most this many steps per cycle
constexpr int kLdsBytes = 144 * 1024;      // for the basis (160 KB less the static part)
constexpr long kSpinTicks = 20000000;      // 0.2 s at 100 MHz

typedef unsigned long long u64;

__device__ __forceinline__ void put_word(u64 *p, u64 v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 get_word(const u64 *p) {
    return __hip_atomic_load(const_cast<u64 *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int CPL, int RW>
__global__ __launch_bounds__(kTS, 2) void k_small_gmres(SmallArgs a) {
    extern __shared__ double basis[];      // slot i: v_i, NP doubles (zero past n)
    constexpr int NP = 64 * CPL;
    constexpr int NE = (NP + kTS - 1) / kTS;
    __shared__ double h1[kSmallSteps + 2], h2[kSmallSteps + 2];
    __shared__ double R[kSmallSteps * (kSmallSteps + 1) / 2];
    __shared__ double cs[kSmallSteps], sn[kSmallSteps], g[kSmallSteps + 1], yv[kSmallSteps];
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
    auto product = [&](const double *v, double (&we)[NE]) __attribute__((always_inline)) {
        double acc[RW];
#pragma unroll
        for (int r = 0; r < RW; ++r) acc[r] = 0.0;
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
            const double vk = v[lane + 64 * k];
#pragma unroll
            for (int r = 0; r < RW; ++r) acc[r] += m[r][k] * vk;
        }
        u64 *buf = xch + (long)(tag & 1u) * 2 * NP;
        const u64 tg = (u64)tag << 32;
        double mine = 0.0;
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const double s = wave_total(acc[r]);
            if (lane == r) mine = s;
        }
        if (lane < RW && row0 + lane < n) {
            const u64 u = (u64)__double_as_longlong(mine);
            put_word(buf + 2 * (row0 + lane), tg | (u & 0xffffffffu));
            put_word(buf + 2 * (row0 + lane) + 1, tg | (u >> 32));
        }
        const long t0 = wall_clock64();
        int quit = 0;
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int i = t + kTS * e;
            u64 lo = 0, hi = 0;
            if (i < n) {
                for (int spin = 1;; ++spin) {
                    lo = get_word(buf + 2 * i);
                    hi = get_word(buf + 2 * i + 1);
                    if ((unsigned)(lo >> 32) == tag && (unsigned)(hi >> 32) == tag) break;
                    if ((spin & 63) == 0 &&
                        (wall_clock64() - t0 > kSpinTicks ||
                         __hip_atomic_load(a.abort_tag, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT) == a.tag)) {
                        quit = 1;
                        break;
                    }
                }
            }
            we[e] = i < n ? __longlong_as_double((long long)((lo & 0xffffffffu) | (hi << 32))) : 0.0;
        }
        if (quit) {
            stop = 2;
            a.out[sys].aborted = 1;        // whatever block 0 reports
            __hip_atomic_store(a.abort_tag, a.tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        ++tag;
    };
    // h[i] = <slot i, slot q> for i <= last, wave wv taking i = wv, wv + kWS, ...
    auto dots = [&](int q, int last, double *h) __attribute__((always_inline)) {
        double wl[CPL];
        const double *wq = basis + (long)q * NP;
#pragma unroll
        for (int k = 0; k < CPL; ++k) wl[k] = wq[lane + 64 * k];
        for (int i = wv; i <= last; i += 2 * kWS) {
            const bool two = i + kWS <= last;
            const double *v0 = basis + (long)i * NP, *v1 = two ? v0 + (long)kWS * NP : v0;
            double s0 = 0.0, s1 = 0.0;
#pragma unroll
            for (int k = 0; k < CPL; ++k) {
                s0 += v0[lane + 64 * k] * wl[k];
                s1 += v1[lane + 64 * k] * wl[k];
            }
            s0 = wave_total(s0);
            s1 = wave_total(s1);
            if (lane == 0) {
                h[i] = s0;
                if (two) h[i + kWS] = s1;
            }
        }
    };
    // we -= sum_{i <= j} h_i v_i on the thread's elements
    auto project = [&](int j, const double *h, double (&we)[NE]) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int i = t + kTS * e;
            if (i < NP) {
                const double *v = basis + i;
                double s0 = 0.0, s1 = 0.0;
                int q = 0;
                for (; q + 1 <= j; q += 2) {
                    s0 += h[q] * v[(long)q * NP];
                    s1 += h[q + 1] * v[(long)(q + 1) * NP];
                }
                if (q <= j) s0 += h[q] * v[(long)q * NP];
                we[e] -= s0 + s1;
            }
        }
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
    const double tol_abs = a.tol * bnorm;
    double beta = bnorm, prev = HUGE_VAL;
    bool aborted = false;
    // the residual of the solution in xe (through slot 0): re, its norm beta
    auto residual = [&]() __attribute__((always_inline)) {
        __syncthreads();
        store_slot(0, xe, 1.0);
        __syncthreads();
        double we[NE];
        product(basis, we);
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
    if (a.x0) {
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
        if (!(beta > tol_abs)) { status = WWBI_OK; break; }
        if (!isfinite(beta)) { status = WWBI_STAGNATED; break; }
        if (its >= a.max_iter || cycles >= a.max_cycles) { status = WWBI_NOT_CONVERGED; break; }
        if (cycles > 0 && beta > 0.99 * prev) { status = WWBI_STAGNATED; break; }
        prev = beta;
        __syncthreads();                   // slot 0 has been read by every wave
        store_slot(0, re, 1.0 / beta);
        if (t == 0) g[0] = beta;
        __syncthreads();
        const int len = min(a.steps, a.max_iter - its);
        int j = 0;
        for (;; ++j) {
            double we[NE];
            product(basis + (long)j * NP, we);
            store_slot(j + 1, we, 1.0);
            __syncthreads();
            if (stop == 2) { aborted = true; break; }
            dots(j + 1, j, h1);
            __syncthreads();
            project(j, h1, we);
            store_slot(j + 1, we, 1.0);
            __syncthreads();
            dots(j + 1, j + 1, h2);        // h2[j + 1] = ||w'||^2
            __syncthreads();
            // ||w''||^2 = ||w'||^2 - ||h2||^2: h2 is at rounding level
            double s2 = 0.0;
            for (int i = 0; i <= j; ++i) s2 += h2[i] * h2[i];
            const double q = h2[j + 1] - s2;
            const double nrm = q > 0.0 ? sqrt(q) : 0.0;
            if (t == 0) {
                // the Hessenberg column through the previous rotations, the
                // new rotation and the residual estimate
                double *col = R + j * (j + 1) / 2;
                double c = h1[0] + h2[0];
                for (int i = 0; i < j; ++i) {
                    const double d = h1[i + 1] + h2[i + 1];
                    col[i] = cs[i] * c + sn[i] * d;
                    c = cs[i] * d - sn[i] * c;
                }
                const double r = sqrt(c * c + nrm * nrm);
                const double cj = r > 0.0 ? c / r : 1.0, sj = r > 0.0 ? nrm / r : 0.0;
                cs[j] = cj;
                sn[j] = sj;
                col[j] = r;
                const double gj = g[j];
                g[j] = cj * gj;
                g[j + 1] = -sj * gj;
                if (fabs(g[j + 1]) <= tol_abs || !(nrm > 0.0) || j + 1 >= len) stop = 1;
            }
            project(j, h2, we);
            store_slot(j + 1, we, nrm > 0.0 ? 1.0 / nrm : 0.0);
            __syncthreads();
            if (stop) break;
        }
        if (aborted) break;
        const int k = j + 1;
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

template <int CPL, int RW>
int launch_cpl(SmallArgs a, int nsys, hipStream_t st) {
    const int slots = kLdsBytes / (64 * CPL * 8);
    a.steps = a.steps < slots - 1 ? a.steps : slots - 1;
    a.steps = a.steps < kSmallSteps ? a.steps : kSmallSteps;
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

int launch_small_gmres(SmallArgs a, int nsys, hipStream_t st) {
    // columns per lane in steps of two; the rows per wave keep the matrix
    // within 144 registers a lane and a launch within 32 blocks (of whole
    // systems; 128 at the largest coarse one)
    const int cpl = (cdiv(a.n, 64) + 1) / 2 * 2;
    // A block's basis fills the LDS of its CU.  Where many systems would not
    // all be resident, more rows per wave run more of them at once (32 of 512
    // unknowns: 8 blocks each, one round of 256 blocks instead of four).
    if (nsys > 1 && cpl <= 10 && (long)nsys * cdiv(a.n, 2 * kWS) > 256) {
        switch (cpl) {
        case 2: return launch_cpl<2, 8>(a, nsys, st);
        case 4: return launch_cpl<4, 8>(a, nsys, st);
        case 6: return launch_cpl<6, 8>(a, nsys, st);
        case 8: return launch_cpl<8, 8>(a, nsys, st);
        default: return launch_cpl<10, 10>(a, nsys, st);
        }
    }
    switch (cpl) {
    case 2: return launch_cpl<2, 2>(a, nsys, st);
    case 4: return launch_cpl<4, 2>(a, nsys, st);
    case 6: return launch_cpl<6, 2>(a, nsys, st);
    case 8: return launch_cpl<8, 2>(a, nsys, st);
    case 10: return launch_cpl<10, 3>(a, nsys, st);
    case 12: return launch_cpl<12, 4>(a, nsys, st);
    case 14: return launch_cpl<14, 4>(a, nsys, st);
    case 16: return launch_cpl<16, 4>(a, nsys, st);
    case 18: case 20: return launch_cpl<20, 3>(a, nsys, st);
    case 22: case 24: return launch_cpl<24, 2>(a, nsys, st);
    case 26: case 28: return launch_cpl<28, 2>(a, nsys, st);
    case 30: case 32: return launch_cpl<32, 2>(a, nsys, st);
    default: return WWBI_EINVAL_SIZE;
    }
}

}  // namespace wwbi
