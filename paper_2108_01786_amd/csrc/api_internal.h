// Host context of libwwbi (shared by the translation units of the host side).
#pragma once

#include <hip/hip_runtime.h>

#include <climits>
#include <cstddef>
#include <vector>

#include "internal.h"

namespace wwbi {

inline long round_up(long a, long b) { return (a + b - 1) / b * b; }

// Linear operators GMRES can run on.
enum OpKind {
    OP_A_S64 = 0,   // velocity-potential A, stored FP64
    OP_A_S32,       // stored FP32 (FP64 accumulation)
    OP_A_O64,       // on the fly FP64
    OP_A_O32,       // on the fly FP32 (FP64 band and limits)
    OP_AT_O64,      // transposes on the fly (a stored transpose is assembled as
    OP_AT_O32,      // A^T and applied with OP_A_S64 / OP_A_S32)
    OP_W_S64,       // vortex-sheet wall operator, stored FP64
    OP_W_O64,       // on the fly FP64
    OP_GT_S64,      // gamma_t operator (Sec. 4.2), stored FP64
    OP_GT_O64,      // on the fly FP64
    OP_GT_S32,      // stored FP32 (FP64 accumulation), inside FP64 refinement
    OP_W_S32,       // wall operator, stored FP32, inside FP64 refinement
};

// stored FP64 operators
inline bool stored_fp64(int kind) {
    return kind == OP_A_S64 || kind == OP_GT_S64 || kind == OP_W_S64;
}

// stored FP32 operators, whose products can read the FP32 copy of a basis vector
inline bool stored_fp32(int kind) {
    return kind == OP_A_S32 || kind == OP_GT_S32 || kind == OP_W_S32;
}

// The multiple of the identity in S times the operator (S: Op::flip).
inline double identity_part(int kind) {
    const bool half = kind == OP_W_S64 || kind == OP_W_O64 || kind == OP_W_S32 || kind == OP_GT_S64 ||
                      kind == OP_GT_O64 || kind == OP_GT_S32;
    return half ? -0.5 : 0.5;
}

struct Op {
    int kind;
    int n;          // operator size
    long ld;        // leading dimension of the stored matrix
    int flags;
    int band;
    int flip;       // rows [0, flip) of the operator are negated (Ctx::gmres)
};

struct SolveStats {
    int iters = 0;
    int cycles = 0;
    int refine_steps = 0;
    double rel_resid = 0.0;
};

// workspace vectors (each round_up(n, 64) doubles)
enum VecId { VR = 0, VW, VB, VX, VRR, VD, VG, VHG, VUM, VTMP, VTMP2, VLAM, VMU, VC,
             VOM, VU0, VFV, VFU, VKF, VGF, VHF, VQG, VTM, VE, kNumVec };

constexpr int kProfPairs = 2048;
constexpr int kStateSlotOffset = 8192;   // byte offset of the two polled GState slots in hst
constexpr int kStateSlotBytes = 8192;    // bytes per slot (up to kMaxMulti states)
constexpr int kTailOffset = 24576;       // byte offset of the Fourier-tail energies in hst
constexpr int kHostStaging = 32768;      // pinned host staging bytes
constexpr int kMaxMulti = 32;            // right-hand sides per multi solve
constexpr int kTwoGridPart = 100, kTwoGridNone = 101;   // Ctx::two_grid

double inner_tolerance(const wwbi_opts &o, double bnorm, double rnorm);

// One buffer of the per-solve workspace: the context's pointer and capacity
// (elements) and the element count and size a solve needs.
struct WsItem {
    void **p;
    size_t *cap;
    size_t count;
    size_t esize;
};
constexpr int kMaxWsItems = 64;

// Batched Krylov workspace of a multi right-hand-side solve.
struct MultiWS {
    double *V = nullptr; size_t cV = 0;
    float *v32 = nullptr; size_t cv32 = 0;
    float *x32 = nullptr; size_t cx32 = 0;
    double *w = nullptr, *r = nullptr, *x = nullptr, *b = nullptr, *d = nullptr, *rr = nullptr;
    size_t cw = 0, cr = 0, cx = 0, cb = 0, cd = 0, crr = 0;
    double *P = nullptr; size_t cP = 0;
    double *H = nullptr; size_t cH = 0;
    double *cs = nullptr, *sn = nullptr, *g = nullptr, *y = nullptr;
    size_t ccs = 0, csn = 0, cg = 0, cy = 0;
    double *part = nullptr; size_t cpart = 0;
    double *nrm = nullptr; size_t cnrm = 0;
    GState *gs = nullptr; size_t cgs = 0;
};

struct Ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    int restart_cap = 100;

    Layout L{};
    Flow F{};
    Nodes N{};
    const double *psi_wall = nullptr;

    void *A = nullptr;      size_t capA = 0;
    double *A64 = nullptr;  size_t capA64 = 0;   // FP64 copy beside an FP32 A (multi refine)
    double *V = nullptr;    size_t capV = 0;      // vpre recycled rows, then the basis
    int vpre = 0;
    float *v32 = nullptr;   size_t capv32 = 0;
    double *Urec = nullptr; size_t capUrec = 0;   // U of the recycled space (A U = C)
    double *Brec = nullptr; size_t capBrec = 0;   // B (kRecycleMax x restart) | z
    double *vec[kNumVec] = {};  size_t capvec[kNumVec] = {};
    double *H = nullptr;    size_t capH = 0;
    double *cs = nullptr;   size_t capcs = 0;
    double *sn = nullptr;   size_t capsn = 0;
    double *gv = nullptr;   size_t capg = 0;
    double *yv = nullptr;   size_t capy = 0;
    double *P = nullptr;    size_t capP = 0;
    double *part = nullptr; size_t cappart = 0;
    double *pw = nullptr;   size_t cappw = 0;     // partials of the fused Arnoldi product
    double *hsum = nullptr; size_t caphsum = 0;   // their row sums
    // one-launch solves of small systems: exchange words and the abort tag
    // (device), results (host-mapped), and the next launch's first tag
    unsigned long long *xch = nullptr; size_t capxch = 0;
    SmallRes *hsmall = nullptr, *dsmall = nullptr;
    unsigned xtag = 1;
    int launches = 0;           // of the call so far,
    int give_up_from = INT_MAX; // and the first that gives up at once (WWBI_GIVE_UP: tests)
    bool small_cold = false;    // the queued one started from zero
    bool small_cut = false;     // and may stop short of what was asked for
    bool handed_on = false;     // it did: gmres() goes on with its own loop
    bool cold_hist = false;     // hist begins with the residual of a zero start
    // two-grid iteration: the coarse matrix, the coarse nodes' fine indices and
    // weight factors, and the coarse solution
    double *cA = nullptr;   size_t capcA = 0;
    int *cmap = nullptr;    size_t capcmap = 0;
    double *cfac = nullptr; size_t capcfac = 0;
    double *ce = nullptr;   size_t capce = 0;
    bool want_coarse = false;   // setup() measures the strips for choose_coarse()
    bool have_strips = false;
    bool a_ready = false;       // A holds the matrix of the last potential solve
    double strip[kMaxB] = {};   // strip half-width of each boundary's nodes
    int *bid = nullptr;     size_t capbid = 0;
    int *loc = nullptr;     size_t caploc = 0;
    int *Mk = nullptr;      size_t capMk = 0;
    double *wq = nullptr;   size_t capwq = 0;
    double *s = nullptr;    size_t caps = 0;
    double *lre = nullptr;  size_t caplre = 0;
    double *lim = nullptr;  size_t caplim = 0;
    double *rowD = nullptr; size_t caprowD = 0;
    double *rowH = nullptr; size_t caprowH = 0;
    double *hrow = nullptr; size_t caphrow = 0;     // (1/2) cot(pi n / M_0)
    double *eR = nullptr;   size_t capeR = 0;       // E = e^{i zeta}
    double *eI = nullptr;   size_t capeI = 0;
    double *eRl = nullptr;  size_t capeRl = 0;      // trailing parts of E
    double *eIl = nullptr;  size_t capeIl = 0;
    double *cell = nullptr; size_t capcell = 0;     // E discs of the 64-node cells
    int *nlist = nullptr;   size_t capnlist = 0;    // near-pair cell lists
    double *val = nullptr;  size_t capval = 0;
    double *apart = nullptr; size_t capapart = 0;   // adjoint partial sums
    // surface evolution: rows of D, the antiderivative and the filter on the
    // M_0 grid (recomputed when M_0 changes), stage work vectors and the
    // Runge-Kutta stage derivatives
    int ev_M = 0;
    double *evrow = nullptr; size_t capevrow = 0;    // D | INT | FILTER | sigma
    double *ew = nullptr;    size_t capew = 0;
    double *ek = nullptr;    size_t capek = 0;
    double *hop = nullptr;   size_t caphop = 0;      // interior evaluation partials
    int *hoi = nullptr;      size_t caphoi = 0;
    MultiWS mw;
    GState *gs = nullptr;
    void *hst = nullptr;    // pinned host staging (4 KiB)
    double *hstd = nullptr;     // its address on the device
    // host-mapped coherent copy of the single-solve cycle state, written by
    // the device kernels (hmir on the host, dmir its device address)
    GState *hmir = nullptr;
    GState *dmir = nullptr;
    int cyc_id = 0;            // id of the latest GMRES cycle enqueued on gs

    hipEvent_t ev[5] = {};
    hipEvent_t pollev[3] = {};   // two convergence polls and the input checks' copy
    // the single-system solve's two step polls: they only pace the host, which
    // then reads the coherent host mirror, so they skip the system-scope fence
    hipEvent_t stepev[2] = {};
    hipEvent_t prof[2 * kProfPairs] = {};
    bool profiling = false;
    // launch -> (cycle, step) of every profiled matvec; steps at or beyond a
    // cycle's completed count were no-ops (enqueued ahead of the flag poll)
    int prof_cycle[kProfPairs] = {};
    int prof_step[kProfPairs] = {};
    std::vector<int> cyc_done;   // completed steps per cycle, -1 while unknown
    // relative residuals for wwbi_report.resid_hist (capacity reserved at
    // creation; values past it are dropped, never reallocated)
    std::vector<double> hist;
    void note_resid(double r) {
        if (hist.size() < hist.capacity()) hist.push_back(r);
    }
    int cur_cycle = -1;
    int cur_step = 0;
    int last_cycle = -1;
    bool trace = false;     // WWBI_TRACE set: one stderr line per GMRES cycle
    int nprof = 0;

    long near_pairs = 0;       // near pairs outside the band of the last geometry
    int val_blocks = 1;        // blocks of the data check of the last setup
    // workspace carved from a fixed region for one call (the allocation-free
    // entry point): ensure() then checks capacities and never allocates
    bool fixed_ws = false;

    // recycle: room for the recycled space of the refinement's inner solves
    int ws_plan(int n, int restart, WsItem *it, bool recycle = true);
    // 128 doubles of norm partials behind the Gram-Schmidt partials
    double *norm_partials() const { return P + 3L * 64 * (restart_cap + 1 + vpre); }
    int ensure(int n, int restart);
    int ensure_matrix(size_t bytes);
    int ensure_matrix64(size_t bytes);
    void release();
    // check = false leaves the device-side input checks to setup_check(), so
    // that work which writes only internal buffers can be queued meanwhile
    int setup(const wwbi_geom *g, const double *phi, int nphi, bool check = true);
    int setup_check();
    // x32 (may be null): an FP32 copy of x for the stored FP32 operators
    void apply(const Op &op, const double *x, const float *x32, const double *c, double *y,
               const int *active);
    double op_bytes(const Op &op) const;
    int read_state(GState &out);
    // state at the end of the latest cycle: the published copy when it is that
    // cycle's (after a synchronisation past the cycle's end), else a copy of gs
    int final_state(GState &out);
    void prof_begin();
    void prof_end();
    // kc > 0: deflate the kc recycled vectors in front of the basis (one
    // cycle, no verification, x = the solution from zero)
    int gmres(const Op &op, const double *b, double *x, bool x_zero, double tol, int restart,
              int max_iter, int poll, bool verify, SolveStats &st, int kc = 0);
    // whether a system of n unknowns is solved in one launch (in FP64, whichever
    // precision was asked for); not for profiled calls, which time the products.
    bool small_system(int n, const wwbi_opts &o);
    // one-launch solve: the launch (false when it is not available), and the
    // wait and the result (false when gmres() has to solve, from x unless
    // x_zero)
    bool queue_small(const Op &op, const double *b, double *x, bool x_zero, double tol,
                     int restart, int max_iter);
    bool small_result(SolveStats &st, int &status, bool &x_zero);
    int small_rc = 0;
    // the launch, with its results marked as missing
    int launch_small(SmallArgs &a, int nsys);
    // words and results for nsys one-launch solves; false when out of memory
    bool ensure_small(int nsys);
    int ensure_coarse(int n, int nsys = 1);
    bool take_tags(long need, unsigned &first);
    // Coarse grid for boundaries k0.. of the current geometry, resolving its
    // strips to the best of a few accuracies that fits; false when none does
    // or the grid would be no coarser than half the nodes
    bool choose_coarse(int k0, Coarse &C) const;
    // Two-grid iteration (kernels_coarse.hip) for the operator of `mode`, op
    // its on-the-fly FP64 form, from a zero start: kTwoGridNone when it does
    // not apply or was given up (x is of no use then), kTwoGridPart when x holds
    // an unconverged iterate, WWBI_OK when ||b - op x|| <= tol ||b||, or an
    // error (< 0)
    int two_grid(int mode, const Op &op, int k0, const double *b, double *x, const wwbi_opts &o,
                 bool check_rough, SolveStats &st);
    // The same for nr systems with A and stored matrices: A64 (row stride ld)
    // for the residuals, K (n x coarse unknowns) for the corrections
    int two_grid_multi(const double *A64, long ld, double *K, size_t kcap, const double *B,
                       double *X, int nr, const wwbi_opts &o, SolveStats &st);
    void assemble_multi(int n, long ld, const wwbi_opts &o, bool stored64);
    int solve_multi(int n, long ld, int nr, const wwbi_opts &o, bool stored64, SolveStats &st);
    // Solve one second-kind system: two-grid, then (or instead) GMRES or
    // refinement on the stored matrix, which `assemble(fp32)` forms when
    // `assembled` is not yet set
    template <class Assemble>
    int solve_system(int mode, Op op, int k0, const int (&kinds)[4], const double *b, double *x,
                     bool x_zero, const wwbi_opts &o, bool check_rough, bool &assembled,
                     Assemble assemble, SolveStats &st, double &bytes);
    // the report of a small FP64 solve that was asked for in refined FP32: its
    // cycles are the refinement steps, and its stagnation a stalled refinement
    int as_refined(int status, SolveStats &st);
    double device_norm(const double *v, int n);
    int refine(const Op &op32, const Op &op64, const double *b, double *x, bool x_zero,
               const wwbi_opts &o, SolveStats &st);
    int ensure_multi(int n, int nr, int restart);
    void apply_multi(int kind, int n, long ld, const double *X, const float *X32, long xs, int nr,
                     const double *c, double *Y);
    int read_states(GState *out, int nr);
    int gmres_multi(int kind, int n, long ld, const double *B, double *X, int nr, double tol,
                    int restart, int max_iter, int poll, bool verify, SolveStats &st);
    int refine_multi(int n, long ld, const double *B, double *X, int nr, const wwbi_opts &o,
                     bool stored64, SolveStats &st);
    void eval_U_from_gamma(const double *gamma, double *U);
    void gamma_from_omega(const double *omega, double *gamma);
    static int check_opts(const wwbi_opts *o);
    void begin_report(bool prof);
    void finish_report(wwbi_report *rep, int status, const SolveStats &st, double bytes);
};

// The velocity-potential solve behind wwbi_solve_phi (its workspace is the
// context's, grown on demand unless Ctx::fixed_ws).
int solve_phi_impl(Ctx *c, const wwbi_geom *g, const double *phi, const wwbi_opts *o,
                   double *U, double *omega, double *psi_k, wwbi_report *rep);

// Looks up, once per device and with that device current, the device address
// of the allocation-free entry point's static scratch array.
void scratch_init(int device);

}  // namespace wwbi
