// The active-set Levenberg-Marquardt fit of the Asp-Clean2016 minor cycle
// (Zhang, Bhatnagar, Rau & Zhang 2016, Sect. 3, Eq. 4) spread over the whole
// GPU.
//
// One cooperative launch, one work-group per CU.  Work-group 0 owns the fit:
// it takes the peak, applies the stop test (Sect. 2 step 4), forms the start
// values (the simple initial values of Sect. 3, or a clamped proposal),
// selects the active set, keeps the LM state in its LDS, and after every
// trial reduces, solves and publishes the next trial point.  Every LM trial
// evaluates
//     F(theta) = sum_{U(theta)} M (M - 2 D),   H = J^T J,   g = J^T (D - M)
// over U(theta), the union of the members' windows at theta (a truncated
// Gaussian is zero outside its window, so F is the whole-image objective of
// Eq. 4 up to a constant); D is the residual with the old members' stored
// Gaussians added back.  The 256-pixel tiles of U are dealt to the first
// geff work-groups.  Per pixel, D, M, the residual r = D - M and M (M - 2 D)
// are formed in FP64 (r is a small difference of O(1) terms); J and r go to
// FP32 for the augmented Gram matrix [J r]^T [J r], summed per tile and
// Kahan-compensated across tiles, while F and chi2 stay FP64.
//
// The work-groups with tiles of a trial arrive at their group's counter (kGroup
// work-groups); work-group 0 waits for all of them before it publishes again.
// Up to eight parameters it sums their partial rows itself; above, the last
// of a group sums the group's rows in order and arrives at the top counter.
// Work-groups without tiles of a trial only take note of it.  Every wait is
// bounded; a wait that runs out marks the context with ASP_ERR_DEVICE and
// every work-group leaves.
//
// A trial is a chain of latencies, not of work: 54 k pixels on 105
// work-groups take about 2 us of arithmetic.  So the data that cross between
// work-groups inside a fit (the trial point, the partial rows) go through
// agent-scope atomic stores and loads, which write through and read the
// coherent copy, and a store is known to be there when its wave's vmcnt is
// zero.  No release or acquire of a whole cache is then needed per trial
// (measured for one publication and one arrival of 256 work-groups: 1.64 us
// against 3.58 us with releases), and a message is read in one round trip
// (FitGlobal::mail).
#include <math.h>

#include "asp_device.h"
#include "cycle.h"

namespace asp {

constexpr int kT = kFitThreads;
constexpr int kOwnMax = (kNOutMax + kT - 1) / kT;
constexpr size_t kTileBytes = sizeof(float) * kT * kTileStride;
constexpr size_t kMatBytes = sizeof(double) * kMaxN * kMaxN;
constexpr size_t kFitLds = kTileBytes + 2 * kMatBytes;   // tile (or L) | two Gram buffers
// The work-group's own partial row, at the end of the tile buffer: it is
// written when the tile is no longer read.
constexpr size_t kRowOffset = kTileBytes - sizeof(double) * kPartStride;
static_assert(kRowOffset % sizeof(double) == 0, "row alignment");
constexpr int kGroup = 16;        // work-groups per first-level arrival group
static_assert(kTileBytes >= sizeof(float) * kUpdTabFloats, "the update's tables share the tile buffer");

// Phase timer slots of DevState::prof.
enum { kPCheckin = 0, kPSetup, kPEval, kPWait, kPReduce, kPLmStep, kPCommit, kPPrepare,
       kPArrive, kPTrials, kPFits, kPEvalPx, kPSoloTrials, kPSoloPx };
static_assert(kPSoloPx + 1 == kProfSlots, "profile slots");

__device__ inline unsigned long long now_ticks() { return wall_clock64(); }

// Polling loops sleep this many units of 64 clocks between reads of a
// counter another work-group advances (fewer reads of one line while waiting).
constexpr int kPollSleep = 8;

// A member at the parameters under evaluation, and an old member's stored
// Gaussian: one run of 16-byte LDS reads each.
struct alignas(16) Member {
    double x, y, amp, inv2, invs2, invs3;   // 1 / (2 s^2), 1 / s^2, 1 / s^3
    int32_t win[4];
    double inv_wc;                          // 1 / columns of the window
    int64_t wc;
};
struct alignas(16) Stored {
    double x, y, amp, inv2;
    int32_t win[4];
};

struct WGShared {
    Member mem[kMaxM];
    Stored old[kMaxM];
    int64_t pref[kMaxM + 1];
    int32_t m, n;
    double wsum[4][3];
    unsigned long long prof[kProfSlots];   // phase timers and counts of this fit (leader)
    unsigned long long eval_px, gram_flops;   // of this fit's trials (thread 0 of the leader)
    double wred[kT / 64][4][48];
    // the reduced trial (work-group 0)
    double ge[kMaxN], Fe, chi2e;
    int64_t npx_e;
    // LM state (work-group 0)
    double th_c[kMaxN], g_c[kMaxN], lo[kMaxN], hi[kMaxN], th0[kMaxN];
    // the trial point and the old members' stored parameters; the other
    // work-groups receive them as 32-bit halves
    union { double th_e[kMaxN]; uint32_t th_e32[2 * kMaxN]; };
    union { double th_old[kMaxN]; uint32_t th_old32[2 * kMaxN]; };
    double dd[kMaxN], rhs[kMaxN], delta[kMaxN];
    double ldiag[kMaxN];           // L_kk of the work-group Cholesky
    int32_t frozen[kMaxN];
    double F_c, chi2_c, mu, nu, pred, chi2_init, peak;
    int32_t trials, trials_total, converged, used_fallback, use_prop, pass, phase;
    int32_t members[kMaxM];
    int64_t idx, npx_c;
    // selection scratch
    uint32_t mask[kT];
    double t0[4];                  // the start of the new component (simple or smoothing)
    double alt[4];                 // a proposal start, compared with t0 by the objective
    int32_t alt_pending, chose_prop;
    int32_t hsel;                  // which of the two Gram buffers holds the current point
    double sel[3];                 // (x, y, s) of the start: the active set is selected around it
    int32_t use_smooth;            // the start is the smoothing method's
    int32_t nch, sel_done;
    unsigned long long key;        // the peak key of this fit (collect_peak_key)
    // batched fields (leader and followers)
    int32_t cmd, fld, go;
    int64_t k_target, upx;
    // messages (the other work-groups: the last one read)
    unsigned int gen;              // sequence number
    unsigned int fit_no;           // leader: the fit's number, 0 before its first trial
    unsigned int fit_have;         // others: the fit whose th_old is held
    unsigned int epoch, epoch_have;   // of R (batched fields)
    int32_t geff, poll_n;          // geff: work-groups of the trial, 0 = the leader alone
    // control
    unsigned long long tmark;      // phase timer mark (thread 0)
    unsigned long long tfit;       // start of the fit (thread 0)
    unsigned long long tlaunch;    // start of the launch (thread 0)
    int32_t fresh;                 // the message opened a fit: th_old is new
    int32_t last, abort, solve, pd, ok, finished, accept, stop;
    int32_t upd;                   // the fit committed and this launch also updates R
    int32_t more;                  // and another iteration follows it in this launch
};

// A launch of several iterations ends after the iteration that passes this
// share of the wait limit of 2 s: 10 ms.
constexpr unsigned long long kLaunchShare = 200;

// Phase timers of the driving work-group (thread 0): the mark lives in LDS so
// that no tick value stays in registers across a phase.
__device__ inline void mark(WGShared &S)
{
    if (threadIdx.x == 0) S.tmark = now_ticks();
}

__device__ __forceinline__ void lap(WGShared &S, int slot)
{
    if (threadIdx.x == 0) {
        const unsigned long long now = now_ticks();
        S.prof[slot] += now - S.tmark;
        S.tmark = now;
    }
}

// The timers and counts of this fit into the device state; they start again
// from zero.  Thread 0 keeps them in LDS meanwhile: a read-modify-write of the
// device state per trial would put a memory round trip on the LM chain.
__device__ __forceinline__ void flush_counts(const Params &p, WGShared &S)
{
    if (threadIdx.x != 0) return;
    DevState *st = p.st;
    for (int i = 0; i < kProfSlots; ++i) {
        st->prof[i] += S.prof[i];
        S.prof[i] = 0ull;
    }
    st->sum_eval_px += S.eval_px;
    st->sum_gram_flops += S.gram_flops;
    S.eval_px = S.gram_flops = 0ull;
}

// Orders the LDS accesses of one wave: the lanes of a wave issue LDS
// instructions together and the LDS serves them in program order, so after
// this point every lane sees what any lane of the wave wrote before it; the
// wavefront-scope fences keep the compiler from moving accesses across.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A condition that is the same in every lane, as a scalar.
__device__ __forceinline__ bool uniform(bool b) { return __builtin_amdgcn_readfirstlane(b ? 1 : 0) != 0; }

// ---------------------------------------------------------------------------
// Synchronisation between work-groups.  Polling is relaxed (no cache
// maintenance per poll).  Data written with ordinary stores (the residual, the
// update's plan) cross by a release and an acquire at agent scope; trial points
// and partial rows cross by atomic stores and loads.
// ---------------------------------------------------------------------------

__device__ inline void acquire_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent"); }

// Loads and stores of data that cross between work-groups at agent scope: they
// read and write the coherent copy.
template <typename T>
__device__ inline T ld_shared(const T *q)
{
    return __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ inline void st_shared(T *q, T v)
{
    __hip_atomic_store(q, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Every store of this wave has reached the scope it was made at.
__device__ inline void wave_stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

enum { kCmdPeak = 1, kCmdEval = 2, kCmdUpdate = 3, kCmdExit = 4 };

// The leader's next message, by its wave 0: a command, and with kCmdEval the
// trial point S.th_e for geff work-groups, with the old members' stored
// parameters before the first trial of a fit.  release: the work-group's plain
// stores go before it (each wave has waited for its own, and a barrier).
__device__ __forceinline__ void post(FitGlobal *G, WGShared &S, int cmd, int geff, int field,
                                     bool release)
{
    static_assert(kMaxM < 32 && kCmdExit < 8 && kMaxGroups * kGroup < (1 << 24), "header bits");
    const int t = threadIdx.x;
    // the counters reset after the last trial are in place before this message
    wave_stores_done();
    if (release) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    const unsigned int gen = S.gen + 1u;
    const bool first = cmd == kCmdEval && S.fit_no == 0u;
    const unsigned int fit_no = first ? gen : S.fit_no;
    const unsigned long long tag = (unsigned long long)gen << 32;
    const int nw = cmd == kCmdEval ? 2 * S.n : 0;
    for (int w = t; w < kMailHead + nw; w += 64) {
        uint32_t v;
        if (w == 0) v = (nw ? (uint32_t)S.m : 0u) | ((uint32_t)cmd << 5) | ((uint32_t)geff << 8);
        else if (w == 1) v = fit_no;
        else if (w == 2) v = (uint32_t)field;
        else if (w == 3) v = S.epoch;
        else v = S.th_e32[w - kMailHead];
        st_shared(&G->mail[w], tag | v);
    }
    if (first)
        for (int w = 8 + t; w < nw; w += 64)
            st_shared(&G->old[w], ((unsigned long long)fit_no << 32) | S.th_old32[w]);
    if (t == 0) {
        S.gen = gen;
        if (first) S.fit_no = fit_no;
    }
    wave_lds_sync();
}

// A message by the whole work-group.
__device__ __forceinline__ void publish(FitGlobal *G, WGShared &S, int cmd, int field = 0,
                                        bool release = false)
{
    if (release) wave_stores_done();
    __syncthreads();
    if (threadIdx.x < 64) post(G, S, cmd, 0, field, release);
}

// The next message, into S (command, geff, field, epoch and, for a trial in
// which work-group `wg` has tiles, m, n, th_e and th_old); S.abort when none
// came.  For wave 0; a barrier follows before the others read S.  It polls the
// words the last message had.  A work-group without tiles may find that the
// leader has moved on; one with tiles cannot, as the leader waits for it.
// Bounded in time: `limit` device wall-clock ticks.  With `beat`, the bound
// restarts whenever the heartbeat moves: a leader that works alone for a long
// time (small fields of a batch) keeps its followers waiting without letting
// them time out.
__device__ __forceinline__ void wait_mail(FitGlobal *G, WGShared &S, int wg,
                                          unsigned long long limit, bool beat = false)
{
    const int t = threadIdx.x;
    if (t < 64) {
        const unsigned int seen = S.gen;
        int nw = S.poll_n;
        unsigned int last_beat = beat ? ld_shared(&G->beat.n) : 0u;
        unsigned long long t0 = now_ticks();
        unsigned long long w = 0ull;
        unsigned int gen = seen;
        uint32_t head = 0;
        int need = 0;
        bool ok = false;
        for (;;) {
            w = t < nw ? ld_shared(&G->mail[t]) : 0ull;
            gen = (unsigned int)__builtin_amdgcn_readfirstlane((int)(w >> 32));
            if (gen != seen) {
                head = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)w);
                const bool mine = ((head >> 5) & 7u) == kCmdEval && wg < (int)(head >> 8);
                need = kMailHead + (mine ? 8 * (int)(head & 31u) : 0);
                const int want = need < 64 ? need : 64;
                if (nw >= want && __all(t >= want || (unsigned int)(w >> 32) == gen)) {
                    ok = true;
                    break;
                }
                if (nw < want) nw = want;
            }
            const unsigned long long tn = now_ticks();
            if (beat) {
                const unsigned int b = ld_shared(&G->beat.n);
                if (b != last_beat) { last_beat = b; t0 = tn; }
            }
            if (tn - t0 > limit) break;
            if (gen == seen) __builtin_amdgcn_s_sleep(kPollSleep);
        }
        if (ok) {
            const bool mine = need > kMailHead;
            if (t >= kMailHead && t < need) S.th_e32[t - kMailHead] = (uint32_t)w;
            for (int b = 64; b < need && ok; b += 64) {
                unsigned long long x = 0ull;
                for (;;) {
                    x = b + t < need ? ld_shared(&G->mail[b + t]) : 0ull;
                    if (__all(b + t >= need || (unsigned int)(x >> 32) == gen)) break;
                    if (now_ticks() - t0 > limit) { ok = false; break; }
                }
                if (b + t < need) S.th_e32[b + t - kMailHead] = (uint32_t)x;
            }
            const unsigned int fit_no = (unsigned int)__builtin_amdgcn_readlane((int)(uint32_t)w, 1);
            const int no = 8 * (int)(head & 31u);
            const bool fresh = mine && fit_no != S.fit_have;
            if (fresh) {
                for (int b = 0; b < no && ok; b += 64) {
                    const int i = b + t;
                    const bool want = i >= 8 && i < no;
                    unsigned long long x = 0ull;
                    for (;;) {
                        x = want ? ld_shared(&G->old[i]) : 0ull;
                        if (__all(!want || (unsigned int)(x >> 32) == fit_no)) break;
                        if (now_ticks() - t0 > limit) { ok = false; break; }
                    }
                    if (want) S.th_old32[i] = (uint32_t)x;
                }
                if (t == 0) S.fit_have = fit_no;
            }
            const int field = __builtin_amdgcn_readlane((int)(uint32_t)w, 2);
            const unsigned int epoch = (unsigned int)__builtin_amdgcn_readlane((int)(uint32_t)w, 3);
            if (t == 0) {
                S.cmd = (int32_t)((head >> 5) & 7u);
                S.geff = (int32_t)(head >> 8);
                S.fld = field;
                S.epoch = epoch;
                if (mine) {
                    S.m = (int32_t)(head & 31u);
                    S.n = 4 * S.m;
                    S.poll_n = need < 64 ? need : 64;
                }
                S.fresh = fresh ? 1 : 0;
            }
        }
        if (t == 0) {
            S.gen = gen;
            S.abort = ok ? 0 : 1;
        }
        wave_lds_sync();
    }
}

// Before the first message of a launch: the number of the last one, and
// nothing held (thread 0; a barrier follows).
__device__ __forceinline__ void mail_begin(FitGlobal *G, WGShared &S)
{
    S.gen = (unsigned int)(ld_shared(&G->mail[0]) >> 32);
    S.fit_no = 0u;
    S.fit_have = 0u;
    S.epoch = S.epoch_have = 0u;
    S.poll_n = kMailHead + 8;
    S.abort = 0;
    for (int i = 0; i < kProfSlots; ++i) S.prof[i] = 0ull;
    S.eval_px = S.gram_flops = 0ull;
}

// Thread 0 waits until *ctr reaches target; returns false on timeout.
__device__ __forceinline__ bool spin_until(unsigned int *ctr, unsigned int target,
                                           unsigned long long limit)
{
    const unsigned long long t0 = now_ticks();
    while (ld_shared(ctr) < target) {
        if (now_ticks() - t0 > limit) return false;
        __builtin_amdgcn_s_sleep(kPollSleep);
    }
    return true;
}

// The leader waits until work-groups 1 .. count-1 have each arrived once at the
// counter of their group of gs, then clears the counters: lane g of wave 0
// polls group g's.  Bounded in time.
__device__ __forceinline__ bool wait_groups(FitGlobal *G, WGShared &S, int count, int gs,
                                            unsigned long long limit)
{
    const int t = threadIdx.x;
    if (t < 64) {
        const int lo = t * gs, hi = lo + gs < count ? lo + gs : count;
        const int need = hi - lo - (t == 0 ? 1 : 0);
        const bool live = need > 0;
        const unsigned long long t0 = now_ticks();
        bool ok = true;
        for (;;) {
            const unsigned int v = live ? ld_shared(&G->arrive_g[t].n) : 0u;
            if (__all(!live || (int)v >= need)) break;
            if (now_ticks() - t0 > limit) { ok = false; break; }
        }
        if (live) st_shared(&G->arrive_g[t].n, 0u);
        if (t == 0) S.abort = ok ? 0 : 1;
    }
    __syncthreads();
    return S.abort == 0;
}

// ---------------------------------------------------------------------------
// Active set (the paper names the heuristic; its definition is in the 2004
// paper).  Candidates are components whose amplitude has the peak's sign and
// whose centre lies inside the window of the simple start (the peak pixel,
// width omega_b), most recent first; skip one closer than
// max(omega_b, min(s_j, s_m)) to a member already taken (the new component
// first: at the peak pixel with width omega_b and, with a proposal, at the
// proposal too); at most K_max - 1.  FP64 products and sums are rounded
// separately, so membership is reproducible bit for bit.
// ---------------------------------------------------------------------------

__device__ inline bool too_close(double xj, double yj, double sj, double xm, double ym,
                                 double sm, double omega_b)
{
    double ex = __dsub_rn(xj, xm), ey = __dsub_rn(yj, ym);
    double rs = sj < sm ? sj : sm;
    if (rs < omega_b) rs = omega_b;
    return __dadd_rn(__dmul_rn(ex, ex), __dmul_rn(ey, ey)) <= __dmul_rn(rs, rs);
}

// Lane 0 of wave 0: greedy acceptance of candidate j.
__device__ __forceinline__ void consider(const Params &p, WGShared &S, int64_t j, double omega_b)
{
    const double xj = p.cx[j], yj = p.cy[j], sj = p.cs[j];
    if (too_close(xj, yj, sj, S.sel[0], S.sel[1], S.sel[2], omega_b)) return;
    // a proposal start is a second place of the new component
    if (S.alt_pending && too_close(xj, yj, sj, S.alt[1], S.alt[2], S.alt[3], omega_b)) return;
    for (int u = 0; u < S.nch; ++u) {
        const int64_t mj = S.members[u + 1];
        if (too_close(xj, yj, sj, p.cx[mj], p.cy[mj], p.cs[mj], omega_b)) return;
    }
    S.members[1 + S.nch] = (int32_t)j;
    S.nch++;
    if (S.nch >= p.max_active - 1) S.sel_done = 1;
}

// Start values, active set, bounds; the start point goes to S.th_e.
// Work-group 0, whole work-group.
__device__ __forceinline__ void setup_fit(const Params &p, WGShared &S, bool use_prop)
{
    const int t = threadIdx.x;
    const double omega_b = p.st->omega_b;
    if (t == 0) {
        const int64_t pr = S.idx / p.W, pc = S.idx % p.W;
        const double pv = S.peak;
        double *t0 = S.t0;
        const double cap = width_cap(p);
        if (S.use_smooth) {
            // the smoothing method's start (Sect. 2 step 1, Sect. 3)
            const double *q = p.st->smooth_start;
            t0[0] = q[0]; t0[1] = q[1]; t0[2] = q[2]; t0[3] = q[3];
        } else {
            t0[0] = pv; t0[1] = (double)pc; t0[2] = (double)pr; t0[3] = omega_b;
        }
        S.alt_pending = use_prop ? 1 : 0;
        S.chose_prop = 0;
        if (use_prop) {
            // the proposal, clamped: the peak's sign, within 16 px of the peak
            // and inside the image, omega_b <= s <= the width cap
            const double *q = p.st->proposal;
            double *a = S.alt;
            a[0] = q[0]; a[1] = q[1]; a[2] = q[2]; a[3] = q[3];
            if (!(a[0] * pv > 0.0)) a[0] = pv;     // also NaN
            if (!(a[1] >= (double)pc - 16.0)) a[1] = (double)pc - 16.0;
            if (a[1] > (double)pc + 16.0) a[1] = (double)pc + 16.0;
            if (!(a[2] >= (double)pr - 16.0)) a[2] = (double)pr - 16.0;
            if (a[2] > (double)pr + 16.0) a[2] = (double)pr + 16.0;
            if (a[1] < 0.0) a[1] = 0.0;
            if (a[1] > (double)(p.W - 1)) a[1] = (double)(p.W - 1);
            if (a[2] < 0.0) a[2] = 0.0;
            if (a[2] > (double)(p.H - 1)) a[2] = (double)(p.H - 1);
            if (!(a[3] >= omega_b)) a[3] = omega_b;
            if (a[3] > cap) a[3] = cap;
        }
        // candidates: inside the start's window (the simple start, peak pixel
        // and omega_b, also when a proposal competes; or the smoothing start)
        S.sel[0] = t0[1];
        S.sel[1] = t0[2];
        S.sel[2] = t0[3];
        make_window(t0[1], t0[2], halfwidth(t0[3], p.window_sigmas), p.H, p.W, S.mem[0].win);
        S.nch = 0;
        S.sel_done = (p.max_active <= 1) ? 1 : 0;
    }
    __syncthreads();
    const double a0 = S.t0[0];
    const int32_t b0 = S.mem[0].win[0], b1 = S.mem[0].win[1], b2 = S.mem[0].win[2],
                  b3 = S.mem[0].win[3];
    const int64_t L = p.st->L;
    constexpr int64_t kSeg = (int64_t)kT * 32;
    for (int64_t top = L; top > 0; top -= kSeg) {
        __syncthreads();
        if (S.sel_done) break;
        const int64_t lo = top - kSeg > 0 ? top - kSeg : 0;
        S.mask[t] = 0u;
        __syncthreads();
        for (int64_t j = lo + t; j < top; j += kT) {
            const double aj = p.ca[j];
            if (!(__dmul_rn(aj, a0) > 0.0)) continue;
            const double xj = p.cx[j], yj = p.cy[j];
            if (!(yj >= (double)b0 && yj <= (double)b1 && xj >= (double)b2 && xj <= (double)b3))
                continue;
            const int64_t o = j - lo;
            atomicOr(&S.mask[o >> 5], 1u << (o & 31));
        }
        __syncthreads();
        if (t < 64) {
            // words from the highest index down: lane l holds word wbase + 63 - l
            for (int wbase = kT - 64; wbase >= 0; wbase -= 64) {
                const uint32_t word = S.mask[wbase + 63 - t];
                unsigned long long nz = __ballot(word != 0u);
                while (nz) {
                    const int l = __ffsll((long long)nz) - 1;
                    nz &= nz - 1ull;
                    const uint32_t wv = __shfl(word, l, 64);
                    if (t == 0 && !S.sel_done) {
                        uint32_t bits = wv;
                        while (bits && !S.sel_done) {
                            const int b = 31 - __clz(bits);
                            bits &= ~(1u << b);
                            consider(p, S, lo + 32 * (wbase + 63 - l) + b, omega_b);
                        }
                    }
                    if (__shfl(S.sel_done, 0, 64)) break;
                }
                if (__shfl(S.sel_done, 0, 64)) break;
            }
        }
    }
    __syncthreads();
    const int m = 1 + S.nch;
    if (t == 0) {
        S.members[0] = -1;
        S.hsel = 0;
        S.m = m;
        S.n = 4 * m;
        S.phase = 0;
        S.trials = 0;
        S.converged = 0;
        S.fit_no = 0u;                 // the next message opens a fit
    }
    __syncthreads();
    if (t < m) {
        double th[4];
        if (t == 0) {
            th[0] = S.t0[0]; th[1] = S.t0[1]; th[2] = S.t0[2]; th[3] = S.t0[3];
        } else {
            const int64_t j = S.members[t];
            th[0] = p.ca[j]; th[1] = p.cx[j]; th[2] = p.cy[j]; th[3] = p.cs[j];
        }
        int32_t w[4];
        make_window(th[1], th[2], halfwidth(th[3], p.window_sigmas), p.H, p.W, w);
        if (t == 0 && S.alt_pending) {
            // two starts: the centre may range over the hull of both windows
            int32_t wa[4];
            make_window(S.alt[1], S.alt[2], halfwidth(S.alt[3], p.window_sigmas), p.H, p.W, wa);
            w[0] = wa[0] < w[0] ? wa[0] : w[0];
            w[1] = wa[1] > w[1] ? wa[1] : w[1];
            w[2] = wa[2] < w[2] ? wa[2] : w[2];
            w[3] = wa[3] > w[3] ? wa[3] : w[3];
        }
        // bounds: the start sign of the amplitude; the centre inside its start
        // window; omega_b <= s <= the width cap
        const bool neg = th[0] < 0.0;
        const double lo4[4] = {neg ? -INFINITY : 0.0, (double)w[2], (double)w[0], omega_b};
        const double hi4[4] = {neg ? 0.0 : INFINITY, (double)w[3], (double)w[1], width_cap(p)};
        for (int q = 0; q < 4; ++q) {
            const int i = 4 * t + q;
            S.lo[i] = lo4[q];
            S.hi[i] = hi4[q];
            S.th0[i] = th[q];
            S.th_old[i] = (t == 0) ? 0.0 : th[q];
            double v = th[q];
            if (!(v >= lo4[q])) v = lo4[q];
            if (v > hi4[q]) v = hi4[q];
            S.th_e[i] = v;
        }
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Evaluation of one work-group's share of U(theta).
// ---------------------------------------------------------------------------

// Entry o of the augmented Gram matrix [J r]^T [J r]: the upper triangle of
// the columns 0..n (J then the residual), row by row.
__device__ inline void out_pair(int o, int n, int &i, int &k)
{
    int r = 0, start = 0;
    while (start + (n + 1 - r) <= o) { start += n + 1 - r; ++r; }
    i = r;
    k = r + (o - start);
}

// make_window(x, y, halfwidth(s, ws), ...) in FP64: the bounds are whole
// numbers, exact there, and need no 64-bit integer conversions.
__device__ __forceinline__ void window_of(double x, double y, double s, double ws, int64_t H,
                                          int64_t W, int32_t box[4])
{
    double h = ceil(ws * s);
    if (!(h >= 3.0)) h = 3.0;
    if (h > 1073741823.0) h = 1073741823.0;
    const double cx = floor(x + 0.5), cy = floor(y + 0.5);
    const double r0 = cy - h, r1 = cy + h, c0 = cx - h, c1 = cx + h;
    const double hr = (double)(H - 1), hc = (double)(W - 1);
    box[0] = (int32_t)(r0 < 0.0 ? 0.0 : r0);
    box[1] = (int32_t)(r1 > hr ? hr : r1);
    box[2] = (int32_t)(c0 < 0.0 ? 0.0 : c0);
    box[3] = (int32_t)(c1 > hc ? hc : c1);
}

// The members' windows at S.th_e and their pixel counts laid end to end, by the
// first lanes of wave 0 (which wrote th_e, or read it after a barrier).
__device__ __forceinline__ void prepare_windows(const Params &p, WGShared &S)
{
    const int t = threadIdx.x;
    const int m = S.m;
    int64_t area = 0;
    if (t < m) {
        int32_t w[4];
        window_of(S.th_e[4 * t + 1], S.th_e[4 * t + 2], S.th_e[4 * t + 3], p.window_sigmas, p.H,
                  p.W, w);
        Member &M = S.mem[t];
        for (int q = 0; q < 4; ++q) M.win[q] = w[q];
        M.wc = w[3] - w[2] + 1;
        area = (int64_t)(w[1] - w[0] + 1) * (w[3] - w[2] + 1);
    }
    for (int off = 1; off < m; off <<= 1) {
        const int64_t v = __shfl_up((long long)area, off, 64);
        if (t >= off) area += v;
    }
    if (t < m) S.pref[t + 1] = area;
    if (t == 0) S.pref[0] = 0;
    wave_lds_sync();
}

// The members' constants, after the windows.
__device__ __forceinline__ void prepare_members(WGShared &S)
{
    const int t = threadIdx.x;
    if (t < S.m) {
        Member &M = S.mem[t];
        const double s = S.th_e[4 * t + 3], s2 = s * s;
        M.amp = S.th_e[4 * t];
        M.x = S.th_e[4 * t + 1];
        M.y = S.th_e[4 * t + 2];
        M.inv2 = 1.0 / (2.0 * s2);
        M.invs2 = 1.0 / s2;
        M.invs3 = 1.0 / (s2 * s);
        M.inv_wc = 1.0 / (double)M.wc;
    }
    wave_lds_sync();
}

// The old members' stored Gaussians at S.th_old, once per fit (wave 0).
__device__ __forceinline__ void prepare_old(const Params &p, WGShared &S)
{
    const int t = threadIdx.x;
    if (t > 0 && t < S.m) {
        const double ox = S.th_old[4 * t + 1], oy = S.th_old[4 * t + 2], os = S.th_old[4 * t + 3];
        Stored &O = S.old[t];
        O.x = ox;
        O.y = oy;
        O.amp = S.th_old[4 * t];
        O.inv2 = 1.0 / (2.0 * os * os);
        window_of(ox, oy, os, p.window_sigmas, p.H, p.W, O.win);
    }
    wave_lds_sync();
}

__device__ inline double wave_sum(double v)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Whether pixel (r, c) lies in the window, without branches between the
// comparisons (each would wait for its own LDS read).
__device__ __forceinline__ bool inside(const int32_t b[4], int32_t r, int32_t c)
{
    return (r >= b[0]) & (r <= b[1]) & (c >= b[2]) & (c <= b[3]);
}

// a / d for a < 2^32, 0 < d < 2^32 and inv = 1.0 / d: the FP64 product is off
// by less than one, so the quotient is it or a neighbour.
__device__ __forceinline__ uint32_t divide(uint32_t a, uint32_t d, double inv)
{
    uint32_t q = (uint32_t)((double)a * inv);
    const uint32_t lo = q * d;
    q -= lo > a ? 1u : 0u;
    q += a - q * d >= d ? 1u : 0u;
    return q;
}

// Pixel `lin` of the members' windows laid end to end: its place, whether it is
// a first occurrence in U, and its residual value.
struct Pixel {
    int32_t r, c;
    bool valid;
    float rv;
};

__device__ __forceinline__ Pixel locate(const Params &p, const WGShared &S, int m, int64_t lin,
                                        int64_t total)
{
    Pixel q;
    q.r = q.c = 0;
    q.rv = 0.0f;
    q.valid = lin < total;
    if (q.valid) {
        int w = 0;
        for (int k = 1; k < m; ++k) w += lin >= S.pref[k] ? 1 : 0;
        // a window lies inside the image (fewer than 2^32 pixels): 32-bit division
        const Member &M = S.mem[w];
        const uint32_t local = (uint32_t)(lin - S.pref[w]);
        const uint32_t wc = (uint32_t)M.wc;
        const uint32_t dr = divide(local, wc, M.inv_wc);
        q.r = M.win[0] + (int32_t)dr;
        q.c = M.win[2] + (int32_t)(local - dr * wc);
        bool seen = false;
        for (int i = 0; i < m - 1; ++i) seen |= (i < w) & inside(S.mem[i].win, q.r, q.c);
        q.valid = !seen;
        if (q.valid) q.rv = p.R[(int64_t)q.r * p.W + q.c];
    }
    return q;
}

// One pixel of a fit of m members: D, the model M and the row of [J r], which
// goes through put(column, value), and the sums of M (M - 2 D), (D - M)^2 and
// the pixels.  Members are taken two at a time: their exponentials (a chain of
// some 40 dependent FP64 operations each) run side by side, and a window's
// test selects the result.  A pair that no lane's pixel meets is skipped.
// The fused multiply-adds are written out (here and in evaluate_tiles_reg), so
// that every copy the compiler makes of this code rounds alike: a fit of several
// close members can turn on the last bit of F.
template <typename Put>
__device__ __forceinline__ void form_pixel(const WGShared &S, int m, const Pixel &px, Put put,
                                           double &f_acc, double &c_acc, double &npx)
{
    const double cd = (double)px.c, rd = (double)px.r;
    double D = (double)px.rv;
    for (int j = 1; j < m; j += 2) {
        const Stored a = S.old[j], b = S.old[j + 1 < m ? j + 1 : j];
        const bool ia = px.valid & inside(a.win, px.r, px.c);
        const bool ib = px.valid & (j + 1 < m) & inside(b.win, px.r, px.c);
        if (!__any(ia | ib)) continue;
        const double ax = cd - a.x, ay = rd - a.y, bx = cd - b.x, by = rd - b.y;
        const double ea = exp(-fma(ax, ax, ay * ay) * a.inv2);
        const double eb = exp(-fma(bx, bx, by * by) * b.inv2);
        const double Da = fma(a.amp, ea, D);
        D = ia ? Da : D;
        const double Db = fma(b.amp, eb, D);
        D = ib ? Db : D;
    }
    double M = 0.0;
    for (int j = 0; j < m; j += 2) {
        const bool two = j + 1 < m;
        const Member a = S.mem[j], b = S.mem[two ? j + 1 : j];
        const bool ia = px.valid & inside(a.win, px.r, px.c);
        const bool ib = px.valid & two & inside(b.win, px.r, px.c);
        float va[4] = {0.0f, 0.0f, 0.0f, 0.0f}, vb[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (__any(ia | ib)) {
            const double ax = cd - a.x, ay = rd - a.y, bx = cd - b.x, by = rd - b.y;
            const double qa = fma(ax, ax, ay * ay), qb = fma(bx, bx, by * by);
            const double ea = exp(-qa * a.inv2), eb = exp(-qb * b.inv2);
            const double Ga = a.amp * ea, Gb = b.amp * eb;
            const double Ma = fma(a.amp, ea, M);
            M = ia ? Ma : M;
            const double Mb = fma(b.amp, eb, M);
            M = ib ? Mb : M;
            va[0] = ia ? (float)ea : 0.0f;
            va[1] = ia ? (float)(Ga * ax * a.invs2) : 0.0f;
            va[2] = ia ? (float)(Ga * ay * a.invs2) : 0.0f;
            va[3] = ia ? (float)(Ga * qa * a.invs3) : 0.0f;
            vb[0] = ib ? (float)eb : 0.0f;
            vb[1] = ib ? (float)(Gb * bx * b.invs2) : 0.0f;
            vb[2] = ib ? (float)(Gb * by * b.invs2) : 0.0f;
            vb[3] = ib ? (float)(Gb * qb * b.invs3) : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) put(4 * j + u, va[u]);
        if (two) {
#pragma unroll
            for (int u = 0; u < 4; ++u) put(4 * j + 4 + u, vb[u]);
        }
    }
    const double res = D - M;
    put(4 * m, px.valid ? (float)res : 0.0f);
    const double fn = fma(M, fma(-2.0, D, M), f_acc), cn = fma(res, res, c_acc);
    f_acc = px.valid ? fn : f_acc;
    c_acc = px.valid ? cn : c_acc;
    npx += px.valid ? 1.0 : 0.0;
}

// F, chi2 and the pixel count of the work-group into out[0..2]: wave sums, then
// the four waves in order.
__device__ __forceinline__ void store_scalars(WGShared &S, double f_acc, double c_acc, double npx,
                                              double *out)
{
    const int t = threadIdx.x;
    const double f_w = wave_sum(f_acc), c_w = wave_sum(c_acc), p_w = wave_sum(npx);
    if ((t & 63) == 0) {
        S.wsum[t >> 6][0] = f_w;
        S.wsum[t >> 6][1] = c_w;
        S.wsum[t >> 6][2] = p_w;
    }
    __syncthreads();
    if (t < 3) {
        double v = 0.0;
        for (int w = 0; w < kT / 64; ++w) v += S.wsum[w][t];
        out[t] = v;
    }
    __syncthreads();
}

// Tiles tile0, tile0 + stride, ... of U for fits of sixteen members; the
// work-group's partial (FP64: n_out Gram entries, F, chi2, the pixel count)
// goes to out.  Each thread owns up to kOwnMax Gram entries: a plain FP32 sum
// over the tile's pixels, Kahan-compensated across tiles.
__device__ __forceinline__ void evaluate_tiles(const Params &p, WGShared &S, float *tile,
                                               int64_t tile0, int64_t stride, double *out)
{
    const int t = threadIdx.x;
    const int m = S.m, n = S.n;
    const int n_out = (n + 1) * (n + 2) / 2;
    int n_own = 0;
    int oi[kOwnMax], ok_[kOwnMax];
#pragma unroll
    for (int u = 0; u < kOwnMax; ++u) {
        const int o = t + u * kT;
        if (o < n_out) { out_pair(o, n, oi[u], ok_[u]); n_own = u + 1; }
    }
    float acc_s[kOwnMax], acc_c[kOwnMax];
#pragma unroll
    for (int u = 0; u < kOwnMax; ++u) { acc_s[u] = 0.0f; acc_c[u] = 0.0f; }

    const int64_t total = S.pref[m];
    const int64_t ntiles = (total + kT - 1) / kT;
    double npx = 0.0, f_acc = 0.0, c_acc = 0.0;
    float *row = tile + t * kTileStride;
    Pixel nx = locate(p, S, m, tile0 * kT + t, total);
    for (int64_t ti = tile0; ti < ntiles; ti += stride) {
        const Pixel px = nx;
        nx = locate(p, S, m, (ti + stride) * kT + t, total);   // one tile ahead
        form_pixel(S, m, px, [&](int c, float v) { row[c] = v; }, f_acc, c_acc, npx);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kOwnMax; ++u) {
            if (u >= n_own) break;
            const int ci = oi[u], ck = ok_[u];
            // four interleaved chains (pixels q, q + 4, ... in turn), added in
            // a fixed order: a quarter of the dependent adds per tile
            float ts0 = 0.0f, ts1 = 0.0f, ts2 = 0.0f, ts3 = 0.0f;
            for (int q = 0; q < kT; q += 4) {
                const float *r0 = tile + q * kTileStride, *r1 = r0 + kTileStride;
                const float *r2 = r1 + kTileStride, *r3 = r2 + kTileStride;
                ts0 += r0[ci] * r0[ck];
                ts1 += r1[ci] * r1[ck];
                ts2 += r2[ci] * r2[ck];
                ts3 += r3[ci] * r3[ck];
            }
            const float ts = (ts0 + ts1) + (ts2 + ts3);
            const float y = ts - acc_c[u];
            const float tt = acc_s[u] + y;
            acc_c[u] = (tt - acc_s[u]) - y;
            acc_s[u] = tt;
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < kOwnMax; ++u) {
        if (u >= n_own) break;
        out[t + u * kT] = (double)acc_s[u] - (double)acc_c[u];
    }
    store_scalars(S, f_acc, c_acc, npx, out + n_out);
}

// The same partial for fits of three to fifteen members with the Gram sums on
// the matrix cores.  Wave w forms its 64 rows of [J r] and keeps them in its
// own quarter of the tile buffer, column by column, and accumulates G = X^T X
// over them with v_mfma_f32_16x16x4f32 (four pixels per instruction), one
// 16 x 16 block per pair of 16-column groups (bi >= bj) of X; columns past n
// are read as zeros.  A tile's FP32 block sums are added into FP64
// accumulators, so the sums across tiles lose nothing.  No wave reads another's
// rows, so a tile costs no barrier; a column is 64 floats at a stride of 68, so
// that neither the writes (64 pixels of a column) nor the reads (16 columns of
// 4 pixels) meet in a bank.  At the end the four waves' FP64 sums are added
// through LDS in a fixed order: (w0 + w2) + (w1 + w3).
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int NB>
__device__ __forceinline__ void evaluate_tiles_mfma(const Params &p, WGShared &S, float *tile,
                                                    int64_t tile0, int64_t stride, double *out)
{
    constexpr int NBL = NB * (NB + 1) / 2, XS = 68;
    static_assert(sizeof(float) * XS * (kMaxN - 3) * (kT / 64) <= kTileBytes, "columns of 15 members");
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int m = S.m, n = S.n, C = n + 1;
    const int n_out = C * (C + 1) / 2;
    double g[NBL][4];
#pragma unroll
    for (int q = 0; q < NBL; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) g[q][r] = 0.0;

    const int64_t total = S.pref[m];
    const int64_t ntiles = (total + kT - 1) / kT;
    double npx = 0.0, f_acc = 0.0, c_acc = 0.0;
    float *xw = tile + wave * (C * XS);
    float *xput = xw + lane;
    const int kr = lane >> 4, cc = lane & 15;
    const bool last_in = (NB - 1) * 16 + cc < C;
    const float *xget = xw + cc * XS + kr;
    const float *xlast = xw + (last_in ? (NB - 1) * 16 + cc : 0) * XS + kr;
    Pixel nx = locate(p, S, m, tile0 * kT + t, total);
    for (int64_t ti = tile0; ti < ntiles; ti += stride) {
        const Pixel px = nx;
        nx = locate(p, S, m, (ti + stride) * kT + t, total);   // one tile ahead
        form_pixel(S, m, px, [&](int c, float v) { xput[c * XS] = v; }, f_acc, c_acc, npx);
        wave_lds_sync();
        f32x4 acc[NBL];
#pragma unroll
        for (int q = 0; q < NBL; ++q) acc[q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < 16; ++ks) {
            float x[NB];
#pragma unroll
            for (int b = 0; b < NB - 1; ++b) x[b] = xget[b * 16 * XS + 4 * ks];
            const float xl = xlast[4 * ks];
            x[NB - 1] = last_in ? xl : 0.0f;
            int q = 0;
#pragma unroll
            for (int bi = 0; bi < NB; ++bi)
#pragma unroll
                for (int bj = 0; bj <= bi; ++bj, ++q)
                    acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[bi], x[bj], acc[q], 0, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < NBL; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) g[q][r] += (double)acc[q][r];
        wave_lds_sync();                   // the columns are rewritten next
    }
    // Lane l of wave w holds, for block (bi, bj), the entries of rows
    // 16 bi + 4 (l / 16) + r and column 16 bj + l % 16 of G.  Entry (i, k),
    // i <= k, of the output is G[k][i], taken from block (k / 16, i / 16).
    double *buf = reinterpret_cast<double *>(tile);
    static_assert(2 * sizeof(double) * (kMaxN + 1) * (kMaxN + 2) / 2 <= kRowOffset, "wave sums");
    __syncthreads();                       // every wave's columns are read
    for (int half = 0; half < 2; ++half) {
        if ((wave >> 1) == half) {
            double *dst = buf + (wave & 1) * n_out;
            int q = 0;
#pragma unroll
            for (int bi = 0; bi < NB; ++bi)
#pragma unroll
                for (int bj = 0; bj <= bi; ++bj, ++q)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int k = 16 * bi + 4 * kr + r, i = 16 * bj + cc;
                        if (k < C && i <= k) {
                            const int o = i * C - i * (i - 1) / 2 + (k - i);
                            dst[o] = half ? dst[o] + g[q][r] : g[q][r];
                        }
                    }
        }
        __syncthreads();
    }
    for (int o = t; o < n_out; o += kT) out[o] = buf[o] + buf[n_out + o];
    store_scalars(S, f_acc, c_acc, npx, out + n_out);
}

// The same partial for fits of at most two members (n <= 8): each thread keeps
// the 15 or 45 Gram entries of its own pixels in registers, with no barrier per
// tile.  J and r are FP32 values; their products are exact in FP64 and are
// accumulated there (one FP64 FMA per entry, half the work of a Kahan update
// in FP32 on this hardware and a smaller error).  The threads' sums are
// combined once at the end through LDS and the four waves in order.
//
// With one wave per SIMD the loop is a chain of latencies (the residual's
// load, then an exponential of some 40 dependent FP64 operations), so a thread
// takes two tiles side by side, without branches between them, and loads the
// residual of the next two before it starts: the sums still add the tiles in
// order.  Over many tiles it is bound by the instructions of the one wave, some
// five clocks each: a pixel's place is advanced from the last one's, its load
// has no branch, a window's test selects the exponential alone, and a window
// that no pixel of the wave lies in is left out.  Two members on eight
// work-groups in a field of 1024 x 1024: 246 -> 203 us per trial.
template <int M>
__device__ __forceinline__ void evaluate_tiles_reg(const Params &p, WGShared &S, int64_t tile0, int64_t stride,
                                   double *out, float *stage)
{
    constexpr int N = 4 * M, C = N + 1, NO = C * (C + 1) / 2;
    const int t = threadIdx.x;
    const int64_t total = S.pref[M], first = S.pref[1];
    const int64_t ntiles = (total + kT - 1) / kT;
    Member mem[M];
#pragma unroll
    for (int j = 0; j < M; ++j) mem[j] = S.mem[j];
    Stored old = {};
    if (M > 1) old = S.old[1];
    struct Px {
        int64_t lin;
        int32_t r, c;
        bool valid, in0, in1;              // in0: listed by the first window; in1: in the last
        float rv;
    };
    // `step` pixels further in a window of wc columns: whole rows and columns
    // (found once), so that only the first pixel in a window takes a division.
    const uint32_t step = (uint32_t)(2 * stride * kT);
    uint32_t step_r[M], step_c[M];
#pragma unroll
    for (int j = 0; j < M; ++j) {
        const uint32_t wc = (uint32_t)mem[j].wc;
        step_r[j] = divide(step, wc, mem[j].inv_wc);
        step_c[j] = step - step_r[j] * wc;
    }
    // Whether the pixel is a first occurrence in U, and its residual value.
    auto look = [&](Px &q) __attribute__((always_inline)) {
        q.valid = q.lin < total;
        if (M > 1) q.valid &= q.in0 | !inside(mem[0].win, q.r, q.c);
        q.in1 = q.valid & (M == 1 || !q.in0 || inside(mem[M - 1].win, q.r, q.c));
        q.rv = p.R[q.valid ? (int64_t)q.r * p.W + q.c : 0];
    };
    // This thread's pixel of a tile: row-major within the window it falls in.
    auto enter = [&](Px &q) __attribute__((always_inline)) {
        q.r = q.c = 0;
        q.in0 = true;
        if (q.lin < total) {
            const bool second = M > 1 && q.lin >= first;
            // a window lies inside the image (fewer than 2^32 pixels): 32-bit division
            const uint32_t local = (uint32_t)(q.lin - (second ? first : 0));
            const uint32_t wc = (uint32_t)(second ? mem[M - 1].wc : mem[0].wc);
            const uint32_t dr = divide(local, wc, second ? mem[M - 1].inv_wc : mem[0].inv_wc);
            q.r = (second ? mem[M - 1].win[0] : mem[0].win[0]) + (int32_t)dr;
            q.c = (second ? mem[M - 1].win[2] : mem[0].win[2]) + (int32_t)(local - dr * wc);
            q.in0 = !second;
        }
    };
    auto place = [&](int64_t ti) __attribute__((always_inline)) {
        Px q;
        q.lin = ti * kT + t;
        enter(q);
        look(q);
        return q;
    };
    auto advance = [&](Px q) __attribute__((always_inline)) {
        q.lin += step;
        if (M > 1 && q.in0 && q.lin >= first) {
            enter(q);
        } else {
            const bool second = M > 1 && !q.in0;
            q.c += (int32_t)(second ? step_c[M - 1] : step_c[0]);
            q.r += (int32_t)(second ? step_r[M - 1] : step_r[0]);
            const bool wrap = q.c > (second ? mem[M - 1].win[3] : mem[0].win[3]);
            q.c -= wrap ? (int32_t)(second ? mem[M - 1].wc : mem[0].wc) : 0;
            q.r += wrap ? 1 : 0;
        }
        look(q);
        return q;
    };
    double acc[NO];
#pragma unroll
    for (int o = 0; o < NO; ++o) acc[o] = 0.0;
    double npx = 0.0, f_acc = 0.0, c_acc = 0.0;
    struct Cols { float col[C]; double e[M], D, Mv, res; };
    // The old member's Gaussian into D; a window's test selects the exponential,
    // so that two pixels run side by side.
    auto form_old = [&](const Px &q, bool in, Cols &o) __attribute__((always_inline)) {
        const double dx = (double)q.c - old.x, dy = (double)q.r - old.y;
        const double e = exp(-fma(dy, dy, dx * dx) * old.inv2);
        o.D = fma(old.amp, in ? e : 0.0, o.D);
    };
    // Member j's exponential and its columns of the row of [J r].
    auto form_member = [&](const Px &q, int j, bool in, Cols &o) __attribute__((always_inline)) {
        const double dx = (double)q.c - mem[j].x, dy = (double)q.r - mem[j].y;
        const double qq = fma(dy, dy, dx * dx);
        const double ew = exp(-qq * mem[j].inv2), e = in ? ew : 0.0;
        const double G = mem[j].amp * e;
        o.e[j] = e;
        o.col[4 * j] = (float)e;
        o.col[4 * j + 1] = (float)(G * dx * mem[j].invs2);
        o.col[4 * j + 2] = (float)(G * dy * mem[j].invs2);
        o.col[4 * j + 3] = (float)(G * qq * mem[j].invs3);
    };
    auto form_rest = [&](const Px &q, Cols &o) __attribute__((always_inline)) {
        o.res = o.D - o.Mv;
        o.col[N] = q.valid ? (float)o.res : 0.0f;
    };
    auto add_scalars = [&](const Px &q, const Cols &o) __attribute__((always_inline)) {
        const double fn = fma(o.Mv, fma(-2.0, o.D, o.Mv), f_acc), cn = fma(o.res, o.res, c_acc);
        f_acc = q.valid ? fn : f_acc;
        c_acc = q.valid ? cn : c_acc;
        npx += q.valid ? 1.0 : 0.0;
        acc[NO - 1] = fma((double)o.col[N], (double)o.col[N], acc[NO - 1]);
    };
    // The products of the columns of members i <= k (i = k: with the residual's
    // too), rows and columns in the order of the upper triangle.
    auto add_block = [&](const Cols &o, int bi, int bk) __attribute__((always_inline)) {
        double x[4], y[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            x[u] = (double)o.col[4 * bi + u];
            y[u] = (double)o.col[4 * bk + u];
        }
        const double r = (double)o.col[N];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = 4 * bi + u, row = i * C - i * (i - 1) / 2 - i;   // + k: entry (i, k)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (bi != bk || v >= u) acc[row + 4 * bk + v] = fma(x[u], y[v], acc[row + 4 * bk + v]);
            if (bi == bk) acc[row + N] = fma(x[u], r, acc[row + N]);
        }
    };
    Px a = place(tile0), b = place(tile0 + stride);
    for (int64_t ti = tile0; ti < ntiles; ti += 2 * stride) {
        Px na = a, nb = b;
        if (ti + 2 * stride < ntiles) {
            na = advance(a);
            nb = advance(b);
        }
        Cols ca, cb;
        ca.D = (double)a.rv;
        cb.D = (double)b.rv;
        ca.Mv = cb.Mv = 0.0;
        // A wave whose pixels all lie outside the first window leaves its
        // exponential and products (of zeros) out: most of a large second
        // window does.
        const bool a0 = a.valid & a.in0, b0 = b.valid & b.in0;
        const bool any0 = M > 1 && __any(a0 | b0);
        if (M > 1) {
            form_old(a, a.valid & inside(old.win, a.r, a.c), ca);
            form_old(b, b.valid & inside(old.win, b.r, b.c), cb);
        }
        form_member(a, M - 1, a.in1, ca);
        form_member(b, M - 1, b.in1, cb);
        if (any0) {
            form_member(a, 0, a0, ca);
            form_member(b, 0, b0, cb);
            ca.Mv = fma(mem[0].amp, ca.e[0], ca.Mv);
            cb.Mv = fma(mem[0].amp, cb.e[0], cb.Mv);
        }
        ca.Mv = fma(mem[M - 1].amp, ca.e[M - 1], ca.Mv);
        cb.Mv = fma(mem[M - 1].amp, cb.e[M - 1], cb.Mv);
        form_rest(a, ca);
        form_rest(b, cb);
        add_block(ca, M - 1, M - 1);
        add_scalars(a, ca);
        add_block(cb, M - 1, M - 1);
        add_scalars(b, cb);
        if (any0) {
            add_block(ca, 0, 0);
            add_block(ca, 0, M - 1);
            add_block(cb, 0, 0);
            add_block(cb, 0, M - 1);
        }
        a = na;
        b = nb;
    }
    const int lane = t & 63, wave = t >> 6;
    // Wave sums of the Gram entries, F, chi2 and the pixel count, through the
    // tile buffer (idle in this path), CH values at a time: each wave writes
    // its lanes' values; then lane (q, c) adds value q over lanes 16 c ..
    // 16 c + 15 in order, 16 values by all lanes and the rest by the first
    // lanes.  The four chains of the four waves meet at the end: (0 + 1) +
    // (2 + 3) of a wave, then the waves in order.  Rows are padded to 65
    // doubles, so the 32 lanes served together read 32 different bank pairs.
    constexpr int NV = NO + 3, CH = M == 1 ? 18 : 24, ROW = 65, REST = CH - 16;
    static_assert(NV % CH == 0 && REST > 0 && REST <= 8, "chunks of 17 .. 24 values");
    static_assert(sizeof(double) * (kT / 64) * CH * ROW <= kRowOffset, "reduction buffer");
    double v[NV];
#pragma unroll
    for (int o = 0; o < NO; ++o) v[o] = acc[o];
    v[NO] = f_acc;
    v[NO + 1] = c_acc;
    v[NO + 2] = npx;
    double *buf = reinterpret_cast<double *>(stage) + wave * (CH * ROW);
    const int qa = lane & 15, va = lane >> 4;
    const int qb = 16 + (lane & 7), vb = (lane >> 3) & 3;
    const bool has_b = lane < 32 && qb < CH;
    const double *ra = buf + qa * ROW + 16 * va, *rb = buf + (has_b ? qb : 0) * ROW + 16 * vb;
#pragma unroll
    for (int h = 0; h < NV / CH; ++h) {
        if (h > 0) wave_lds_sync();        // the buffer has been read
#pragma unroll
        for (int q = 0; q < CH; ++q) buf[q * ROW + lane] = v[h * CH + q];
        wave_lds_sync();
        double sa = 0.0, sb = 0.0;
#pragma unroll
        for (int l = 0; l < 16; ++l) {
            sa += ra[l];
            sb += rb[l];
        }
        S.wred[wave][va][h * CH + qa] = sa;
        if (has_b) S.wred[wave][vb][h * CH + qb] = sb;
    }
    __syncthreads();
    if (t < NV) {
        double tot = 0.0;
#pragma unroll
        for (int w = 0; w < kT / 64; ++w)
            tot += (S.wred[w][0][t] + S.wred[w][1][t]) + (S.wred[w][2][t] + S.wred[w][3][t]);
        out[t] = tot;
    }
    __syncthreads();
}

// Rows w0..w1-1 of the partials summed in row order, sixteen loads in flight.
__device__ __forceinline__ double sum_column(const Params &p, int w0, int w1, int o)
{
    double v = 0.0;
    for (int w = w0; w < w1; w += 16) {
        double a[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int r = w + u < w1 ? w + u : w1 - 1;   // rows past the last: read, not added
            a[u] = ld_shared(p.partials + (int64_t)r * kPartStride + o);
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const double s = v + a[u];
            v = w + u < w1 ? s : v;
        }
    }
    return v;
}

// Entry o of a trial's sums, to where the LM step reads it: He, S.ge, S.Fe,
// S.chi2e, S.npx_e.
__device__ __forceinline__ void put_sum(WGShared &S, double *He, int n, int o, double v)
{
    const int n_out = (n + 1) * (n + 2) / 2;
    if (o >= n_out) {
        if (o == n_out) S.Fe = v;
        else if (o == n_out + 1) S.chi2e = v;
        else S.npx_e = (int64_t)v;
        return;
    }
    int i, k;
    out_pair(o, n, i, k);
    if (i < n && k < n) { He[i * n + k] = v; He[k * n + i] = v; }
    else if (i < n) S.ge[i] = v;
}

// ---------------------------------------------------------------------------
// The LM bookkeeping (Marquardt 1963) after one evaluation, work-group 0.
// Damped system (H + mu D) delta = g with D = diag(max(H_ii, 1e-12 max
// H_ii)); a parameter on a bound whose gradient leaves the box is held for
// the trial; the trial point is clipped to the bounds; accept iff F
// decreases; gain-ratio damping (mu *= max(1/3, 1 - (2 rho - 1)^3) on accept,
// mu *= nu, nu *= 2 on reject); converged when an accepted step has
// max |delta_k| / scale_k < tol, or stalled once mu passes 1e8; the budget
// counts trials.  Sets S.finished when the fit is over; otherwise S.th_e
// holds the next trial point.
// ---------------------------------------------------------------------------

// Lane l's value in every lane (l the same for all lanes).
__device__ __forceinline__ double lane_value(double v, int l)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
    return __hiloint2double(hi, lo);
}

// The largest of the lanes' values, none below 0 (a NaN counts as 0).
__device__ __forceinline__ double wave_max0(double v)
{
    v = v > 0.0 ? v : 0.0;
    for (int off = 32; off > 0; off >>= 1) {
        const double o = __shfl_xor(v, off, 64);
        v = o > v ? o : v;
    }
    return v;
}

// Acceptance of the evaluated trial and the damping update, by wave 0.  The
// relative step of parameter i is lane i's.
__device__ __forceinline__ void lm_accept(const Params &p, WGShared &S)
{
    const int t = threadIdx.x, n = S.n;
    const int phase = S.phase;
    double Ft = S.Fe;
    if (!isfinite(Ft)) Ft = INFINITY;
    const double F_c = S.F_c, chi2e = S.chi2e;
    const bool better = Ft < F_c;
    const bool accept = phase == 0 || better;
    if (phase != 1) {
        if (t == 0) {
            S.finished = 0;
            S.accept = accept ? 1 : 0;
            if (phase == 0) {
                S.mu = p.lm_mu0;
                S.nu = 2.0;
                S.trials = 0;
                S.converged = 0;
                S.chi2_init = chi2e;
                S.phase = S.alt_pending ? 2 : 1;
            } else {
                // the proposal against the simple start: the lower objective is
                // the start of LM; the damping is untouched
                S.chose_prop = S.accept;
                if (accept) {
                    S.chi2_init = chi2e;
                    for (int i = 0; i < 4; ++i) S.th0[i] = S.th_e[i];
                }
                S.phase = 1;
            }
        }
    } else if (accept) {
        // the step relative to the trial's amplitude or width
        double v = 0.0;
        if (t < n) {
            const double tn = S.th_e[t], w = S.th_e[t | 3];
            const double sa = fabs(tn) > 1e-30 ? fabs(tn) : 1e-30;
            v = fabs(tn - S.th_c[t]) / ((t & 3) == 0 ? sa : w);
        }
        const double pred = S.pred;
        const double rho = pred > 0.0 ? (F_c - Ft) / pred : 1.0;
        const double tt = 2.0 * rho - 1.0;
        double f = 1.0 - tt * tt * tt;
        if (f < 1.0 / 3.0) f = 1.0 / 3.0;
        double mu = S.mu * f;
        if (mu < 1e-12) mu = 1e-12;
        const bool end = !__any(!(v < p.lm_tol) && v == v);
        if (t == 0) {
            S.accept = 1;
            S.mu = mu;
            S.nu = 2.0;
            S.finished = 0;
            if (end) { S.converged = 1; S.finished = 1; }
        }
    } else if (t == 0) {
        S.accept = 0;
        S.finished = 0;
        S.mu *= S.nu;
        S.nu *= 2.0;
        if (S.mu > 1e8) { S.converged = 1; S.finished = 1; }
    }
    // the evaluated point becomes the current one; its Gram matrix buffer
    // becomes the current buffer (no copy)
    if (accept) {
        if (t < n) { S.th_c[t] = S.th_e[t]; S.g_c[t] = S.ge[t]; }
        if (t == 0) {
            S.F_c = S.Fe; S.chi2_c = chi2e; S.npx_c = S.npx_e;
            S.hsel ^= 1;
        }
    }
    wave_lds_sync();
}

// h + mu d with the product rounded on its own (not fused).
__device__ __forceinline__ double damped(double h, double mu, double d)
{
#pragma clang fp contract(off)
    const double q = mu * d;
    return h + q;
}

// The damped solve for n = N <= 8 by wave 0: every lane holds the factor's
// lower triangle and does the same arithmetic (each Cholesky column scaled by
// one reciprocal square root), so that nothing crosses lanes on the way; the
// per-parameter steps around it (bounds, clipping, the store) are one lane per
// parameter.  The chain is a square root, a division and two multiply-adds per
// column, about 260 clocks.
template <int N>
__device__ __forceinline__ void lm_solve_small(int32_t lm_max_iter, WGShared &S, const double *Hc)
{
    const int t = threadIdx.x;            // lane of wave 0
    const int q = t < N ? t : 0;          // its parameter
    const double th = S.th_c[q], g = S.g_c[q], lo = S.lo[q], hi = S.hi[q];
    double h[N][N];
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int k = 0; k <= i; ++k) h[i][k] = Hc[i * N + k];
    double rhs[N], dd[N];
#pragma unroll
    for (int i = 0; i < N; ++i) rhs[i] = S.g_c[i];
    const bool fr = (th <= lo && g <= 0.0) || (th >= hi && g >= 0.0);
    const unsigned int frozen = (unsigned int)__ballot(fr && t < N);
    double mu = S.mu, nu = S.nu;
    int trials = S.trials, finished = S.finished, converged = S.converged;
    double dmax = 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i) dmax = h[i][i] > dmax ? h[i][i] : dmax;
    const double dmin = 1e-12 * dmax;
#pragma unroll
    for (int i = 0; i < N; ++i) dd[i] = h[i][i] < dmin ? dmin : h[i][i];
    if (frozen) {
        // a parameter held on its bound: an identity row and column
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const bool fi = (frozen >> i) & 1u;
            rhs[i] = fi ? 0.0 : rhs[i];
#pragma unroll
            for (int k = 0; k < i; ++k) h[i][k] = (fi || ((frozen >> k) & 1u)) ? 0.0 : h[i][k];
        }
    }
    while (!uniform(finished != 0)) {
        if (uniform(trials >= lm_max_iter)) { finished = 1; break; }
        trials++;
        double a[N][N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
#pragma unroll
            for (int k = 0; k < i; ++k) a[i][k] = h[i][k];
            const double v = fma(mu, dd[i], h[i][i]);
            a[i][i] = ((frozen >> i) & 1u) ? 1.0 : v;
        }
        bool ok = true;
        double rinv[N];                  // 1 / L_kk
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const double d = a[k][k];
            ok = ok && d > 0.0 && isfinite(d);
            const double r = 1.0 / sqrt(d);
            rinv[k] = r;
#pragma unroll
            for (int i = k + 1; i < N; ++i) a[i][k] *= r;
#pragma unroll
            for (int i = k + 1; i < N; ++i)
#pragma unroll
                for (int j = k + 1; j <= i; ++j) a[i][j] -= a[i][k] * a[j][k];
        }
        double x[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            double v = rhs[i];
#pragma unroll
            for (int j = 0; j < i; ++j) v -= a[i][j] * x[j];
            x[i] = v * rinv[i];
        }
#pragma unroll
        for (int i = N - 1; i >= 0; --i) {
            double v = x[i];
#pragma unroll
            for (int j = i + 1; j < N; ++j) v -= a[j][i] * x[j];
            x[i] = v * rinv[i];
        }
#pragma unroll
        for (int i = 0; i < N; ++i) ok = ok && isfinite(x[i]);
        if (uniform(ok)) {
            double xi = x[0];
#pragma unroll
            for (int k = 1; k < N; ++k) xi = q == k ? x[k] : xi;
            double v = th + xi;
            if (!(v >= lo)) v = lo;
            if (v > hi) v = hi;
            if (t < N) S.th_e[t] = v;
            double pred = 0.0;
#pragma unroll
            for (int i = 0; i < N; ++i) pred += x[i] * (rhs[i] + mu * dd[i] * x[i]);
            if (t == 0) S.pred = pred;
            break;
        }
        // not positive definite: treated as a rejected trial
        mu *= nu;
        nu *= 2.0;
        if (mu > 1e8) { converged = 1; finished = 1; }
    }
    if (t == 0) {
        S.mu = mu;
        S.nu = nu;
        S.trials = trials;
        S.finished = finished;
        S.converged = converged;
    }
}

// Cholesky factor of A and the solution of L y = b (n < 64: b takes the place of
// row 0, which has no entry below the diagonal; n = 64: without b), in the
// textbook arithmetic: L_kk = sqrt(d_k), L_ik = A_ik / L_kk,
// A_ij -= L_ik L_jk.  Lane i of wave w keeps the entries of row i in the
// columns w, w + 4, ... w + 4 (V - 1) in registers.  The owner of column k scales it (one
// square root, one division per lane) and writes it to row k of Lt; after one
// barrier every wave updates its own columns from there, uniform reads of L_jk
// and one of L_ik.  Entries above the diagonal and of finished columns are
// carried along unread, so a column has no conditions.  Lt[k][i] = L_ik for
// i > k, y_k at i = 0; the L_kk go to S.ldiag.  S.pd is cleared when A is not
// positive definite.
constexpr int kLtStride = kMaxN + 2;
template <int V>
__device__ __forceinline__ void chol_factor(WGShared &S, const double *Hc, int n, double mu, double *Lt)
{
    static_assert(kT == 256 && kMaxN <= 64, "four waves, one lane per row");
    static_assert(sizeof(double) * (size_t)kMaxN * kLtStride <= kTileBytes, "L in the tile buffer");
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    double a[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int j = wave + 4 * v;
        double x = 0.0;
        if (j < n) {
            if (lane == 0) x = n == kMaxN ? 0.0 : S.rhs[j];
            else if (lane == j) x = S.frozen[j] ? 1.0 : damped(Hc[j * n + j], mu, S.dd[j]);
            else if (lane < n && !(S.frozen[lane] || S.frozen[j])) x = Hc[j * n + lane];   // symmetric
        }
        a[v] = x;
    }
    // the first pivot has no lane of its own
    const double d0 = S.frozen[0] ? 1.0 : damped(Hc[0], mu, S.dd[0]);
#pragma unroll
    for (int vk = 0; vk < V; ++vk) {
        if (4 * vk >= n) break;
#pragma unroll 1
        for (int w = 0; w < 4; ++w) {
            const int k = 4 * vk + w;            // n is a multiple of 4
            double *Lk = Lt + k * kLtStride;
            if (wave == w) {
                const double d = k == 0 ? d0 : lane_value(a[vk], k);
                const double l = sqrt(d);
                Lk[lane] = a[vk] / l;
                if (lane == 0) {
                    S.ldiag[k] = l;
                    if (!(d > 0.0 && isfinite(d))) S.pd = 0;
                }
            }
            __syncthreads();
            const double li = Lk[lane];
            double lj[V];
#pragma unroll
            for (int v = vk; v < V; ++v) lj[v] = Lk[wave + 4 * v];
#pragma unroll
            for (int v = vk; v < V; ++v) a[v] -= li * lj[v];
        }
    }
}

// The damped solve for n > 8: the factorisation above, then L^T x = y by wave
// 0, one lane per row.
__device__ __forceinline__ bool chol_solve(WGShared &S, const double *Hc, int n, double mu, double *Lt)
{
    const int t = threadIdx.x;
    if (t == 0) S.pd = 1;
    if (n <= 16) chol_factor<4>(S, Hc, n, mu, Lt);
    else if (n <= 32) chol_factor<8>(S, Hc, n, mu, Lt);
    else chol_factor<kMaxN / 4>(S, Hc, n, mu, Lt);
    __syncthreads();
    if (t < 64) {
        const double ld = t < n ? S.ldiag[t] : 1.0;
        const double *Lj = Lt + (t < n ? t : 0) * kLtStride;
        double x;
        if (n < kMaxN) {
            x = t < n ? Lj[0] : 0.0;             // y_t
        } else {
            // 64 rows leave no lane for the right-hand side: L y = b apart
            x = S.rhs[t];
            for (int i = 0; i < n; ++i) {
                const double yi = lane_value(x, i) / lane_value(ld, i);
                const double l = Lt[i * kLtStride + t];
                if (t == i) x = yi;
                else if (t > i) x -= l * yi;
            }
        }
        // lane j keeps x_j; L_ij of the next row is loaded ahead of its use
        double l = Lj[n - 1];
        for (int i = n - 1; i >= 0; --i) {
            const double ln = Lj[i > 0 ? i - 1 : 0];
            const double xi = lane_value(x, i) / lane_value(ld, i);
            const double xn = x - l * xi;
            x = t == i ? xi : t < i ? xn : x;
            l = ln;
        }
        if (t < n) S.delta[t] = x;
        const bool good = __all(t >= n || isfinite(x));
        if (t == 0) S.ok = good && S.pd ? 1 : 0;
    }
    __syncthreads();
    return S.ok != 0;
}

// The LM decision on the evaluated trial by wave 0: acceptance, then the next
// point (S.th_e) or the end (S.finished).  S.solve: the solve is left to the
// whole work-group (n > 8).
__device__ __forceinline__ void lm_decide(const Params &p, WGShared &S, const double *H2)
{
    const int t = threadIdx.x, n = S.n;
    const bool simple = uniform(S.phase == 0 && S.alt_pending);
    lm_accept(p, S);
    if (simple) {
        // the simple start is evaluated; the next evaluation is the proposal
        // start with the other members unchanged
        if (t < 4) {
            double v = S.alt[t];
            if (!(v >= S.lo[t])) v = S.lo[t];
            if (v > S.hi[t]) v = S.hi[t];
            S.th_e[t] = v;
        }
        if (t == 0) S.alt_pending = 0;
    } else if (n <= 8) {
        const double *Hc = H2 + S.hsel * (kMaxN * kMaxN);
        if (n == 4) lm_solve_small<4>(p.lm_max_iter, S, Hc);
        else lm_solve_small<8>(p.lm_max_iter, S, Hc);
    }
    if (t == 0) S.solve = !simple && n > 8 ? 1 : 0;
    wave_lds_sync();
}

// The next point for n > 8, by the whole work-group after lm_decide.  Thread 0
// writes S.finished only before the barrier at the loop's top (it wrote it last
// itself), or behind the solve's barriers, so that every wave takes the same
// way after it.
__device__ __forceinline__ void lm_solve_large(const Params &p, WGShared &S, const double *H2, double *Lt)
{
    const int t = threadIdx.x, n = __builtin_amdgcn_readfirstlane(S.n);
    const double *Hc = H2 + S.hsel * (kMaxN * kMaxN);
    for (;;) {
        if (t == 0 && !S.finished) {
            if (S.trials >= p.lm_max_iter) S.finished = 1;
            else S.trials++;
        }
        __syncthreads();
        if (S.finished) break;
        if (t < 64) {
            const double d = t < n ? Hc[t * n + t] : 0.0;
            const double dmax = wave_max0(d);
            if (t < n) {
                S.dd[t] = d < 1e-12 * dmax ? 1e-12 * dmax : d;
                const double th = S.th_c[t], g = S.g_c[t];
                S.frozen[t] = ((th <= S.lo[t] && g <= 0.0) || (th >= S.hi[t] && g >= 0.0)) ? 1 : 0;
                S.rhs[t] = S.frozen[t] ? 0.0 : g;
            }
        }
        __syncthreads();
        const double mu = S.mu;
        const bool ok = chol_solve(S, Hc, n, mu, Lt);
        if (ok) {
            if (t < 64) {
                const double x = t < n ? S.delta[t] : 0.0;
                const double u = t < n ? S.rhs[t] + mu * S.dd[t] * x : 0.0;
                if (t < n) {
                    double v = S.th_c[t] + x;
                    if (!(v >= S.lo[t])) v = S.lo[t];
                    if (v > S.hi[t]) v = S.hi[t];
                    S.th_e[t] = v;
                }
                double pred = 0.0;
                for (int i = 0; i < n; ++i) pred += lane_value(x, i) * lane_value(u, i);
                if (t == 0) S.pred = pred;
                wave_lds_sync();
            }
            break;
        }
        if (t == 0) {       // not positive definite: treated as a rejected trial
            S.mu *= S.nu;
            S.nu *= 2.0;
            if (S.mu > 1e8) { S.converged = 1; S.finished = 1; }
        }
    }
}

// Commit and the residual-update plan, work-group 0.  The loop gain (Sect. 3)
// scales every change the fit makes to the model image: the new component
// joins with gain times its fitted amplitude at its fitted centre and width,
// and each old member moves the fraction gain of the way from its stored
// parameters to its refit.  A new component whose fitted amplitude is zero
// (held on its sign bound: the old members explain the peak) models no
// emission and is not added to the list.
__device__ __forceinline__ void commit(const Params &p, WGShared &S)
{
    DevState *st = p.st;
    const int t = threadIdx.x;
    const int m = S.m;
    if (t == 0) {
        const int64_t L = st->L, k = st->k;
        const int trials = S.trials_total + S.trials;
        st->n_active = m;
        st->lm_iters = trials;
        st->converged = S.converged;
        st->used_fallback = S.used_fallback;
        st->chi2_init = S.chi2_init;
        st->chi2_final = S.chi2_c;
        st->fit_px = S.npx_c;
        st->sum_trials += (unsigned long long)trials;
        st->not_converged += S.converged ? 0ull : 1ull;
        st->fallbacks += (unsigned long long)S.used_fallback;
        st->init_source = S.use_prop ? st->have_proposal : (S.use_smooth ? 3 : 0);
        // a fallback follows only a fit that started from the proposal
        st->start_prop = (S.chose_prop || S.used_fallback) ? 1 : 0;
        for (int i = 0; i < 4; ++i)
            st->init[i] = S.use_prop ? st->proposal[i] : (S.use_smooth ? S.t0[i] : 0.0);
        st->have_proposal = 0;
        if (p.smooth) {
            // Sect. 3's switch: the simple values next time when the new
            // component's fitted area fell below 5 % of its start's area
            const double s0 = S.t0[3], s1 = S.th_c[3], wb = st->omega_b;
            const bool shrank = p.sm.switch_area
                                    ? __dsub_rn(__dmul_rn(s1, s1), __dmul_rn(wb, wb)) <
                                          __dmul_rn(0.05, __dsub_rn(__dmul_rn(s0, s0), __dmul_rn(wb, wb)))
                                    : __dmul_rn(s1, s1) < __dmul_rn(0.05, __dmul_rn(s0, s0));
            st->smooth_now = shrank ? 0 : 1;
            st->smooth_ready = 0;
            st->sum_smoothed += S.use_smooth ? 1ull : 0ull;
        }
        if (p.rec_cap > 0 && st->rec_n < p.rec_cap) {
            // the training pair of this iteration: the patch is already in place
            const int64_t n = st->rec_n;
            const int64_t r0 = S.idx / p.W, c0 = S.idx % p.W;
            float *tg = p.rec_target + 4 * n;
            tg[0] = (float)(S.th_c[0] / S.peak);
            tg[1] = (float)log(S.th_c[3] / st->omega_b);
            tg[2] = (float)(S.th_c[1] - (double)c0);
            tg[3] = (float)(S.th_c[2] - (double)r0);
            p.rec_flag[n] = S.converged | (S.used_fallback << 1) | (st->init_source << 2);
            st->rec_n = n + 1;
        }
        int nr = 0;
        int32_t bb[4] = {INT32_MAX, -1, INT32_MAX, -1};
        auto add_rect = [&](double a, double x, double y, double s, float sign) {
            Rect &R = st->rects[nr++];
            int32_t w[4];
            make_window(x, y, halfwidth(s, p.window_sigmas), p.H, p.W, w);
            R.r0 = w[0]; R.r1 = w[1]; R.c0 = w[2]; R.c1 = w[3];
            R.a = a; R.x = x; R.y = y; R.s = s; R.sign = sign;
            bb[0] = w[0] < bb[0] ? w[0] : bb[0];
            bb[1] = w[1] > bb[1] ? w[1] : bb[1];
            bb[2] = w[2] < bb[2] ? w[2] : bb[2];
            bb[3] = w[3] > bb[3] ? w[3] : bb[3];
        };
        for (int j = 1; j < m; ++j) {
            const int64_t cj = S.members[j];
            const double *to = S.th_old + 4 * j, *tn = S.th_c + 4 * j;
            double tc[4];
            // t + gain (t* - t), each operation rounded on its own
            for (int q = 0; q < 4; ++q)
                tc[q] = __dadd_rn(to[q], __dmul_rn(p.gain, __dsub_rn(tn[q], to[q])));
            add_rect(to[0], to[1], to[2], to[3], +1.0f);
            add_rect(tc[0], tc[1], tc[2], tc[3], -1.0f);
            p.ca[cj] = tc[0]; p.cx[cj] = tc[1]; p.cy[cj] = tc[2]; p.cs[cj] = tc[3];
            p.c_updated[cj] = k;
        }
        const bool added = S.th_c[0] != 0.0;
        if (added) {
            const double anew = __dmul_rn(p.gain, S.th_c[0]);
            add_rect(anew, S.th_c[1], S.th_c[2], S.th_c[3], -1.0f);
            p.ca[L] = anew; p.cx[L] = S.th_c[1]; p.cy[L] = S.th_c[2]; p.cs[L] = S.th_c[3];
            p.c_added[L] = k;
            p.c_updated[L] = k;
        }
        st->added = added ? 1 : 0;
        st->not_added += added ? 0ull : 1ull;
        st->n_rects = nr;
        if (nr == 0) { bb[0] = 0; bb[1] = -1; bb[2] = 0; bb[3] = -1; }
        st->bb[0] = bb[0]; st->bb[1] = bb[1]; st->bb[2] = bb[2]; st->bb[3] = bb[3];
        st->L = added ? L + 1 : L;
        st->k = k + 1;
        st->fit_ready = 1;
    }
    if (t < m) st->members[t] = S.members[t];
    if (t < 4 * m) {
        st->theta0[t] = S.th0[t];
        st->theta[t] = S.th_c[t];
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------

// Evaluate this work-group's tiles of the trial prepared in S; its partial row
// is left in LDS (the returned pointer), complete for every thread.
__device__ __forceinline__ double *evaluate_row(const Params &p, WGShared &S, float *tile,
                                                int64_t tile0, int64_t stride)
{
    double *row = reinterpret_cast<double *>(reinterpret_cast<unsigned char *>(tile) + kRowOffset);
    if (S.m == 1) evaluate_tiles_reg<1>(p, S, tile0, stride, row, tile);
    else if (S.m == 2) evaluate_tiles_reg<2>(p, S, tile0, stride, row, tile);
    else if (S.m <= 3) evaluate_tiles_mfma<1>(p, S, tile, tile0, stride, row);
    else if (S.m <= 7) evaluate_tiles_mfma<2>(p, S, tile, tile0, stride, row);
    else if (S.m <= 11) evaluate_tiles_mfma<3>(p, S, tile, tile0, stride, row);
    else if (S.m <= 15) evaluate_tiles_mfma<4>(p, S, tile, tile0, stride, row);
    else evaluate_tiles(p, S, tile, tile0, stride, row);
    return row;
}

// Work-groups of a shared trial: at least min_tiles tiles each.
__device__ inline int eval_groups(int64_t ntiles, int nwg, int min_tiles)
{
    const int64_t want = (ntiles + min_tiles - 1) / min_tiles;
    return (int)(want < nwg ? want : nwg);
}

// Up to this many parameters the leader sums all the rows of a shared trial
// itself (sum_groups): a row is at most 48 values, and the second level's
// hop between work-groups costs more than the reads.  Above, the last arrival
// of a group sums the group's rows.
constexpr int kFlatMaxN = 8;
constexpr int kFlatMaxV = (kFlatMaxN + 1) * (kFlatMaxN + 2) / 2 + 3;
static_assert(sizeof(double) * kFlatMaxV * kMaxGroups <= kRowOffset,
              "group sums of the flat reduction in the tile buffer, before the leader's row");

// One work-group's arrival after its tiles of a shared trial: the row goes to
// the partials, then the group's counter moves.  With the flat sums that is
// all (the leader keeps its own row in LDS and does not arrive); otherwise the
// last evaluating work-group of the group sums the group's rows in order into
// the group row, clears the counter and arrives at the top counter.
__device__ __forceinline__ void arrive(const Params &p, FitGlobal *G, WGShared &S, const double *row,
                                       int wg, int nwg, int geff)
{
    const int t = threadIdx.x, n = S.n;
    const int nv = (n + 1) * (n + 2) / 2 + 3;
    const int gs = p.group, grp = wg / gs;
    double *dst = p.partials + (int64_t)wg * kPartStride;
    if (n <= kFlatMaxN) {
        static_assert(kFlatMaxV <= 64, "one wave stores the row");
        if (t < 64) {
            if (t < nv) st_shared(dst + t, row[t]);
            wave_stores_done();
            if (t == 0)
                __hip_atomic_fetch_add(&G->arrive_g[grp].n, 1u, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
        }
        return;
    }
    for (int o = t; o < nv; o += kT) st_shared(dst + o, row[o]);
    wave_stores_done();
    __syncthreads();
    const int r0 = grp * gs, r1 = r0 + gs < geff ? r0 + gs : geff;
    if (t == 0) {
        const unsigned prev = __hip_atomic_fetch_add(&G->arrive_g[grp].n, 1u, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
        S.last = (prev == (unsigned)(r1 - r0) - 1u) ? 1 : 0;
        if (S.last) st_shared(&G->arrive_g[grp].n, 0u);
    }
    __syncthreads();
    if (!S.last) return;
    if (geff > gs) {
        double *sum = p.partials + (int64_t)(nwg + grp) * kPartStride;
        for (int o = t; o < nv; o += kT) st_shared(sum + o, sum_column(p, r0, r1, o));
    }
    wave_stores_done();
    __syncthreads();
    if (t == 0) __hip_atomic_fetch_add(&G->top.n, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Arrival after a command that changed or read plain data (the residual).
__device__ __forceinline__ void arrive_released(FitGlobal *G, int wg, int gs)
{
    wave_stores_done();
    __syncthreads();
    if (threadIdx.x == 0)
        __hip_atomic_fetch_add(&G->arrive_g[wg / gs].n, 1u, __ATOMIC_RELEASE,
                               __HIP_MEMORY_SCOPE_AGENT);
}

// The leader's wait for the arrivals of work-groups 1 .. T-1 after a command on
// plain data, and the acquire of what they wrote; false when it ran out.
__device__ __forceinline__ bool team_wait(FitGlobal *G, WGShared &S, int T, int gs,
                                          unsigned long long limit)
{
    const bool ok = wait_groups(G, S, T, gs, limit);
    if (threadIdx.x == 0) acquire_fence();
    __syncthreads();
    return ok;
}

// Work-group `wg`'s share of the peak search (Sect. 2 step 1): of the whole
// residual, or of the listed tiles.
__device__ __forceinline__ void peak_share(const Params &p, int wg, int nwg)
{
    if (p.st->pk.tiles_x > 0) peak_tiles_scan(p, (unsigned)wg, (unsigned)nwg);
    else peak_scan(p.R, p.H * p.W, (uint32_t)wg, (uint32_t)nwg, p.st->peak_keys);
}

// The evaluated rows 0 .. geff-1 (row 0 the leader's own, in LDS) of NV values
// summed per group of gs work-groups, in row order, into `scratch` (NV x groups
// doubles, LDS); sixteen loads in flight per thread.
template <int NV>
__device__ __forceinline__ void sum_groups(const Params &p, int geff, int gs, const double *row,
                                           double *scratch)
{
    const int ng = (geff + gs - 1) / gs;
    for (int e = threadIdx.x; e < NV * ng; e += kT) {
        const int g = e / NV, o = e - g * NV;
        const int r0 = g * gs, r1 = r0 + gs < geff ? r0 + gs : geff;
        double v = 0.0;
        for (int w = r0; w < r1; w += 16) {
            // rows past the group's last are read as the last and not added
            const double *src = p.partials + o;
            double a[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int r = w + u < r1 ? w + u : r1 - 1;
                a[u] = ld_shared(src + (int64_t)r * kPartStride);
            }
            a[0] = w == 0 ? row[o] : a[0];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const double s = v + a[u];
                v = w + u < r1 ? s : v;
            }
        }
        scratch[e] = v;
    }
    __syncthreads();
}

// A flat trial's sums by wave 0, lane o's value o: the groups in order (the
// association of the two-level sums), or the leader's own row (ng = 0).
// (i, k) is the lane's Gram entry, from out_pair.
template <int NV>
__device__ __forceinline__ void final_sums(WGShared &S, const double *row, const double *scratch,
                                           int ng, int i, int k, double *He)
{
    const int o = threadIdx.x;
    if (o < NV) {
        double v;
        if (ng == 0) {
            v = row[o];
        } else {
            v = scratch[o];
            for (int g = 1; g < ng; g += 8) {
                double a[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) a[u] = scratch[(g + u < ng ? g + u : 0) * NV + o];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const double s = v + a[u];
                    v = g + u < ng ? s : v;
                }
            }
        }
        const int n = S.n;
        if (o == NV - 3) S.Fe = v;
        else if (o == NV - 2) S.chi2e = v;
        else if (o == NV - 1) S.npx_e = (int64_t)v;
        else if (k < n) { He[i * n + k] = v; He[k * n + i] = v; }
        else if (i < n) S.ge[i] = v;
    }
    wave_lds_sync();
}

// The peak and the stop test (Sect. 2 steps 1 and 4) of one fit, thread 0 of
// the leading work-group: sets S.idx, S.peak, S.stop and the fit's
// bookkeeping.  `abort` reports a wait that ran out before it.
__device__ __forceinline__ void fit_begin(const Params &p, WGShared &S, bool abort)
{
    DevState *st = p.st;
    S.prof[kPFits] += 1ull;
    st->fit_ready = 0;
    const unsigned long long key = S.key;
    int64_t idx = st->forced_idx >= 0
                      ? st->forced_idx
                      : (int64_t)(0xFFFFFFFFu - (uint32_t)(key & 0xFFFFFFFFull));
    const bool bad_idx = (st->forced_idx < 0 && key == 0ull) || idx < 0 || idx >= p.H * p.W;
    st->forced_idx = -1;
    S.stop = 0;
    if (abort) S.stop = ASP_ERR_DEVICE;
    else if (bad_idx) S.stop = ASP_ERR_STATE;
    if (bad_idx) idx = 0;
    const float v = p.R[idx];
    if (S.stop == 0) {
        if (fabs((double)v) < p.threshold) S.stop = ASP_STOP_THRESHOLD;
        else if (st->k >= p.max_iter) S.stop = ASP_STOP_MAXITER;
        else if (st->L >= p.cap) S.stop = ASP_ERR_CAPACITY;
    }
    st->idx = idx;
    st->peak = v;
    S.idx = idx;
    S.peak = (double)v;
    S.pass = 0;
    S.trials_total = 0;
    S.used_fallback = 0;
    S.use_prop = (p.use_proposal && st->have_proposal) ? 1 : 0;
    S.use_smooth = (p.smooth && !S.use_prop && st->smooth_now && st->smooth_ready) ? 1 : 0;
    if (S.stop) st->stop = S.stop;
}

// The trial at S.th_e, by wave 0 of the leader: member constants and windows,
// and whether it is shared: a trial larger than p.solo_tiles tiles is published
// (with the field, for a batch team).  S.geff: its work-groups, 0 for the
// leader alone.
__device__ __forceinline__ void next_trial(const Params &p, FitGlobal *G, WGShared &S, int nwg,
                                           int field)
{
    const bool first = uniform(S.fit_no == 0u);
    prepare_windows(p, S);
    const int64_t ntiles = (S.pref[S.m] + kT - 1) / kT;
    int geff = 0;
    if (ntiles > p.solo_tiles) {
        geff = eval_groups(ntiles, nwg, p.min_tiles);
        // a batch's leader may have changed R since its last message
        const bool release = uniform(S.epoch != S.epoch_have);
        post(G, S, kCmdEval, geff, field, release);
        if (threadIdx.x == 0) S.epoch_have = S.epoch;
    }
    if (threadIdx.x == 0) S.geff = geff;
    // the message is on its way
    if (first) prepare_old(p, S);
    prepare_members(S);
    lap(S, kPPrepare);
}

// The evaluation of the trial next_trial prepared and its sums: F, chi2, the
// pixel count and [J r]^T [J r] into S.Fe, S.chi2e, S.npx_e, S.ge and the Gram
// buffer H2 + (1 - S.hsel) n^2, complete for wave 0.  Returns false when a wait
// ran out; the context is then marked with ASP_ERR_DEVICE.
__device__ __forceinline__ bool trial_sums(const Params &p, FitGlobal *G, WGShared &S, float *tile,
                                           double *H2, int nwg)
{
    const int t = threadIdx.x;
    const int geff = S.geff, n = S.n;
    const int ng = (geff + p.group - 1) / p.group;
    double *He = H2 + (1 - S.hsel) * (kMaxN * kMaxN);   // the trial's buffer
    double *scratch = reinterpret_cast<double *>(tile);
    const double *row = evaluate_row(p, S, tile, 0, geff ? geff : 1);
    lap(S, kPEval);
    bool ok = true;
    int i = 0, k = 0;
    if (n <= kFlatMaxN) {
        if (t < (n + 1) * (n + 2) / 2) out_pair(t, n, i, k);
        if (geff) {
            ok = wait_groups(G, S, geff, p.group, p.spin_ticks);
            lap(S, kPWait);
        }
    } else if (geff) {
        arrive(p, G, S, row, 0, nwg, geff);
        lap(S, kPArrive);
        if (t == 0) {
            S.abort = spin_until(&G->top.n, (unsigned)ng, p.spin_ticks) ? 0 : 1;
            st_shared(&G->top.n, 0u);
        }
        __syncthreads();
        lap(S, kPWait);
        ok = S.abort == 0;
    }
    if (!ok) {
        if (t == 0) p.st->stop = ASP_ERR_DEVICE;
        __syncthreads();
        return false;
    }
    if (n == 4) {
        if (geff) sum_groups<18>(p, geff, p.group, row, scratch);
        if (t < 64) final_sums<18>(S, row, scratch, ng, i, k, He);
    } else if (n == 8) {
        if (geff) sum_groups<48>(p, geff, p.group, row, scratch);
        if (t < 64) final_sums<48>(S, row, scratch, ng, i, k, He);
    } else {
        const int nv = (n + 1) * (n + 2) / 2 + 3;
        const int w0 = ng > 1 ? nwg : 0, w1 = ng > 1 ? nwg + ng : geff;
        for (int o = t; o < nv; o += kT)
            put_sum(S, He, n, o, geff ? sum_column(p, w0, w1, o) : row[o]);
        __syncthreads();
    }
    lap(S, kPReduce);
    if (t == 0 && geff == 0) {
        S.prof[kPSoloTrials] += 1ull;
        S.prof[kPSoloPx] += (unsigned long long)S.npx_e;
    }
    return true;
}

// Start values, active set, the LM trials and the commit of one fit, by the
// leading work-group (share 0 of nwg).  Returns false when a wait ran out; the
// context is then marked with ASP_ERR_DEVICE.
__device__ __forceinline__ bool fit_trials(const Params &p, FitGlobal *G, WGShared &S, float *tile,
                                           double *H2, int nwg, int field)
{
    DevState *st = p.st;
    const int t = threadIdx.x;
    mark(S);
    if (t == 0) S.tfit = S.tmark;
    for (;;) {
        setup_fit(p, S, S.use_prop != 0 && S.pass == 0);
        lap(S, kPSetup);
        if (t < 64) next_trial(p, G, S, nwg, field);
        __syncthreads();
        for (;;) {
            if (!trial_sums(p, G, S, tile, H2, nwg)) return false;
            if (t < 64) {
                if (t == 0) {
                    const unsigned long long npx = (unsigned long long)S.npx_e;
                    S.eval_px += npx;
                    S.gram_flops += npx * (unsigned long long)((S.n + 1) * (S.n + 2));
                    S.prof[kPTrials] += 1ull;
                    S.prof[kPEvalPx] += npx;
                }
                lm_decide(p, S, H2);
                if (S.n <= kFlatMaxN || !uniform(S.solve != 0)) {
                    lap(S, kPLmStep);
                    if (!uniform(S.finished != 0)) next_trial(p, G, S, nwg, field);
                }
            }
            __syncthreads();
            if (S.solve) {
                lm_solve_large(p, S, H2, reinterpret_cast<double *>(tile));
                if (t < 64) {
                    lap(S, kPLmStep);
                    if (!uniform(S.finished != 0)) next_trial(p, G, S, nwg, field);
                }
                __syncthreads();
            }
            if (S.finished) break;
        }
        if (S.use_prop && S.chose_prop && S.pass == 0 && (!S.converged || S.th_c[0] == 0.0)) {
            // LM started from the proposal and did not converge, or converged
            // to a new component of zero amplitude (which can leave the model
            // unchanged, so that the same peak and proposal come back): the
            // simple values instead
            __syncthreads();
            if (t == 0) {
                S.trials_total += S.trials;
                S.used_fallback = 1;
                S.pass = 1;
            }
            __syncthreads();
            continue;
        }
        break;
    }
    mark(S);
    commit(p, S);
    lap(S, kPCommit);
    if (t == 0) {
        const int m = S.m;
        st->fits_m[m] += 1ull;
        st->trials_m[m] += (unsigned long long)(S.trials_total + S.trials);
        st->ticks_m[m] += now_ticks() - S.tfit;
    }
    flush_counts(p, S);
    return true;
}

__global__ __launch_bounds__(kT) void k_fit(Params p)
{
    extern __shared__ __align__(16) unsigned char lds[];
    float *tile = reinterpret_cast<float *>(lds);
    double *H2 = reinterpret_cast<double *>(lds + kTileBytes);   // two Gram buffers
    __shared__ WGShared S;
    FitGlobal *G = p.fg;
    DevState *st = p.st;
    const int t = threadIdx.x;
    const int wg = blockIdx.x, nwg = gridDim.x;

    // Nothing writes the stop flag (or the evaluation request) before every
    // work-group has checked in, so all of them agree here.
    if (st->stop && st->diag_m == 0) return;

    // Check in: every work-group reads the last message's number before
    // work-group 0 may publish.
    if (t == 0) {
        mail_begin(G, S);
        if (wg != 0) {
            // the number has been read
            wave_stores_done();
            __hip_atomic_fetch_add(&G->top.n, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
    mark(S);

    if (wg != 0) {
        // Workers: evaluate the shared trials work-group 0 publishes.
        // The residual does not change before the update at the end of an
        // iteration and everything else that crosses is read with atomic loads,
        // so the workers need no acquire fence for a trial: their L2 keeps the
        // residual's lines from trial to trial.
        for (;;) {
            if (t < 64) {
                wait_mail(G, S, wg, p.spin_ticks);
                if (uniform(S.abort == 0 && S.cmd == kCmdEval && wg < S.geff)) {
                    if (uniform(S.fresh != 0)) prepare_old(p, S);
                    prepare_windows(p, S);
                    prepare_members(S);
                }
            }
            __syncthreads();
            if (S.abort) {
                if (t == 0) st->stop = ASP_ERR_DEVICE;
                return;
            }
            if (S.cmd == kCmdUpdate || S.cmd == kCmdPeak) {
                // the plan was written by work-group 0, and the residual by
                // every work-group, with plain stores: acquire before reading
                const bool peak = S.cmd == kCmdPeak, last = S.fld != 0;
                if (t == 0) acquire_fence();
                __syncthreads();
                if (peak) peak_share(p, wg, nwg);
                else update_tiles(p, wg, nwg, tile);
                if (last) return;
                arrive_released(G, wg, p.group);
                __syncthreads();
                continue;
            }
            if (S.cmd != kCmdEval) return;
            const int geff = S.geff;
            if (wg < geff) {
                const double *row = evaluate_row(p, S, tile, wg, geff);
                arrive(p, G, S, row, wg, nwg, geff);
            }
            __syncthreads();               // S is rewritten by the next message
        }
    }

    // Work-group 0 drives the fit.
    if (t == 0) {
        S.abort = spin_until(&G->top.n, (unsigned)nwg - 1u, p.spin_ticks) ? 0 : 1;
        st_shared(&G->top.n, 0u);
        lap(S, kPCheckin);
        S.tlaunch = S.tmark;
    }
    __syncthreads();
    if (st->diag_m > 0) {
        // one evaluation of a given trial (asp_eval_trial): no peak, no LM
        // step, no commit
        if (t == 0) {
            S.m = st->diag_m;
            S.n = 4 * S.m;
            S.hsel = 0;
        }
        __syncthreads();
        if (t < S.n) {
            S.th_e[t] = st->diag_theta[t];
            S.th_old[t] = st->diag_stored[t];
        }
        __syncthreads();
        bool ok = !S.abort;
        if (t < 64 && ok) next_trial(p, G, S, nwg, 0);
        __syncthreads();
        ok = ok && trial_sums(p, G, S, tile, H2, nwg);
        __syncthreads();
        const int n = S.n;
        double *o = st->diag_out;
        if (ok) {
            const double *He = H2 + kMaxN * kMaxN;        // 1 - hsel
            for (int e = t; e < n * n; e += kT) o[e] = He[e];
            if (t < n) o[n * n + t] = S.ge[t];
            if (t == 0) {
                o[n * n + n] = S.Fe;
                o[n * n + n + 1] = S.chi2e;
                o[n * n + n + 2] = (double)S.npx_e;
            }
        }
        if (t == 0) {
            if (!ok) st->stop = ASP_ERR_DEVICE;
            st->diag_m = 0;
        }
        flush_counts(p, S);
        publish(G, S, kCmdExit);
        return;
    }
    for (int it = 1;; ++it) {
        if (p.iters > 0 && S.abort == 0) {
            publish(G, S, kCmdPeak, 0, true);
            peak_share(p, 0, nwg);
            wave_stores_done();
            team_wait(G, S, nwg, p.group, p.spin_ticks);
            if (st->pk.tiles_x > 0) peak_tiles_reduce(p);
        }
        collect_peak_key(st, true, &S.key);
        if (t == 0) {
            fit_begin(p, S, S.abort != 0);
            S.upd = S.more = 0;
        }
        __syncthreads();
        if (!S.stop) {
            const bool committed = fit_trials(p, G, S, tile, H2, nwg, 0);
            if (!committed) flush_counts(p, S);
            // with fuse_update every work-group takes its tiles of the update
            // (Sect. 2 step 3) after this publication; the end of the kernel,
            // or the wait for every work-group, is the barrier before the next
            // iteration reads R
            if (t == 0) {
                S.upd = committed && p.fuse_update ? 1 : 0;
                S.more = S.upd && it < p.iters && now_ticks() - S.tlaunch < p.spin_ticks / kLaunchShare ? 1 : 0;
            }
        } else {
            flush_counts(p, S);
        }
        __syncthreads();
        const bool upd = S.upd != 0, last = S.more == 0;
        publish(G, S, upd ? kCmdUpdate : kCmdExit, last ? 1 : 0, upd);
        if (upd) update_tiles(p, 0, nwg, tile);
        if (last) return;
        wave_stores_done();
        team_wait(G, S, nwg, p.group, p.spin_ticks);
        mark(S);
    }
}

// ===========================================================================
// Batched fields: one persistent launch for many independent fields.
//
// The work-groups form teams of T.  Work-groups are dealt to the 8 XCDs round
// robin, so a team is made of work-groups with equal blockIdx % 8: one XCD,
// one L2 for the team's field.  A team takes fields from a queue, largest
// first, and runs each field's minor cycle for up to n_iter iterations:
// rank 0 leads as work-group 0 of k_fit does and the others follow its
// commands -- a share of the peak search, a share of an LM trial, a share of
// the residual update, or exit.  A share of the search or of the update is
// acknowledged by every member before the next command, a trial only by the
// members with tiles of it: the others may find that the leader has moved on and
// never read that message.  What an unread message could have told of R or of
// the update's plan is in every message: the epoch, whose change makes a member
// acquire before it reads them again.  Every wait is bounded.
// ===========================================================================

// The field's parameters with the team's exchange buffers and the batch's
// tile thresholds (thread 0 writes, the work-group reads after the barrier).
__device__ __forceinline__ void load_field(const BatchArgs &b, int f, FitGlobal *G, double *parts,
                                           Params &P)
{
    __syncthreads();
    if (threadIdx.x == 0) {
        P = b.fields[f];
        P.fg = G;
        P.partials = parts;
        P.solo_tiles = b.team_size == 1 ? 0x7FFFFFFF : b.solo_tiles;
        P.min_tiles = b.min_tiles;
        P.group = kGroup;
    }
    __syncthreads();
}

__global__ __launch_bounds__(kT) void k_batch(BatchArgs b)
{
    extern __shared__ __align__(16) unsigned char lds[];
    float *tile = reinterpret_cast<float *>(lds);
    double *H2 = reinterpret_cast<double *>(lds + kTileBytes);   // two Gram buffers
    __shared__ WGShared S;
    __shared__ Params P;
    __shared__ int32_t cur_field;
    const int t = threadIdx.x;
    const int T = b.team_size;
    const int per_xcd = (int)gridDim.x / 8;
    const int xcd = (int)blockIdx.x % 8, slot = (int)blockIdx.x / 8;
    const int team = xcd * (per_xcd / T) + slot / T;
    const int rank = slot % T;
    FitGlobal *G = b.fg + team;
    double *parts = b.partials + (int64_t)team * (T + (T + kGroup - 1) / kGroup) * kPartStride;

    // check in: every follower reads the last message's number before the
    // leader publishes
    if (t == 0) {
        mail_begin(G, S);
        cur_field = -1;
        if (rank != 0) {
            wave_stores_done();
            __hip_atomic_fetch_add(&G->top.n, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();

    if (rank != 0) {
        for (;;) {
            if (t < 64) wait_mail(G, S, rank, b.spin_ticks, true);
            __syncthreads();
            if (S.abort) return;                     // the leader marks its field
            const int cmd = S.cmd;
            if (cmd == kCmdExit || S.fld < 0 || S.fld >= b.n_fields) return;
            if (S.epoch != S.epoch_have) {
                // R or the update's plan changed since this work-group's last
                // acquire (messages may have been skipped: the epoch tells)
                __syncthreads();
                if (t == 0) {
                    acquire_fence();
                    S.epoch_have = S.epoch;
                }
                __syncthreads();
            }
            if (S.fld != cur_field) {
                load_field(b, S.fld, G, parts, P);
                if (t == 0) cur_field = S.fld;
                __syncthreads();
            }
            if (cmd == kCmdPeak) {
                peak_scan(P.R, P.H * P.W, (uint32_t)rank, (uint32_t)T, P.st->peak_keys);
                arrive_released(G, rank, kGroup);
            } else if (cmd == kCmdUpdate) {
                update_tiles<1>(P, rank, T, tile);
                arrive_released(G, rank, kGroup);
            } else if (cmd == kCmdEval) {
                const int geff = S.geff;
                if (rank < geff) {
                    if (t < 64) {
                        if (uniform(S.fresh != 0)) prepare_old(P, S);
                        prepare_windows(P, S);
                        prepare_members(S);
                    }
                    __syncthreads();
                    const double *row = evaluate_row(P, S, tile, rank, geff);
                    arrive(P, G, S, row, rank, T, geff);
                }
            }
            __syncthreads();               // S is rewritten by the next message
        }
    }

    // the leader
    if (t == 0) {
        if (T > 1) S.abort = spin_until(&G->top.n, (unsigned)(T - 1), b.spin_ticks) ? 0 : 1;
        st_shared(&G->top.n, 0u);
    }
    __syncthreads();
    bool ok = S.abort == 0;
    while (ok) {
        if (t == 0) {
            const unsigned q = atomicAdd(b.queue, 1u);
            S.fld = q < (unsigned)b.n_fields ? b.order[q] : -1;
        }
        __syncthreads();
        if (S.fld < 0) break;
        load_field(b, S.fld, G, parts, P);
        if (t == 0) {
            cur_field = S.fld;
            S.epoch += 1u;             // another residual
            S.k_target = P.st->k + b.n_iter;
        }
        for (;;) {
            if (t == 0) {
                S.go = (P.st->stop == 0 && P.st->k < S.k_target) ? 1 : 0;
                // one heartbeat per iteration: the followers' waits restart
                __hip_atomic_fetch_add(&G->beat.n, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __syncthreads();
            if (!S.go) break;
            // the peak of |R| (Sect. 2 step 1)
            const int64_t npx = P.H * P.W;
            if (T == 1 || npx <= b.solo_peak_px) {
                peak_scan(P.R, npx, 0u, 1u, P.st->peak_keys);
            } else {
                publish(G, S, kCmdPeak, cur_field, true);
                if (t == 0) S.epoch_have = S.epoch;
                peak_scan(P.R, npx, 0u, (uint32_t)T, P.st->peak_keys);
                if (!team_wait(G, S, T, kGroup, b.spin_ticks)) { ok = false; break; }
            }
            __syncthreads();
            // the stop test and the fit (Sect. 2 step 4; Sect. 3)
            collect_peak_key(P.st, true, &S.key);
            if (t == 0) fit_begin(P, S, false);
            __syncthreads();
            if (S.stop) {
                flush_counts(P, S);                // the next field counts for itself
                break;
            }
            if (!fit_trials(P, G, S, tile, H2, T, cur_field)) {
                flush_counts(P, S);
                ok = false;
                break;
            }
            // the residual update (Sect. 2 step 3)
            if (t == 0) {
                const int32_t *bb = P.st->bb;
                S.upx = (int64_t)(bb[1] - bb[0] + 1) * (int64_t)(bb[3] - bb[2] + 1);
            }
            __syncthreads();
            if (T == 1 || S.upx <= b.solo_update_px) {
                update_tiles<1>(P, 0, 1, tile);
            } else {
                if (t == 0) S.epoch += 1u;     // the plan
                publish(G, S, kCmdUpdate, cur_field, true);
                update_tiles<1>(P, 0, T, tile);
                if (!team_wait(G, S, T, kGroup, b.spin_ticks)) { ok = false; break; }
            }
            wave_stores_done();                // for the release of a later message
            __syncthreads();
            if (t == 0) S.epoch += 1u;         // R
        }
    }
    if (!ok && t == 0 && cur_field >= 0) P.st->stop = ASP_ERR_DEVICE;
    __syncthreads();
    if (T > 1) publish(G, S, kCmdExit, 0, true);
}

__global__ void k_batch_reset(unsigned int *queue) { *queue = 0u; }

hipError_t fit_kernel_setup()
{
    hipError_t e = hipFuncSetAttribute((const void *)k_fit,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kFitLds);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute((const void *)k_batch, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)kFitLds);
}

// A kernel whose work-groups wait for each other must have all of them
// resident at once.  A private segment (scratch) breaks that guarantee: the
// waves of a dispatch can be held back until scratch is free.
static bool no_private_segment(const void *kernel)
{
    hipFuncAttributes a;
    if (hipFuncGetAttributes(&a, kernel) != hipSuccess) return false;
    return a.localSizeBytes == 0;
}

int batch_grid_size(int device)
{
    int cus = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess)
        return 0;
    if (!no_private_segment((const void *)k_batch)) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)k_batch, kT,
                                                     kFitLds) != hipSuccess || per_cu < 1)
        return 0;
    const int grid = (cus * per_cu / 8) * 8;      // whole XCD rows
    return grid <= cus * per_cu ? grid : 0;
}

hipError_t launch_batch(const BatchArgs &b, int grid, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch_reset, dim3(1), dim3(1), 0, s, b.queue);
    hipLaunchKernelGGL(k_batch, dim3(grid), dim3(kT), kFitLds, s, b);
    return hipGetLastError();
}

int fit_grid_size(int device)
{
    int cus = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess)
        return 0;
    if (!no_private_segment((const void *)k_fit)) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)k_fit, kT, kFitLds) !=
            hipSuccess || per_cu < 1)
        return 0;
    int g = cus * per_cu;
    if (g > kGroup * kMaxGroups) g = kGroup * kMaxGroups;
    return g;
}

hipError_t launch_fit(const Params &p, hipStream_t s)
{
    void *args[] = {(void *)&p};
    return hipLaunchCooperativeKernel((const void *)k_fit, dim3(p.fit_grid), dim3(kT), args,
                                      kFitLds, s);
}

}  // namespace asp
