// Propagation kernels of libcrp for gfx950 (CDNA4, wave64).
//
// One lane holds one candidate in registers (the candidate carries all of its
// propagation state, paper section 3).  Waves are persistent: idle lanes claim
// candidates from a device queue, every loop iteration performs exactly one
// Cash-Karp attempt for all busy lanes (so the expensive part -- six field
// gathers -- is executed by the whole wave together), and lanes whose
// attempt is accepted finish their cycle: continuous loss, the stochastic
// interaction clock (reset after each event, section 3), then the
// observer / trajectory / energy-floor checks after the cycle (Fig. 1).
// Finished records, neutral records, spawned secondaries and budget-parked
// candidates are appended with one atomic per wave (ballot + prefix count).
#include "crp_internal.hpp"
#include "crp_nf_device.hpp"

namespace crp {

enum { LIM_CTRL = 0, LIM_TRAJ = 1, LIM_INTER = 2, LIM_LOSS = 3, LIM_OBS = 4 };
// interaction channel chosen in a cycle: none due, a null event (no channel
// open at this energy), pion-like (neutral record), nucleon loss (secondary)
enum { CH_NONE = -1, CH_PI = 0, CH_N = 1, CH_NULL = 2 };

// A parked candidate whose cycle stopped just before its interaction (no
// slot for the product) carries -(1 + step-limit flag) as its optical depth:
// a stored optical depth is otherwise always positive (an interaction resets
// it to at least 2^-24, and without one it stayed above zero).
__device__ inline double event_due_marker(int flag) { return -1.0 - (double)flag; }
__device__ inline int event_due_flag(double tau) { return (int)(-tau) - 1; }
enum { ST_ACTIVE = 0, ST_OBSERVED = 1, ST_MAX_TRAJ = 2, ST_ENERGY_FLOOR = 3, ST_BOUNDARY = 4 };

struct Cand {
    double x[3], u[3], u0[3];
    double E, L, Lmax, hctrl, tau, E0;
    uint32_t id, lineage, m, nsteps, nrej;
    int A, Z;
};

__device__ inline void store_cand(const QueueSoA& q, int64_t i, const Cand& c)
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        q.x[a * q.cap + i] = c.x[a];
        q.u[a * q.cap + i] = c.u[a];
        q.u0[a * q.cap + i] = c.u0[a];
    }
    q.E[i] = c.E;
    q.L[i] = c.L;
    q.Lmax[i] = c.Lmax;
    q.hctrl[i] = c.hctrl;
    q.tau[i] = c.tau;
    q.E0[i] = c.E0;
    q.id[i] = c.id;
    q.lineage[i] = c.lineage;
    q.m[i] = c.m;
    q.nsteps[i] = c.nsteps;
    q.nrej[i] = c.nrej;
    q.A[i] = c.A;
    q.Z[i] = c.Z;
}

// Bookkeeping: block counters in LDS.  Each lane counts its candidate's steps,
// rejected attempts and forced steps of this run in registers (none can pass
// 2^32 before the candidate's own 32-bit counts do) and adds them when the
// candidate ends or is parked; rare events are added where they happen.
enum {
    WC_STEPS = 0, WC_ATTEMPTS, WC_REJECTS, WC_FORCED, WC_EVENTS, WC_NULL, WC_PI, WC_N,
    WC_FINISHED, WC_OBSERVED, WC_MAXTRAJ, WC_EFLOOR, WC_QDEFER, WC_NDEFER, WC_LANES, WC_BOUNDARY,
    WC_COUNT
};

// Destination of each block counter in the device counter block.
__device__ inline unsigned long long* count_dst(DevCounters* cnt, int i)
{
    switch (i) {
    case WC_STEPS: return &cnt->steps;
    case WC_ATTEMPTS: return &cnt->attempts;
    case WC_REJECTS: return &cnt->rejects;
    case WC_FORCED: return &cnt->forced;
    case WC_EVENTS: return &cnt->events;
    case WC_NULL: return &cnt->null_events;
    case WC_PI: return &cnt->inter_pi;
    case WC_N: return &cnt->inter_n;
    case WC_FINISHED: return &cnt->finished;
    case WC_OBSERVED: return &cnt->observed;
    case WC_MAXTRAJ: return &cnt->max_traj;
    case WC_EFLOOR: return &cnt->energy_floor;
    case WC_QDEFER: return &cnt->queue_deferred;
    case WC_NDEFER: return &cnt->neutral_deferred;
    case WC_LANES: return &cnt->lane_slots;
    default: return &cnt->boundary;
    }
}

__device__ inline void flush_counts(DevCounters* cnt, const unsigned long long* bc)
{
    const int i = (int)threadIdx.x;
    if (i < WC_COUNT && bc[i] != 0ull) {
        atomicAdd(count_dst(cnt, i), bc[i]);
        // every pion-like event emits one neutral secondary, every nucleon-loss
        // event one charged secondary
        if (i == WC_PI)
            atomicAdd(&cnt->neutral_sec, bc[i]);
        if (i == WC_N)
            atomicAdd(&cnt->charged_sec, bc[i]);
    }
}

// Claims up to `want` slots of the region written before the launch with one
// atomicAdd (overshoot past tail0 is harmless: that region does not grow).
__device__ inline void claim_initial(DevCounters* cnt, unsigned long long tail0, int want,
                                     unsigned long long& base, unsigned long long& take,
                                     bool& left)
{
    const unsigned long long b = atomicAdd(&cnt->head, (unsigned long long)want);
    base = b;
    take = 0;
    left = false;
    if (b < tail0) {
        take = tail0 - b < (unsigned long long)want ? tail0 - b : (unsigned long long)want;
        left = b + take < tail0;
    }
}

// True once every candidate of this run is finished or parked: then none is
// active, so no secondary can be appended any more.  The done counts are read
// (acquire) before the append cursor; all three only grow and done never
// exceeds the written slots, so equality means that at the last read every
// written slot was done.  Slots past the queue capacity are never written.
// `done` receives the finished + parked count that was read.
__device__ inline bool run_drained(DevCounters* cnt, unsigned long long fin0,
                                   unsigned long long cap, unsigned long long& done)
{
    const unsigned long long f =
        __hip_atomic_load(&cnt->fin_n, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long p =
        __hip_atomic_load(&cnt->park_n, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
    unsigned long long t = __hip_atomic_load(&cnt->tail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (t > cap)
        t = cap;
    done = (f - fin0) + p;
    return done == t;
}

// A wave with nothing to do sleeps in units of s_sleep 127 (~3.4 us), one
// unit more per idle iteration up to IDLE_BACKOFF (its polls of the queue
// must not load the memory system that busy waves use).  If IDLE_SLEEP_LIMIT
// units (about 28 s) pass with no candidate of the run finishing anywhere and
// the run not drained, it records an error and leaves.
constexpr uint32_t IDLE_BACKOFF = 16u;
constexpr uint32_t IDLE_SLEEP_LIMIT = 1u << 23;

// Per-lane candidate state that is not needed inside a Cash-Karp attempt,
// kept in LDS (structure of arrays over the block's lanes) so that only the
// position, direction, step and curvature occupy registers in the attempt.  What
// only the candidate's end asks for (E0, u0, its counts before this run) is read
// from its queue slot again, and the lineage has a register (the linear layout,
// whose registers are full, reads it again too): with these here, 72 bytes a lane,
// two blocks of 256 on FP32 corner records did not fit a compute unit with more than
// 948 table nodes (1e6 candidates in a 256^3 grid with a patch, 1024 nodes: 287 ms;
// now 190 ms, as with 200 nodes).
template <int BS>
struct LaneShared {
    double E[BS], L[BS], Lmax[BS], tau[BS], R[BS], beta[BS];
    uint32_t id[BS], m[BS];
    uint32_t azf[BS];   // A | Z << 8 | step-limit flag << 16 | claimed to resume << 24
};

__device__ inline int unpack_A(uint32_t v) { return (int)(v & 0xffu); }
__device__ inline int unpack_Z(uint32_t v) { return (int)((v >> 8) & 0xffu); }
__device__ inline int unpack_flag(uint32_t v) { return (int)((v >> 16) & 0xffu); }
__device__ inline int unpack_resumed(uint32_t v) { return (int)(v >> 24); }
__device__ inline uint32_t pack_azf(int A, int Z, int flag, int resumed)
{
    return (uint32_t)A | ((uint32_t)Z << 8) | ((uint32_t)flag << 16) | ((uint32_t)resumed << 24);
}
// The same with another step-limit flag.
__device__ inline uint32_t with_flag(uint32_t v, int flag)
{
    return (v & 0xff00ffffu) | ((uint32_t)flag << 16);
}

// Hides a pointer's value from the optimiser so that loads through it stay
// inside the (rarely taken) branch that needs them instead of being hoisted
// out of the persistent loop into scalar registers.
template <class T>
__device__ inline const T* opaque(const T* p)
{
    asm volatile("" : "+s"(p));
    return p;
}

// Field source of a layout: 0 linear grid with kept corner values, 7 without,
// 1 corner records (per lane),
// 2 corner records gathered by the whole wave, 3 the neural field, 4 the
// analytic galactic field, 5 the multi-resolution grid (linear base grid and
// refinement patches), 6 the multi-resolution grid from corner records
// gathered by the whole wave.
template <class GT, int LAYOUT>
struct FieldOf {
    using T = GridField<GT, LAYOUT>;
};
template <class GT>
struct FieldOf<GT, 0> {
    using T = LinearKeepField<GT>;
};
template <class GT>
struct FieldOf<GT, 7> {
    using T = LinearField<GT>;
};
template <class GT>
struct FieldOf<GT, 3> {
    using T = NeuralFieldSrc;
};
template <class GT>
struct FieldOf<GT, 4> {
    using T = AnalyticFieldSrc;
};
template <class GT>
struct FieldOf<GT, 5> {
    using T = NestedField<GT>;
};
template <class GT>
struct FieldOf<GT, 6> {
    using T = NestedField<GT, true>;
};

// Layouts whose field values are gathered by the whole wave together.
template <int LAYOUT>
constexpr bool wave_gather = LAYOUT == 2 || LAYOUT == 6;

// An event's draws: out of line except in the neural stepper, whose network
// evaluation takes accumulation registers that a kernel with calls gives up
// (54 against 42 ms on 6e4 candidates).
template <int LAYOUT>
__device__ inline EventDraw draw(uint64_t seed, uint32_t id, uint32_t lineage, uint32_t m)
{
    if constexpr (LAYOUT == 3)
        return draw_event_inline(seed, id, lineage, m);
    else
        return draw_event(seed, id, lineage, m);
}

// 16-byte slots of a wave's LDS staging area.
template <class GT, int LAYOUT>
constexpr int stage_float4 = wave_gather<LAYOUT> ? coop_stage_float4<GT>
                             : LAYOUT == 0       ? keep_float4<GT>
                                                 : 0;

template <int MODE>
struct DirType {
    using T = double;
};
template <>
struct DirType<MODE_MIX> {
    using T = float;
};

// Minimum waves per SIMD the register allocation targets (occupancy vs
// spills), per precision form.  Measured on the 1e7 batch, 1024^3 grid: both
// forms are fastest at 2 (8 waves per CU, no spills); at 3 the precision form
// spills (1.36 s vs 1.30 s per batch) and the FP64 form spills inside the
// attempt.
#ifndef CRP_WAVES_MIX
#define CRP_WAVES_MIX 2
#endif
#ifndef CRP_WAVES_FP64
#define CRP_WAVES_FP64 2
#endif
// The analytic field has no memory traffic to overlap: its waves hide the
// latency of FP64 arithmetic instead.
#ifndef CRP_WAVES_ANALYTIC
#define CRP_WAVES_ANALYTIC 2
#endif

template <int MODE, int LAYOUT>
constexpr int min_waves = LAYOUT == 3   ? 1
                          : LAYOUT == 4 ? CRP_WAVES_ANALYTIC
                                        : (MODE == MODE_MIX ? CRP_WAVES_MIX : CRP_WAVES_FP64);

// TRAJ: the variant with the per-step output module compiled in (a run without
// trajectory output uses the variant without it, whose loop carries no trace
// of it).
template <int MODE, class GT, int LAYOUT, int BS, bool TRAJ>
__global__ void __launch_bounds__(BS, (min_waves<MODE, LAYOUT>))
    k_propagate(const PropParams* __restrict__ PP)
{
    using UT = typename DirType<MODE>::T;   // direction storage: FP64 or FP32
    // interaction tables, then (neural field) the network image, whose 16-byte
    // operand loads need 16-byte alignment whatever the static LDS size
    extern __shared__ __attribute__((aligned(16))) double lds[];
    __shared__ LaneShared<BS> S;              // per-lane cold state
    __shared__ unsigned long long bc[WC_COUNT];   // block bookkeeping counters
    // the waves' staging areas: the lanes' corner records or kept corner values
    __shared__ float4 stage_mem[stage_float4<GT, LAYOUT> > 0 ? BS / 64 * stage_float4<GT, LAYOUT> : 1];
    // patch table of the multi-resolution grid (LAYOUT 5 only)
    __shared__ PatchView nest_lds[LAYOUT == 5 || LAYOUT == 6 ? MAX_PATCHES : 1];
    const int t = (int)threadIdx.x;
    const int ntab = PP->tab.n;
    {
        const TableParams tp = PP->tab;
        for (int i = t; i < ntab; i += BS) {
            lds[i] = tp.e[i];
            lds[ntab + i] = tp.v[0][i];
            lds[2 * ntab + i] = tp.v[1][i];
            lds[3 * ntab + i] = tp.v[2][i];
        }
    }
    if (t < WC_COUNT)
        bc[t] = 0ull;
    if constexpr (LAYOUT == 5 || LAYOUT == 6) {
        if (t < PP->nest.np)
            nest_lds[t] = PP->nest.p[t];
    }
    __syncthreads();
    TableView T;
    T.e = lds;
    T.v[0] = lds + ntab;
    T.v[1] = lds + 2 * ntab;
    T.v[2] = lds + 3 * ntab;
    T.n = ntab;
    T.lg0 = PP->tab.lg0;
    T.scale = PP->tab.scale;

    // the wave's index in the block, in a scalar register
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    typename FieldOf<GT, LAYOUT>::T F;
    if constexpr (LAYOUT == 3) {
        // the network image follows the tables in dynamic LDS
        char* img = (char*)(lds + 4 * ntab);
        nf_stage_lds(img, PP->nf.img);
        __syncthreads();
        F.v = nf_view_lds(img, PP->nf.origin, PP->nf.inv_box, PP->nf.b_scale);
    } else if constexpr (LAYOUT == 4) {
        F.a = PP->ana;
    } else if constexpr (LAYOUT == 5 || LAYOUT == 6) {
        F.g = PP->grid;
        F.P = nest_lds;
        F.np = PP->nest.np;
        F.set_first(PP->nest.p[0]);
        if constexpr (LAYOUT == 6)
            F.stage = (float*)(stage_mem + wave * stage_float4<GT, LAYOUT>);
    } else {
        F.g = PP->grid;
        if constexpr (stage_float4<GT, LAYOUT> > 0)
            F.stage = (float*)(stage_mem + wave * stage_float4<GT, LAYOUT>);
    }
    const StepParams sp = PP->sp;
    const int lane = lane_id();
    const unsigned long long qcap = (unsigned long long)PP->q.cap;
    const unsigned long long tail0 = PP->tail0;
    const int lane_cap = PP->lane_cap;
    const int refill = min(PP->refill, lane_cap);
    const bool no_append = PP->no_append != 0;
    const int64_t max_cycles = PP->max_cycles;
    DevCounters* const cnt = PP->cnt;

    // registers through the attempt: position, direction, step, curvature
    double x[3] = {0.0, 0.0, 0.0};
    UT u[3] = {0, 0, 0};
    double h = 0.0, kappa = 0.0;
    int64_t slot = 0;
    bool active = false, fresh = true;
    // S.R, S.beta and kappa belong to the candidate's present species and energy
    bool rated = false;
    uint32_t nacc = 0u, nrejd = 0u, nforced = 0u;   // this candidate's counts in this run
    uint32_t lineage_reg = 0u;
    uint32_t nclaimed = 0u;                         // TRAJ: its steps before this run
    auto lineage = [&]() -> uint32_t {
        if constexpr (LAYOUT != 0)
            return lineage_reg;
        else
            return opaque(PP)->q.lineage[slot];
    };
    uint64_t iters = 0;                             // attempts of the wave
    // the lane holds a candidate whose last cycle stopped just before an
    // interaction for want of an output slot: it finishes that cycle first
    bool resume = false;
    // field at the current position (first stage of the next attempt, kept for
    // the retry after a rejection).  Cooperative layouts: its record is fetched
    // as soon as the position is known (after the attempt that moved there, or
    // at the claim), while the rest of the cycle runs
    using BT = typename DirType<MODE>::T;
    BT b1[3] = {0, 0, 0};
    enum { B_NONE = 0, B_FETCHED = 1, B_KNOWN = 2 };
    int bst = B_NONE;
    bool initial_left = true;
    // this wave's reservation of appended slots [rb, re): taken with one
    // atomicAdd, handed to idle lanes as their producers publish them
    unsigned long long rb = 0, re = 0;
    uint32_t sleeps = 0, backoff = 0;
    unsigned long long seen_done = 0;   // progress of the run seen while idle
    const unsigned long long fin0 = PP->fin0;

    for (;;) {
        // ---- refill idle lanes from the queue -------------------------------
        const uint64_t idle = __ballot(!active);
        const int nidle = __popcll(idle);
        // lanes it may fill: up to lane_cap with injected candidates, any with
        // appended ones, which a wave with work looks for every eighth iteration
        const int nfree = initial_left ? nidle - (64 - lane_cap) : nidle;
        bool claim = nfree > 0 && (idle == ~0ull || nfree >= refill);
        if (!initial_left)
            claim = claim && !no_append && (idle == ~0ull || (iters & 7u) == 0u);
        if (claim) {
            const int rank = lanes_below(idle);
            unsigned long long base = 0, take = 0, ibase = 0, itake = 0;
            // appended candidates first: a long secondary taken up after the
            // injected ones runs on alone at the end of the launch (1e6 nuclei in
            // a 512^3 FP32 grid, 3.8e5 secondaries: 164 -> 147 ms).  A wave with
            // work looks for them every eighth iteration only: the look is two
            // dependent loads of contended counters, and taking a few at a time an
            // acquire (looking at every claim: 147 against 133 ms there; 1e7 in a
            // 1024^3 grid, refill 4, 1103 against 989 ms, before either 1048 ms)
            if (!no_append &&
                (!initial_left || rb < re || idle == ~0ull || (iters & 7u) == 0u)) {
                if (rb >= re) {
                    unsigned long long b = 0, want = (unsigned long long)nidle;
                    if (lane == 0) {
                        // while injected candidates are left only what is there
                        if (initial_left) {
                            unsigned long long tl = __hip_atomic_load(
                                &cnt->tail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            const unsigned long long hd = __hip_atomic_load(
                                &cnt->head1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            if (tl > qcap)
                                tl = qcap;
                            want = (unsigned long long)nfree;
                            if (tl < hd + want)
                                want = tl > hd ? tl - hd : 0ull;
                        }
                        if (want != 0ull)
                            b = atomicAdd(&cnt->head1, want);
                    }
                    rb = __shfl(b, 0);
                    re = rb + __shfl(want, 0);
                }
                if (rb < re) {
                    // idle lane of rank r looks at slot rb + r; the published
                    // prefix of the reservation is handed out in order
                    const unsigned long long sl = rb + (unsigned long long)rank;
                    const bool mine = !active && sl < re;
                    bool pub = false;
                    if (mine && sl < qcap)
                        pub = __hip_atomic_load(opaque(PP)->q.ready + sl, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT) != 0u;
                    const uint64_t gap = __ballot(mine && !pub);
                    if (gap)
                        take = (unsigned long long)__popcll(
                            idle & ((1ull << __builtin_ctzll(gap)) - 1ull));
                    else
                        take = re - rb < (unsigned long long)nidle ? re - rb
                                                                   : (unsigned long long)nidle;
                    base = rb;
                    rb += take;
                    // the slots' contents are read after their flags; a poll that
                    // finds none does not pay for the acquire, which empties the
                    // compute unit's vector cache
                    if (take != 0ull)
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                }
            }
            if (initial_left) {
                // a lane is kept for each reserved slot that is being written (its
                // producer publishes it within its iteration; a slot reserved
                // past the tail may never be)
                int want = nfree - (int)take;
                if (rb < re) {
                    unsigned long long tl = 0;
                    if (lane == 0)
                        tl = __hip_atomic_load(&cnt->tail, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                    tl = __shfl(tl, 0);
                    tl = tl < qcap ? tl : qcap;
                    tl = tl < re ? tl : re;
                    want -= tl > rb ? (int)(tl - rb) : 0;
                }
                if (want > 0) {
                    bool left = false;
                    if (lane == 0)
                        claim_initial(cnt, tail0, want, ibase, itake, left);
                    ibase = __shfl(ibase, 0);
                    itake = __shfl(itake, 0);
                    initial_left = __shfl((int)left, 0) != 0;
                }
            }
            if (!active && (unsigned long long)rank < take + itake) {
                const QueueSoA& q = opaque(PP)->q;
                slot = (int64_t)((unsigned long long)rank < take
                                     ? base + (unsigned long long)rank
                                     : ibase + ((unsigned long long)rank - take));
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    x[a] = q.x[a * q.cap + slot];
                    u[a] = (UT)q.u[a * q.cap + slot];
                }
                S.E[t] = q.E[slot];
                S.L[t] = q.L[slot];
                S.Lmax[t] = q.Lmax[slot];
                h = q.hctrl[slot];
                S.tau[t] = q.tau[slot];
                S.id[t] = q.id[slot];
                S.m[t] = q.m[slot];
                if constexpr (LAYOUT != 0)
                    lineage_reg = q.lineage[slot];
                if constexpr (TRAJ)
                    nclaimed = q.nsteps[slot];
                resume = S.tau[t] < 0.0;
                // a resumed cycle keeps the step limit its step had
                S.azf[t] = pack_azf(q.A[slot], q.Z[slot],
                                    resume ? event_due_flag(S.tau[t]) : LIM_CTRL, resume ? 1 : 0);
                if ((unsigned long long)slot >= tail0)
                    q.ready[slot] = 0u;   // clean for the next run
                active = true;
                fresh = !resume;
                rated = false;
                bst = B_NONE;
            }
        }
        if (__ballot(active) == 0ull) {
            // nothing to do: leave once the run has drained (or nothing can be
            // appended any more), else wait for secondaries that busy waves may
            // still append
            if (!initial_left && no_append)
                break;
            if (!initial_left) {
                bool drained = false;
                unsigned long long done = 0;
                if (lane == 0)
                    drained = run_drained(cnt, fin0, qcap, done);
                if (__shfl((int)drained, 0))
                    break;
                done = __shfl(done, 0);
                if (done != seen_done) {   // the run is progressing: keep waiting
                    seen_done = done;
                    sleeps = 0;
                }
            }
            if (backoff < IDLE_BACKOFF)
                ++backoff;
            for (uint32_t k = 0; k < backoff; ++k)
                __builtin_amdgcn_s_sleep(127);
            sleeps += backoff;
            if (sleeps >= IDLE_SLEEP_LIMIT) {
                if (lane == 0)
                    atomicAdd(&cnt->error, 1ull);
                break;
            }
            continue;
        }
        backoff = 0;

        // cooperative layouts: newly claimed and resumed candidates' records
        if constexpr (wave_gather<LAYOUT>) {
            const bool fetch = active && !resume && bst == B_NONE;
            if (__ballot(fetch) != 0ull) {
                F.prefetch(x, fetch);
                bst = fetch ? B_FETCHED : bst;
            }
        }

        // ---- start of a cycle: rates and step proposal -----------------------
        // (rates follow from species and energy: a candidate that loses none
        // keeps them; on backtracked events they took an eighth of the
        // instructions)
        if (active && fresh && !rated) {
            const uint32_t azf = S.azf[t];
            const int A = unpack_A(azf), Z = unpack_Z(azf);
            const double E = S.E[t];
            const Rates rt = species_rates(T, A, Z, E);
            // backtracking follows the antiparticle: charge -Z
            kappa = ((double)(sp.charge_sign * Z) * kC) / E;
            S.R[t] = rt.r;
            S.beta[t] = rt.beta;
            rated = true;
        }
        if (active && fresh) {
            const double R = S.R[t], beta = S.beta[t];
            const double L = S.L[t], Lmax = S.Lmax[t], tau = S.tau[t];
            int flag = LIM_CTRL;   // h: the controller's step
            if (Lmax - L < h) {
                h = Lmax - L;
                flag = LIM_TRAJ;
            }
            if (R > 0.0 && tau / R < h) {
                h = tau / R;
                flag = LIM_INTER;
            }
            if (beta > 0.0 && sp.eps_loss / beta < h) {
                h = sp.eps_loss / beta;
                flag = LIM_LOSS;
            }
            if (sp.obs_r > 0.0) {
                const double d[3] = {x[0] - sp.obs[0], x[1] - sp.obs[1], x[2] - sp.obs[2]};
                const double dist = sqrt(dot3(d, d));
                const double half = 0.5 * sp.obs_r;
                double hob = dist - half;
                if (hob < half)
                    hob = half;
                if (hob < h) {
                    h = hob;
                    flag = LIM_OBS;
                }
            }
            S.azf[t] = with_flag(S.azf[t], flag);
            fresh = false;
        }

        // ---- the field at this position, where it is not yet known ----------
        if constexpr (wave_gather<LAYOUT>) {
            if (__ballot(bst == B_FETCHED) != 0ull) {
                BT bp[3];
                if constexpr (MODE == MODE_FP64)
                    F.fp64_prefetched(x, bp);
                else
                    F.fp32_prefetched(x, bp);
                if (bst == B_FETCHED) {
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        b1[q] = bp[q];
                    bst = B_KNOWN;
                }
            }
        } else if constexpr (LAYOUT != 3) {
            if (active && !resume && bst == B_NONE) {
                if constexpr (MODE == MODE_FP64)
                    F.fp64(x, b1);
                else
                    F.fp32(x, b1);
                bst = B_KNOWN;
            }
        }

        // ---- one Cash-Karp attempt -------------------------------------------
        int status = ST_ACTIVE;
        bool park = false, rec = false, fin = false;
        // lanes that step in this iteration (a resumed lane only finishes its
        // interrupted cycle)
        const bool stepping = active && !resume;
        // with the cooperative gather every lane of the wave takes part in the
        // attempt (idle lanes on a harmless cell); results are used only by
        // busy lanes
        double x5[3];
        UT u5[3];
        double err = 0.0;
        if (stepping || wave_gather<LAYOUT> || LAYOUT == 3) {
            if constexpr (MODE == MODE_FP64) {
                const double y[6] = {x[0], x[1], x[2], u[0], u[1], u[2]};
                double y5[6];
                err = ck_attempt_fp64(F, kappa, y, h, y5, stepping, b1);
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    x5[q] = y5[q];
                    u5[q] = y5[3 + q];
                }
            } else {
                if constexpr (LAYOUT == 3)
                    err = ck_attempt_mix_rolled(F, kappa, x, u, h, x5, u5);
                else
                    err = ck_attempt_mix_f(F, kappa, x, u, h, x5, u5, stepping, b1);
            }
        }
        const double r = err / sp.tol;
        const bool acc = stepping && (r <= 1.0 || h <= sp.hmin);
        if constexpr (wave_gather<LAYOUT>) {
            // accepted lanes move to x5: start fetching B(x5) now, so that the
            // loads overlap the rest of the cycle
            if (__ballot(acc) != 0ull)
                F.prefetch(x5, acc);
            bst = acc ? B_FETCHED : bst;
        }
        // the cycle's energy and optical depth after the step, and whether an
        // interaction is due
        double E = 0.0, tau = 0.0;
        bool evt = false, cycle = false;
        if (stepping) {
            // step-size factor: r = 0 (and a NaN, accepted at hmin) grow by 5
            double fac = (double)ctrl_k(r) * 0x1p-10;
            if (acc)
                fac = r > 0.0 && fac < 5.0 ? fac : 5.0;
            else if (fac < 0.1)
                fac = 0.1;
            double hn = h * fac;
            if (hn < sp.hmin)
                hn = sp.hmin;
            if (acc) {
                if constexpr (!wave_gather<LAYOUT>)
                    bst = B_NONE;
                nacc += 1u;
                nforced += r > 1.0 ? 1u : 0u;
                if (hn > sp.hmax)
                    hn = sp.hmax;
                // integration module: position, direction, trajectory length
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    x[q] = x5[q];
                if (sp.renorm) {
                    if constexpr (MODE == MODE_FP64) {
                        const double nrm = sqrt(dot3(u5, u5));
#pragma unroll
                        for (int q = 0; q < 3; ++q)
                            u[q] = u5[q] / nrm;
                    } else {
                        const float nrm = sqrtf(dot3f(u5, u5));
#pragma unroll
                        for (int q = 0; q < 3; ++q)
                            u[q] = u5[q] / nrm;
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        u[q] = u5[q];
                }
                const double L = S.L[t] + h;
                S.L[t] = L;
                // continuous loss: (2,2) Pade form of exp(-beta h), 1 where
                // beta is 0 (12 / 12)
                E = S.E[t];
                const double beta = S.beta[t];
                if (beta != 0.0) {
                    const double z = beta * h;
                    const double z2 = z * z;
                    const double num = (12.0 - 6.0 * z) + z2;
                    const double den = (12.0 + 6.0 * z) + z2;
                    const double E0 = E;
                    E = E * (num / den);
                    rated = rated && E == E0;
                }
                // stochastic interactions: optical-depth clock
                tau = S.tau[t] - S.R[t] * h;
                evt = unpack_flag(S.azf[t]) == LIM_INTER || tau <= 0.0;
                cycle = true;
            } else {
                nrejd += 1u;              // same position: b1 keeps its field
                S.azf[t] = with_flag(S.azf[t], LIM_CTRL);
            }
            h = hn;   // the retry's step, or the controller's for the next cycle
        }
        if (resume) {
            // the interrupted cycle: its step and loss are done, its
            // interaction is due (the clock value is replaced after it)
            E = S.E[t];
            evt = true;
            cycle = true;
            resume = false;
        }

        // ---- interaction: channel first, then a slot for its product --------
        // (one atomic per wave for each kind of product); a lane that finds no
        // slot keeps its state as before the interaction and is parked, to
        // finish the cycle in a later run: nothing is lost
        int chan = CH_NONE;
        double dE = 0.0, Esec = 0.0;
        bool defer = false;
        unsigned long long slot_n = 0, slot_pi = 0;
        EventDraw w{0ull, 0.0};
        if (__ballot(evt) != 0ull) {
            if (evt) {
                w = draw<LAYOUT>(opaque(PP)->sp.seed, S.id[t], lineage(), S.m[t] + 1u);
                const uint32_t azf = S.azf[t];
                const Rates ri = species_rates(T, unpack_A(azf), unpack_Z(azf), E);
                const double Ptot = ri.rpi + ri.rn;
                chan = !(Ptot > 0.0) ? CH_NULL
                                     : (unit_uniform(w.w0) * Ptot < ri.rpi ? CH_PI : CH_N);
            }
            const uint64_t mn = __ballot(chan == CH_N);
            if (mn) {
                unsigned long long base = 0;
                if (lane == 0)
                    base = atomicAdd(&cnt->tail, (unsigned long long)__popcll(mn));
                slot_n = __shfl(base, 0) + (unsigned long long)lanes_below(mn);
                defer = chan == CH_N && slot_n >= qcap;
            }
            const uint64_t mpi = __ballot(chan == CH_PI);
            if (mpi) {
                unsigned long long base = 0;
                if (lane == 0)
                    base = atomicAdd(&cnt->neu_n, (unsigned long long)__popcll(mpi));
                slot_pi = __shfl(base, 0) + (unsigned long long)lanes_below(mpi);
                defer = defer || (chan == CH_PI &&
                                  slot_pi >= (unsigned long long)opaque(PP)->neu.cap);
            }
        }
        if (defer) {
            atomicAdd(&bc[chan == CH_N ? WC_QDEFER : WC_NDEFER], 1ull);
            S.E[t] = E;
            S.tau[t] = event_due_marker(unpack_flag(S.azf[t]));
            park = true;
        } else if (cycle) {
            if (evt) {
                const uint32_t m = S.m[t] + 1u;
                S.m[t] = m;
                rated = false;
                const uint32_t azf = S.azf[t];
                int A = unpack_A(azf), Z = unpack_Z(azf);
                const double Eint = E;
                atomicAdd(&bc[WC_EVENTS], 1ull);
                if (chan == CH_PI) {
                    dE = (opaque(PP)->sp.kappa_pi * Eint) / (double)A;
                    E = Eint - dE;
                    atomicAdd(&bc[WC_PI], 1ull);
                    const NeutralSoA& nq = opaque(PP)->neu;
                    const int64_t k = (int64_t)slot_pi;
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        nq.x[a * nq.cap + k] = x[a];
                        nq.u[a * nq.cap + k] = (double)u[a];
                    }
                    nq.E[k] = dE;
                    nq.id[k] = S.id[t];
                    nq.lineage[k] = lineage();
                    nq.m[k] = m;
                    nq.chan[k] = 0;
                } else if (chan == CH_N) {
                    const int pout = (2 * Z > A) ? 1 : 0;
                    Esec = Eint / (double)A;
                    Z -= pout;
                    A -= 1;
                    E = Eint - Esec;
                    S.azf[t] = pack_azf(A, Z, unpack_flag(azf), unpack_resumed(azf));
                    atomicAdd(&bc[WC_N], 1ull);
                    // the secondary proton: a new candidate in the queue
                    const QueueSoA& q = opaque(PP)->q;
                    const int64_t k = (int64_t)slot_n;
                    const uint32_t id = S.id[t];
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        q.x[a * q.cap + k] = x[a];
                        q.u[a * q.cap + k] = (double)u[a];
                        q.u0[a * q.cap + k] = q.u0[a * q.cap + slot];
                    }
                    q.E[k] = Esec;
                    q.L[k] = S.L[t];
                    q.Lmax[k] = S.Lmax[t];
                    q.hctrl[k] = sp.hmin;
                    q.E0[k] = q.E0[slot];
                    q.id[k] = id;
                    q.lineage[k] = m;
                    q.m[k] = 0u;
                    q.nsteps[k] = 0u;
                    q.nrej[k] = 0u;
                    q.A[k] = 1;
                    q.Z[k] = 1;
                    q.tau[k] = draw<LAYOUT>(opaque(PP)->sp.seed, id, m, 0u).tau;
                    __hip_atomic_store(q.ready + k, 1u, __ATOMIC_RELEASE,
                                       __HIP_MEMORY_SCOPE_AGENT);
                } else {
                    atomicAdd(&bc[WC_NULL], 1ull);
                }
                // all interaction state is reset after an interaction
                tau = w.tau;
            }
            S.E[t] = E;
            S.tau[t] = tau;
            // boundary and observer modules, checked after the cycle
            // cycles of this run: its accepted steps and the one resumed, if any
            const uint32_t cyc = nacc + (uint32_t)unpack_resumed(S.azf[t]);
            if (sp.obs_r > 0.0) {
                const double d[3] = {x[0] - sp.obs[0], x[1] - sp.obs[1], x[2] - sp.obs[2]};
                if (sqrt(dot3(d, d)) <= sp.obs_r)
                    status = ST_OBSERVED;
            }
            if (status == ST_ACTIVE && sp.bnd_r > 0.0) {
                const double d[3] = {x[0] - sp.bnd[0], x[1] - sp.bnd[1], x[2] - sp.bnd[2]};
                if (sqrt(dot3(d, d)) >= sp.bnd_r)
                    status = ST_BOUNDARY;
            }
            if (status == ST_ACTIVE &&
                (unpack_flag(S.azf[t]) == LIM_TRAJ || S.L[t] >= S.Lmax[t]))
                status = ST_MAX_TRAJ;
            if (status == ST_ACTIVE && E < sp.e_floor)
                status = ST_ENERGY_FLOOR;
            if (status != ST_ACTIVE) {
                fin = true;
                atomicAdd(&bc[WC_FINISHED], 1ull);
                atomicAdd(&bc[status == ST_OBSERVED   ? WC_OBSERVED
                              : status == ST_BOUNDARY ? WC_BOUNDARY
                              : status == ST_MAX_TRAJ ? WC_MAXTRAJ
                                                      : WC_EFLOOR],
                          1ull);
            } else if (max_cycles > 0 && (int64_t)cyc >= max_cycles) {
                park = true;
            }
            // output module: every traj_every-th step and the last one
            if constexpr (TRAJ) {
                // read here rather than kept in scalar registers all loop long
                const StepParams& spp = opaque(PP)->sp;
                const uint32_t every = spp.traj_every;
                if (every != 0u && S.id[t] < spp.traj_ids)
                    rec = (nclaimed + nacc) % every == 0u || status != ST_ACTIVE;
            }
            fresh = true;
        }
        // ---- appends: one atomic per wave for each kind ----------------------
        if constexpr (TRAJ) {
            const uint64_t mk = __ballot(rec);
            if (mk) {
                unsigned long long base = 0;
                if (lane == 0)
                    base = atomicAdd(&cnt->traj_n, (unsigned long long)__popcll(mk));
                base = __shfl(base, 0);
                if (rec) {
                    const TrajSoA& tq = opaque(PP)->traj;
                    const unsigned long long i = base + (unsigned long long)lanes_below(mk);
                    if (i < (unsigned long long)tq.cap) {
                        const int64_t k = (int64_t)i;
#pragma unroll
                        for (int a = 0; a < 3; ++a)
                            tq.x[a * tq.cap + k] = x[a];
                        tq.L[k] = S.L[t];
                        tq.E[k] = S.E[t];
                        tq.id[k] = S.id[t];
                        tq.lineage[k] = lineage();
                        tq.n[k] = nclaimed + nacc;
                        tq.A[k] = unpack_A(S.azf[t]);
                    }   // points past the capacity are counted by the host
                }
            }
        }
        {
            const uint64_t mk = __ballot(fin);
            if (mk) {
                unsigned long long base = 0;
                if (lane == 0)
                    base = atomicAdd(&cnt->fin_n, (unsigned long long)__popcll(mk));
                base = __shfl(base, 0);
                if (fin) {
                    const unsigned long long i = base + (unsigned long long)lanes_below(mk);
                    const PropParams* Q = opaque(PP);
                    if (i < (unsigned long long)Q->fin.cap) {
                        const FinishedSoA& f = Q->fin;
                        const int64_t k = (int64_t)i;
                        const uint32_t ns = Q->q.nsteps[slot], nr = Q->q.nrej[slot];
#pragma unroll
                        for (int a = 0; a < 3; ++a) {
                            f.x[a * f.cap + k] = x[a];
                            f.u[a * f.cap + k] = (double)u[a];
                            f.u0[a * f.cap + k] = Q->q.u0[a * Q->q.cap + slot];
                        }
                        f.E[k] = S.E[t];
                        f.L[k] = S.L[t];
                        f.E0[k] = Q->q.E0[slot];
                        f.id[k] = S.id[t];
                        f.lineage[k] = lineage();
                        f.m[k] = S.m[t];
                        f.nsteps[k] = ns + nacc;
                        f.nrej[k] = nr + nrejd;
                        f.status[k] = status;
                        f.A[k] = unpack_A(S.azf[t]);
                        f.Z[k] = unpack_Z(S.azf[t]);
                    }
                    active = false;
                }
            }
        }
        {
            const uint64_t mk = __ballot(park);
            if (mk) {
                unsigned long long base = 0;
                if (lane == 0)
                    base = atomicAdd(&cnt->park_n, (unsigned long long)__popcll(mk));
                base = __shfl(base, 0);
                if (park) {
                    const unsigned long long i = base + (unsigned long long)lanes_below(mk);
                    const PropParams* Q = opaque(PP);
                    if (i < (unsigned long long)Q->park.cap) {
                        const QueueSoA& pq = Q->park;
                        const int64_t k = (int64_t)i;
                        const uint32_t ns = Q->q.nsteps[slot], nr = Q->q.nrej[slot];
#pragma unroll
                        for (int a = 0; a < 3; ++a) {
                            pq.x[a * pq.cap + k] = x[a];
                            pq.u[a * pq.cap + k] = (double)u[a];
                            pq.u0[a * pq.cap + k] = Q->q.u0[a * Q->q.cap + slot];
                        }
                        pq.E[k] = S.E[t];
                        pq.L[k] = S.L[t];
                        pq.Lmax[k] = S.Lmax[t];
                        pq.hctrl[k] = h;
                        pq.tau[k] = S.tau[t];
                        pq.E0[k] = Q->q.E0[slot];
                        pq.id[k] = S.id[t];
                        pq.lineage[k] = lineage();
                        pq.m[k] = S.m[t];
                        pq.nsteps[k] = ns + nacc;
                        pq.nrej[k] = nr + nrejd;
                        pq.A[k] = unpack_A(S.azf[t]);
                        pq.Z[k] = unpack_Z(S.azf[t]);
                    }
                    active = false;
                }
            }
        }

        // ---- bookkeeping of candidates that left their lane ------------------
        if (fin || park) {
            atomicAdd(&bc[WC_STEPS], (unsigned long long)nacc);
            atomicAdd(&bc[WC_REJECTS], (unsigned long long)nrejd);
            atomicAdd(&bc[WC_ATTEMPTS], (unsigned long long)nacc + nrejd);
            if (nforced != 0u)
                atomicAdd(&bc[WC_FORCED], (unsigned long long)nforced);
            nacc = nrejd = nforced = 0u;
        }
        ++iters;
    }
    if (lane == 0)
        atomicAdd(&bc[WC_LANES], 64ull * iters);
    __syncthreads();   // every wave of the block has left the loop
    flush_counts(cnt, bc);
}

// Explicit instantiations: FP64 / mixed stage arithmetic x grid element type x
// grid layout (multi-resolution corner records exist for FP32 grids only).
#define CRP_INST(MODE, GT, LAYOUT)                                                          \
    template __global__ void k_propagate<MODE, GT, LAYOUT, 128, false>(const PropParams*); \
    template __global__ void k_propagate<MODE, GT, LAYOUT, 256, false>(const PropParams*); \
    template __global__ void k_propagate<MODE, GT, LAYOUT, 128, true>(const PropParams*);  \
    template __global__ void k_propagate<MODE, GT, LAYOUT, 256, true>(const PropParams*);
CRP_INST(MODE_FP64, double, 0)
CRP_INST(MODE_FP64, double, 7)
CRP_INST(MODE_FP64, double, 2)
CRP_INST(MODE_FP64, double, 4)
CRP_INST(MODE_FP64, double, 5)
CRP_INST(MODE_FP64, float, 5)
CRP_INST(MODE_MIX, double, 5)
CRP_INST(MODE_MIX, float, 5)
CRP_INST(MODE_MIX, float, 6)
CRP_INST(MODE_FP64, float, 6)
CRP_INST(MODE_MIX, double, 4)
CRP_INST(MODE_FP64, float, 0)
CRP_INST(MODE_FP64, float, 7)
CRP_INST(MODE_FP64, float, 2)
CRP_INST(MODE_MIX, double, 0)
CRP_INST(MODE_MIX, double, 7)
CRP_INST(MODE_MIX, double, 2)
CRP_INST(MODE_MIX, float, 0)
CRP_INST(MODE_MIX, float, 7)
CRP_INST(MODE_MIX, float, 2)
#undef CRP_INST
// neural field (precision form, one block of 256 per CU: the network fills LDS)
template __global__ void k_propagate<MODE_MIX, float, 3, 256, false>(const PropParams*);
template __global__ void k_propagate<MODE_MIX, float, 3, 256, true>(const PropParams*);

// -------------------------------------------------------------------------
// Injection: validation (first bad index) and slot initialisation.
// -------------------------------------------------------------------------
__global__ void k_validate(int64_t n, const uint32_t* id, const int32_t* A, const int32_t* Z,
                           const double* E, const double* pos, const double* dir,
                           const double* lmax, double max_extent,
                           unsigned long long* first_bad)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    bool ok = A[i] >= 1 && A[i] <= 255 && Z[i] >= 1 && Z[i] <= A[i];
    ok = ok && isfinite(E[i]) && E[i] > 0.0 && isfinite(lmax[i]) && lmax[i] > 0.0;
    double d2 = 0.0, p2 = 0.0;
    for (int a = 0; a < 3; ++a) {
        ok = ok && isfinite(pos[3 * i + a]) && isfinite(dir[3 * i + a]);
        d2 += dir[3 * i + a] * dir[3 * i + a];
        p2 += pos[3 * i + a] * pos[3 * i + a];
    }
    ok = ok && fabs(sqrt(d2) - 1.0) <= 1e-12;
    ok = ok && (sqrt(p2) + lmax[i] < max_extent);
    (void)id;
    if (!ok)
        atomicMin(first_bad, (unsigned long long)i);
}

// Queue slot base + i takes input candidate perm[i] (perm null: candidate i).
__global__ void k_inject(QueueSoA q, int64_t base, int64_t n, const uint32_t* id,
                         const int32_t* A, const int32_t* Z, const double* E,
                         const double* pos, const double* dir, const double* lmax,
                         const uint32_t* perm, uint64_t seed, double hmin, int mix)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const int64_t s = perm ? (int64_t)perm[i] : i;
    Cand c;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        c.x[a] = pos[3 * s + a];
        const double d = dir[3 * s + a];
        c.u[a] = mix ? (double)(float)d : d;
        c.u0[a] = c.u[a];
    }
    c.E = E[s];
    c.E0 = E[s];
    c.L = 0.0;
    c.Lmax = lmax[s];
    c.hctrl = hmin;
    c.id = id[s];
    c.lineage = 0;
    c.m = 0;
    c.nsteps = 0;
    c.nrej = 0;
    c.A = A[s];
    c.Z = Z[s];
    c.tau = optical_depth(event_draw(seed, c.id, 0, 0).w[1]);
    store_cand(q, base + i, c);
}

// Sort keys of the longest-expected-path-first injection order: w = lmax * Z / E
// (> 0 and finite for a validated candidate) descending, i.e. the bitwise
// complement of w's IEEE pattern ascending (positive doubles order like their
// bit patterns); idx = 0..n-1, the payload the sort permutes.
__global__ void k_inject_keys(int64_t n, const int32_t* Z, const double* E, const double* lmax,
                              unsigned long long* keys, uint32_t* idx)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const double w = lmax[i] * (double)Z[i] / E[i];
    keys[i] = ~(unsigned long long)__double_as_longlong(w);
    idx[i] = (uint32_t)i;
}

// -------------------------------------------------------------------------
// Field evaluation at arbitrary points (mode 0: FP64 weights, 1: FP32).
// -------------------------------------------------------------------------
template <class GT, int LAYOUT>
__global__ void k_eval_field(GridView g, int64_t n, const double* pos, double* B, int mode)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    GridField<GT, LAYOUT> F{g};
    const double p[3] = {pos[3 * i], pos[3 * i + 1], pos[3 * i + 2]};
    if (mode == MODE_FP64) {
        double b[3];
        F.fp64(p, b);
        B[3 * i] = b[0];
        B[3 * i + 1] = b[1];
        B[3 * i + 2] = b[2];
    } else {
        float b[3];
        F.fp32(p, b);
        B[3 * i] = (double)b[0];
        B[3 * i + 1] = (double)b[1];
        B[3 * i + 2] = (double)b[2];
    }
}

// The same on the linear layout for many points, the corner values moved by the
// wave together.  Bound by the 128-byte lines read: a point's four z-pairs (48 or
// 24 bytes) lie in 5.2 (4.7) of them, and where each lane loads its own corners a
// line is touched by several instructions, between which the other waves' lines
// push it out of the caches (7.8 lines read per point, at 6.9 TB/s).  Here
// neighbouring lanes load neighbouring pieces, so one instruction touches all of
// a z-pair: LPP lanes take a point, FP64 three 16-byte pieces per z-pair, FP32 one
// vertex each, and LDS hands the values to the point's own lane.  Points whose
// z-pair wraps around the grid are gathered by their lane.
// 4e6 points on the 256^3 FP64 grid: 581 -> 409 us; FP32: 527 -> 373 us.
template <class GT>
__global__ void __launch_bounds__(256) k_eval_linear(GridView g, int64_t n, const double* pos,
                                                     double* B, int mode)
{
    constexpr bool F64 = sizeof(GT) == 8;
    constexpr int LPP = F64 ? 12 : 8;         // lanes (and pieces) per point
    constexpr int PB = F64 ? 16 : 12;         // bytes per piece
    constexpr int PE = PB / (int)sizeof(GT);  // elements per piece
    __shared__ __attribute__((aligned(16))) char stage[4 * 64 * LPP * PB];
    __shared__ unsigned long long where[256];
    const int t = (int)threadIdx.x, lane = t & 63, wave = t >> 6;
    char* st = stage + wave * (64 * LPP * PB);
    const int64_t first = (int64_t)blockIdx.x * 256 + wave * 64;
    const int64_t i = first + lane;
    const bool live = i < n;
    double p[3] = {0.0, 0.0, 0.0};
    if (live) {
        p[0] = pos[3 * i];
        p[1] = pos[3 * i + 1];
        p[2] = pos[3 * i + 2];
    }
    const Cell c = locate(g, p);
    const bool own = c.i1[2] == 0;            // the z-pair wraps
    // the point's cell number, and whether x and y wrap (bits 61, 62); bit 63: none
    const unsigned long long cell = (unsigned long long)cell_index(g, c);
    where[t] = live && !own ? cell | (c.i1[0] == 0 ? 1ull << 61 : 0ull) |
                                  (c.i1[1] == 0 ? 1ull << 62 : 0ull)
                            : 1ull << 63;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const GT* G = (const GT*)g.data;
    GT e[LPP][PE];
#pragma unroll
    for (int j = 0; j < LPP; ++j) {
        const int idx = 64 * j + lane;
        const int r = idx / LPP;
        // pieces are rotated by the point's number against bank conflicts
        int q = idx - LPP * r - (F64 ? (r >> 2) & 3 : 0);
        if (q < 0)
            q += LPP;
        const int row = F64 ? q / 3 : q >> 1;              // dx + 2 dy
        const int off = F64 ? 2 * (q - 3 * row) : 3 * (q & 1);   // elements into the z-pair
        const unsigned long long w = where[(t & ~63) + r];
#pragma unroll
        for (int k = 0; k < PE; ++k)
            e[j][k] = (GT)0;
        if ((int64_t)w >= 0) {
            int64_t o = (int64_t)(w & ((1ull << 61) - 1ull)) * 3 + off;
            if (row & 1)
                o += ((w >> 61) & 1ull) ? -(int64_t)(g.n[0] - 1) * g.stride[0] : g.stride[0];
            if (row & 2)
                o += ((w >> 62) & 1ull) ? -(int64_t)(g.n[1] - 1) * g.stride[1] : g.stride[1];
            __builtin_memcpy(e[j], G + o, PB);
        }
    }
#pragma unroll
    for (int j = 0; j < LPP; ++j)
        __builtin_memcpy(__builtin_assume_aligned(st + PB * (64 * j + lane), F64 ? 16 : 4), e[j],
                         PB);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    GT v[8][3];
    GT f[24];   // row by row: the z-pair's two vectors
#pragma unroll
    for (int q = 0; q < LPP; ++q) {
        int at = q + (F64 ? (lane >> 2) & 3 : 0);
        if (at >= LPP)
            at -= LPP;
        __builtin_memcpy(f + PE * q,
                         __builtin_assume_aligned(st + PB * (LPP * lane + at), F64 ? 16 : 4), PB);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int a = 0; a < 3; ++a)
            v[k][a] = f[6 * (k & 3) + 3 * (k >> 2) + a];
    if (live && own)
        gather_linear<GT>(g, c, v);
    if (!live)
        return;
    if (mode == MODE_FP64) {
        double b[3];
        interp_fp64(c.t, v, b);
        B[3 * i] = b[0];
        B[3 * i + 1] = b[1];
        B[3 * i + 2] = b[2];
    } else {
        float b[3];
        interp_fp32(c.t, v, b);
        B[3 * i] = (double)b[0];
        B[3 * i + 1] = (double)b[1];
        B[3 * i + 2] = (double)b[2];
    }
}
template __global__ void k_eval_linear<double>(GridView, int64_t, const double*, double*, int);
template __global__ void k_eval_linear<float>(GridView, int64_t, const double*, double*, int);

template __global__ void k_eval_field<double, 0>(GridView, int64_t, const double*, double*, int);

// The multi-resolution grid at n positions (patch table staged in LDS).
template <class GT>
__global__ void k_eval_nested(GridView g, NestView nv, int64_t n, const double* pos, double* B,
                              int mode)
{
    __shared__ PatchView P[MAX_PATCHES];
    if ((int)threadIdx.x < nv.np)
        P[threadIdx.x] = nv.p[threadIdx.x];
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    NestedField<GT> F;
    F.g = g;
    F.P = P;
    F.np = nv.np;
    const double p[3] = {pos[3 * i], pos[3 * i + 1], pos[3 * i + 2]};
    if (mode == MODE_FP64) {
        double b[3];
        F.fp64(p, b);
        B[3 * i] = b[0];
        B[3 * i + 1] = b[1];
        B[3 * i + 2] = b[2];
    } else {
        float b[3];
        F.fp32(p, b);
        B[3 * i] = (double)b[0];
        B[3 * i + 1] = (double)b[1];
        B[3 * i + 2] = (double)b[2];
    }
}
template __global__ void k_eval_nested<double>(GridView, NestView, int64_t, const double*, double*,
                                               int);
template __global__ void k_eval_nested<float>(GridView, NestView, int64_t, const double*, double*,
                                              int);
template __global__ void k_eval_field<float, 0>(GridView, int64_t, const double*, double*, int);
template __global__ void k_eval_field<float, 1>(GridView, int64_t, const double*, double*, int);

// -------------------------------------------------------------------------
// The analytic field at n positions (FP64).
__global__ void k_eval_analytic(AnalyticParams a, int64_t n, const double* __restrict__ pos,
                                double* __restrict__ B)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    AnalyticFieldSrc F;
    F.a = a;
    const double p[3] = {pos[3 * i], pos[3 * i + 1], pos[3 * i + 2]};
    double b[3];
    F.fp64(p, b);
    B[3 * i] = b[0];
    B[3 * i + 1] = b[1];
    B[3 * i + 2] = b[2];
}

// -------------------------------------------------------------------------
// Diagnostic (not a step of the method): the field-gather pattern alone.
// Every wave repeatedly gathers the corner records of 64 pseudo-random cells
// with the propagation kernel's cooperative gather and folds one value of
// each into a checksum, so the rate it reaches is the practical ceiling of
// the field evaluation on this buffer.
// -------------------------------------------------------------------------
__device__ inline uint32_t mix32(uint32_t x)
{
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    x ^= x >> 16;
    return x;
}

__global__ void __launch_bounds__(128) k_gather_ceiling(const float* corner, uint32_t ncell,
                                                        int iters, float* sink)
{
    __shared__ float4 stage[2 * coop_stage_float4<float>];
    const int t = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    float* st = (float*)(stage + wave * coop_stage_float4<float>);
    uint32_t s = mix32((uint32_t)blockIdx.x * 128u + (uint32_t)t + 0x9e3779b9u);
    float acc = 0.0f;
    for (int it = 0; it < iters; ++it) {
        s = mix32(s + 0x9e3779b9u);
        const uint32_t cell = (uint32_t)(((uint64_t)s * ncell) >> 32);   // < ncell
        float v[8][3];
        coop_issue(corner, cell, st, true);
        coop_consume(st, v);
        acc += v[t & 7][0];
    }
    sink[(int64_t)blockIdx.x * 128 + t] = acc;
}

// -------------------------------------------------------------------------
// Corner-replicated layout: record of cell (i,j,k) = the 8 corner vectors
// (c = dx + 2 dy + 4 dz) of the linear grid, as 24 values of the grid's
// element type: FP32 padded to 128 bytes (32 floats), FP64 unpadded (192 bytes).
template <class GT>
__global__ void k_corner_relayout(GridView g, GT* out)
{
    constexpr int RL = sizeof(GT) == 8 ? 24 : 32;   // elements per record
    const int64_t ncell = (int64_t)g.n[0] * g.n[1] * g.n[2];
    const GT* G = (const GT*)g.data;
    for (int64_t cell = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; cell < ncell;
         cell += (int64_t)gridDim.x * blockDim.x) {
        const int k = (int)(cell % g.n[2]);
        const int j = (int)((cell / g.n[2]) % g.n[1]);
        const int i = (int)(cell / ((int64_t)g.n[1] * g.n[2]));
        GT rec[RL];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int ii = (i + (c & 1)) % g.n[0];
            const int jj = (j + ((c >> 1) & 1)) % g.n[1];
            const int kk = (k + ((c >> 2) & 1)) % g.n[2];
            const GT* p = G + (int64_t)ii * g.stride[0] + (int64_t)jj * g.stride[1] +
                          (int64_t)kk * 3;
            rec[3 * c] = p[0];
            rec[3 * c + 1] = p[1];
            rec[3 * c + 2] = p[2];
        }
#pragma unroll
        for (int q = 24; q < RL; ++q)
            rec[q] = (GT)0;
        if constexpr (sizeof(GT) == 8) {
            double2* o = (double2*)(out + cell * RL);
#pragma unroll
            for (int q = 0; q < RL / 2; ++q)
                o[q] = make_double2(rec[2 * q], rec[2 * q + 1]);
        } else {
            float4* o = (float4*)(out + cell * RL);
#pragma unroll
            for (int q = 0; q < RL / 4; ++q)
                o[q] = make_float4(rec[4 * q], rec[4 * q + 1], rec[4 * q + 2], rec[4 * q + 3]);
        }
    }
}
template __global__ void k_corner_relayout<float>(GridView, float*);
template __global__ void k_corner_relayout<double>(GridView, double*);

}  // namespace crp
