// The arrival-order commit kernel (template over diagnostics and constraint
// (d)).  Its instantiations are split over two translation units, so that the
// variants without decode history are compiled as they are without the others
// beside them.
#pragma once

#include "ald_device.h"

namespace ald {

// ---------------------------------------------------------------------------------------------
// Commit.  One wave per scenario walks the tile in arrival order, 64 queries (one
// group of the evaluation's bit words) at a time.  Each lane holds one worker:
// the workers committed to earlier in the tile ("changed") and, in the lanes
// left over, the best-ranked untouched workers that are feasible for some query
// of the group at tile start (their records are read in one go per group, so
// that no decision waits for a worker's figures).  A query is decided by one
// check per lane: for an untouched worker its tile-start bit is exact, for a
// changed one the bit, the latency checks on its current sums and the KV demand.
// Untouched workers beyond the lanes rank after those in them (by tile-start
// rank), and are searched, in rank order, only when they can matter.
//
// The KV demand of a changed worker is first bounded: from above by its last
// exact peak plus everything added since, from below by the demand at the
// iteration where that peak was.  Only between the bounds is it scanned exactly,
// on the worker's end-sorted columns, which are copied into an LDS pool at the
// first such scan and kept there.  A commit appends the request behind the
// worker's sorted columns in HBM (st.tn counts these) and updates the sums; the
// build kernel of the next round sorts the appended requests in.
//
// What bounds it: the chain of decisions (one wave, no parallelism over queries), so
// instructions, taken branches and round trips per decision.  Hence one straight
// block of about 125 instructions for the decisions that need nothing rare,
// single-lane changes by selects and v_writelane, stores only when a group ends,
// and ties told apart by 20 leading bits of the key.  Measured in cycles of the
// deciding wave: 600 to 700 per decision of that block (2,000 as one loop over
// every case), 2,800 to 5,300 where a scan is needed.  With diagnostics the exact
// peaks of the placements, 1,000 cycles each, are taken by all waves of the
// block when the group ends.

constexpr int DBITS_W = 2048;   // changed-worker bitmap words in LDS: scenarios of up to 65536 workers
constexpr int ORDER_W = 4096;   // workers whose rank order is kept in LDS
constexpr int POOL = 12800;     // pool entries (8 B each) for changed workers' columns
constexpr int POOL_SLACK = 48;  // entries a copied worker may grow by before it is copied again
static_assert(POOL >= HOT + POOL_SLACK, "the largest worker fits the pool");

// Orders LDS traffic between the lanes of one wave of the commit block
// without waiting for outstanding global memory operations.
__device__ __forceinline__ void wave_sync() { __builtin_amdgcn_wave_barrier(); }

// Branch hints: the decision loop is one wave's instruction stream, and every
// taken branch over a block that hardly ever runs stalls it.
// (a function of its own could not read the kernel's arguments)
#define ALD_INLINE __attribute__((always_inline))
#define ALD_LIKELY(x) __builtin_expect(!!(x), 1)
#define ALD_RARELY(x) __builtin_expect(!!(x), 0)

// Whether this lane is in the wave-uniform mask m.
__device__ __forceinline__ bool in_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
// Lanes of m below this one.
__device__ __forceinline__ int rank_in(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}
__device__ __forceinline__ int first_lane(uint64_t m) { return __builtin_ctzll(m); }  // (m != 0)

// A value that every lane holds alike, as a scalar: the compiler's analysis gives
// up on loop-carried values here, and without the hint the decision loop runs
// on vector registers and execution masks.
__device__ __forceinline__ int32_t uni(int32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint64_t uni(uint64_t x)
{
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(x >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)x);
}

// The leading bits of a rank key, in its order: the high word of its value as a
// double (20 bits after the leading one; distinct keys hardly ever share them).
__device__ __forceinline__ uint32_t key_lead(uint64_t key)
{
    return (uint32_t)(__builtin_bit_cast(uint64_t, (double)key) >> 32);
}

// The lane of the non-empty mask m whose (key, worker) ranks first by Algorithm
// 1's order (lead = key_lead(key), which nearly always decides).
__device__ __forceinline__ int best_lane(uint64_t m, uint32_t lead, uint64_t key, int32_t w)
{
    if ((m & (m - 1)) == 0) return first_lane(m);
    const uint32_t lm0 = wave_max_u32(in_mask(m) ? lead : 0u);
    m &= ballot(lead == lm0);
    if (ALD_RARELY((m & (m - 1)) != 0)) {
        const uint32_t hi = (uint32_t)(key >> 32), lo = (uint32_t)key;
        const uint32_t hm = wave_max_u32(in_mask(m) ? hi : 0u);
        m &= ballot(hi == hm);
        const uint32_t lm = wave_max_u32(in_mask(m) ? lo : 0u);
        m &= ballot(lo == lm);
        if (m & (m - 1)) {
            const int32_t wm = wave_min32(in_mask(m) ? w : INT32_MAX);
            m &= ballot(w == wm);
        }
    }
    return first_lane(m);
}

// The worker a lane holds: what every decision reads (the rest is in
// CommitLDS).  Single lanes are changed by v_writelane or a select, without a
// branch: a branch that changes some of these leaves the compiler copying all of
// them between registers at every decision.
struct Slot {
    int32_t w;       // scenario-local index, -1 = none
    int32_t B;       // live requests, appended ones included
    int32_t room;    // requests it can still take
    int32_t M;
    // Bounds of its KV peak without a new query: at most M - slack; its demand at
    // end iteration loe is at least M - loe - flo (so with a query that is alive
    // then, sq + loe more).
    int32_t slack, flo, loe;
    uint64_t key;
    uint32_t lead;   // key_lead(key)
    // sums as fp64 (integers below 2^53 and multiples of 2^-8 below 2^31: exact)
    double DS;       // sum of D = 2^-gs * State::DS
    double S1, S2;   // TTFT sums of this heartbeat
    double rhs;
    double dlim;     // constraint (d)'s limit, fixed within a heartbeat (no ongoing request joins or leaves)
};

// The kernel's arguments and its scenario, read where they are needed through a
// pointer that the compiler cannot see through: kept in registers over the
// decision loop, they overflow the scalar registers, and every use of a
// spilled one is an instruction more in the chain.
// (Pointers read this way have lost the knowledge that they are global, and a
// load through an unknown address counts as different per lane; gptr restores
// it.)
template <typename T>
__device__ __forceinline__ T* gptr(T* p)
{
    return (T*)(__attribute__((address_space(1))) T*)(uint64_t)p;
}
typedef const __attribute__((address_space(4))) State* StateArg;
typedef const __attribute__((address_space(4))) Scen* ScenArg;
__device__ __forceinline__ StateArg state_arg()
{
    StateArg p = (StateArg)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}
__device__ __forceinline__ ScenArg scen_arg()
{
    ScenArg p = (ScenArg)(uint64_t)state_arg()->scen + blockIdx.x;  // one block per scenario
    asm volatile("" : "+s"(p));
    return p;
}
__device__ __forceinline__ int64_t q_index(int32_t i)
{
    const int32_t* m = gptr(scen_arg()->qmap);
    return m != nullptr ? (int64_t)m[i] : (int64_t)i;
}
// A wave-uniform value kept in vector registers.
template <typename T>
__device__ __forceinline__ T in_vgpr(T x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// Waves per scenario: with diagnostics every placement needs its worker's exact KV
// peak, which no later decision waits for; the other waves compute them.
constexpr int commit_waves(bool diag) { return diag ? 8 : 1; }

struct CommitLDS {
    int32_t cw[64], cr[64];  // untouched workers picked for the free lanes: index, rank
    uint64_t cword[64];      // and bit word
    int32_t over_w, over_r;  // the first one there was no lane for
    // of the lanes' workers: place in the tile-start rank order, slot range and
    // the sorted live slots in it at tile start, log entries and slack gain
    // (constraint (d): a request placed now logs slack - phi = -phi)
    int64_t base[64];
    int32_t rk[64], head[64], n[64], cap[64], lgn[64];
    double phi[64];
    // and what the tile's requests add to their sums of c and r
    uint64_t dsc[64], dsr[64];
    // their columns in the pool (when copied): first entry, entries there is room
    // for, entries there are (the worker's first so many requests)
    int32_t off[64], room[64], have[64];
    // the changed workers, when dirty_w was last used (note_dirty)
    int32_t dw[MAX_DIRTY];
    uint32_t dbits[DBITS_W];
    int32_t order[ORDER_W];
    int32_t pe[POOL], ps[POOL];
};

// With diagnostics: what the waves of the block exchange.
struct PeakLDS {
    // the workers (by lane) whose placements of this group have no peak yet; 0: the
    // tile is done
    uint64_t jobs, fetch;  // fetch: of these, the ones whose columns must be copied first
    int32_t rl[64], rB[64], lin[64], lp[64];  // the group's placements (as in the kernel's registers)
    int32_t B[64];         // the workers' requests
    int32_t peak[64];      // results: each query's peak
    int32_t last[64];      // and each worker's peak after its last one
    double tt[64], td[64];  // the choices' prefill and decode times
    // short tiles: the waves' shares of the worker blocks' results
    struct Two {
        uint64_t a1, a2;
        int32_t nfeas, ntcnt;
    } two[commit_waves(true)][64];
};

// Has worker w (scenario-local) changed in this tile?  (any lane, any w; nd
// workers listed by note_dirty)
__device__ __forceinline__ bool dirty_w(const CommitLDS& L, int W, int nd, int w)
{
    if (W <= DBITS_W * 32) return (L.dbits[w >> 5] >> (w & 31)) & 1u;
    bool d = false;
    for (int j = 0; j < nd; ++j) d = d | (L.dw[j] == w);
    return d;
}

// Insert (x, y) into the sorted LDS columns e/s[0, B), after every entry with
// e <= x (whole wave; the columns must have room for B + 1 entries).
__device__ __forceinline__ void lds_sorted_insert(int32_t* e, int32_t* s, int B, int32_t x, int32_t y)
{
    const int lane = lane_id();
    int u = 0;
    for (int k0 = 0; k0 < B; k0 += COMMIT_THREADS) u += __popcll(ballot(k0 + lane < B) & ballot(e[min(k0 + lane, B - 1)] <= x));
    // shift [u, B) up by one, highest block first (each pass reads before it writes)
    for (int top = B; top > u; top -= COMMIT_THREADS) {
        const int k = top - COMMIT_THREADS + lane;
        const bool mv = k >= u && k < top;
        int32_t ve = 0, vs = 0;
        if (mv) {
            ve = e[k];
            vs = s[k];
        }
        wave_sync();
        if (mv) {
            e[k + 1] = ve;
            s[k + 1] = vs;
        }
        wave_sync();
    }
    if (lane == 0) {
        e[u] = x;
        s[u] = y;
    }
    wave_sync();
}

// KV demand of a worker from its sorted columns (B entries): the peak with the
// query added, the peak without, and the end iteration at which the latter
// falls.  Whole wave; every lane gets the result.  Beyond 128 slots lane l takes
// chunk 63 - l, so a prefix over lanes is a suffix over slots.  Every value is a KV demand below
// 2^31 (the worker's peak is at most 2^30, the query adds l_in + l_pred).
struct Peak {
    int32_t with, without, at;
};
__device__ __forceinline__ Peak wave_kv_peak(const int32_t* e, const int32_t* s, int B, int32_t sq, int32_t eq)
{
    const int lane = lane_id();
    Peak r;
    if (ALD_LIKELY(B <= 128)) {
        // one or two chunks of 64 slots, a lane per slot; the demand at the query's
        // own end is read off the sum over the slots that end no earlier
        int32_t best = INT32_MIN, best0 = 0, at = 0, sum = 0, own = 0;
        int ahead = B;  // slots ending before the query
#pragma unroll
        for (int c = 1; c >= 0; --c) {
            if (c * 64 >= B) continue;
            const int k = c * 64 + lane;
            const bool in = k < B;
            const int32_t ek = e[min(k, B - 1)], sk = in ? s[min(k, B - 1)] : 0;
            const int32_t inc = wave_incl_scan(sk, 0, Add32());
            const int32_t all = rdlane(inc, 63);
            const int32_t run = sum + all - inc + sk;  // sum of s over slots >= k
            sum += all;
            // (wrap-around arithmetic: the demand itself is below 2^31)
            const int32_t P = (int32_t)((uint32_t)run + (uint32_t)(B - k) * (uint32_t)ek);
            const uint64_t later = ballot(in) & ballot(ek >= eq);
            const int32_t val = ek < eq ? (int32_t)((uint32_t)P + (uint32_t)sq + (uint32_t)ek) : P;
            best = (in && val > best) ? val : best;
            at = (in && P > best0) ? ek : at;
            best0 = (in && P > best0) ? P : best0;
            if (later != 0) {
                ahead = c * 64 + first_lane(later);
                own = rdlane(run, first_lane(later));
            }
        }
        r.without = wave_max32(best0);
        r.at = rdlane(at, first_lane(ballot(best0 == r.without)));  // (some lane holds the maximum)
        const int32_t bmax = wave_max32(best);
        own = (int32_t)((uint32_t)own + (uint32_t)(B - ahead) * (uint32_t)eq + (uint32_t)sq + (uint32_t)eq);
        r.with = bmax > own ? bmax : own;
        return r;
    }
    const int CH = (B + 63) >> 6;
    const int c = 63 - lane;
    const int k0 = min(B, c * CH);
    const int k1 = min(B, k0 + CH);
    int32_t ls = 0;
    for (int k = k0; k < k1; ++k) ls += s[k];
    int32_t run = wave_incl_scan(ls, 0, Add32()) - ls;  // slots after this chunk
    int32_t best = INT32_MIN, best0 = 0, at = 0, ssge = 0, cge = 0;
    for (int k = k1 - 1; k >= k0; --k) {
        const int32_t ek = e[k], sk = s[k];
        run += sk;  // sum of s over slots >= k
        const int32_t P = (int32_t)((uint32_t)run + (uint32_t)(B - k) * (uint32_t)ek);
        const bool before = ek < eq;  // the query is still alive at this end point
        const int32_t val = before ? (int32_t)((uint32_t)P + (uint32_t)sq + (uint32_t)ek) : P;
        best = val > best ? val : best;
        at = P > best0 ? ek : at;
        best0 = P > best0 ? P : best0;
        ssge += before ? 0 : sk;
        cge += before ? 0 : 1;
    }
    r.without = wave_max32(best0);
    r.at = rdlane(at, first_lane(ballot(best0 == r.without)));
    const int32_t bmax = wave_max32(best);
    const int32_t own = (int32_t)((uint32_t)wave_sum32(ssge) + (uint32_t)wave_sum32(cge) * (uint32_t)eq +
                                  (uint32_t)sq + (uint32_t)eq);
    r.with = bmax > own ? bmax : own;
    return r;
}

// The same with the query's request put into the columns (room for B + 1): its
// peak with the query.
__device__ __forceinline__ int32_t wave_peak_insert(int32_t* e, int32_t* s, int B, int32_t sq, int32_t eq)
{
    const int lane = lane_id();
    if (ALD_RARELY(B > 128)) {
        const int32_t with = wave_kv_peak(e, s, B, sq, eq).with;
        lds_sorted_insert(e, s, B, eq, sq);
        return with;
    }
    int32_t ek[2], sk[2], inc[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int k = min(c * 64 + lane, max(B - 1, 0));
        ek[c] = e[k];
        sk[c] = s[k];
    }
    uint64_t later[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const bool in = c * 64 + lane < B;
        sk[c] = in ? sk[c] : 0;
        later[c] = ballot(in) & ballot(ek[c] >= eq);
        inc[c] = wave_incl_scan(sk[c], 0, Add32());
    }
    const int ahead = later[0] != 0 ? first_lane(later[0]) : (later[1] != 0 ? 64 + first_lane(later[1]) : B);
    const int32_t all0 = rdlane(inc[0], 63), all1 = rdlane(inc[1], 63);
    const int32_t run0 = all1 + all0 - inc[0] + sk[0], run1 = all1 - inc[1] + sk[1];  // sums of s over slots >= k
    const int32_t later_s = later[0] != 0 ? rdlane(run0, first_lane(later[0]))
                                          : (later[1] != 0 ? rdlane(run1, first_lane(later[1])) : 0);
    // (wrap-around arithmetic: the demands themselves are below 2^31)
    int32_t best = (int32_t)((uint32_t)later_s + (uint32_t)(B - ahead) * (uint32_t)eq + (uint32_t)sq + (uint32_t)eq);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int k = c * 64 + lane;
        const uint32_t P = (uint32_t)(c ? run1 : run0) + (uint32_t)(B - k) * (uint32_t)ek[c];
        const int32_t val = (int32_t)(P + (ek[c] < eq ? (uint32_t)sq + (uint32_t)ek[c] : 0u));
        best = k < B && val > best ? val : best;
    }
    wave_sync();
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int k = c * 64 + lane;
        if (k >= ahead && k < B) {
            e[k + 1] = ek[c];
            s[k + 1] = sk[c];
        }
    }
    if (lane == 0) {
        e[ahead] = eq;
        s[ahead] = sq;
    }
    wave_sync();
    return wave_max32(best);
}

// A fresh read of data that another lane of this wave wrote earlier in the
// launch (the caller has waited for the wave's stores).
__device__ __forceinline__ int32_t coherent(const int32_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// the control block as the host will read it (after the stream synchronises)
__device__ __forceinline__ void publish_ctl(const Ctl& c)
{
    const StateArg st = state_arg();
    if (st->ctl_host != nullptr) gptr(st->ctl_host)[blockIdx.x] = c;
    if (st->status != nullptr) *gptr(st->status) = ctl_status(c);
}

// Copies the columns of the worker of lane j into the pool (its sorted slots at
// tile start).  One wave.
__device__ __forceinline__ void copy_columns(CommitLDS& L, int j)
{
    constexpr int NT = COMMIT_THREADS;
    const int lane = lane_id();
    const StateArg st = state_arg();
    const int off = uni(L.off[j]), head = uni(L.head[j]), B0 = uni(L.n[j]) - head;
    const int64_t base = (int64_t)uni((uint64_t)L.base[j]);
    const int32_t* const ge = gptr(st->e) + base + head;
    const int32_t* const gs_ = gptr(st->s) + base + head;
    for (int k0 = 0; k0 < B0; k0 += 4 * NT) {
        int32_t ve[4], vs[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = min(k0 + u * NT + lane, B0 - 1);
            ve[u] = ge[k];
            vs[u] = gs_[k];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = k0 + u * NT + lane;
            if (k < B0) {
                L.pe[off + k] = ve[u];
                L.ps[off + k] = vs[u];
            }
        }
    }
    if (lane == 0) L.have[j] = B0;
    wave_sync();
}

// Brings the columns of lane j's worker (in the pool) up to its B requests: those
// of earlier groups from HBM, this group's from its lanes (rl, rB, lin, lp as
// in the kernel), with diagnostics computing their peaks on the way; the last of
// these is returned (-1: none).  One wave; the earlier groups' stores have left.
template <bool DIAG>
__device__ __forceinline__ int32_t advance_columns(CommitLDS& L, int32_t* peak, int j, int B, int32_t tau, int32_t rl,
                                                   int32_t rB, int32_t lin, int32_t lp)
{
    const StateArg st = state_arg();
    const int lane = lane_id();
    const int off = uni(L.off[j]);
    int at = uni(L.have[j]);
    int32_t with = -1;
    if (at >= B) return with;
    const uint64_t here = ballot(rl == j) & ballot(rB >= at);
    const int upto = B - __popcll(here);
    if (ALD_RARELY(at < upto)) {
        const int head = uni(L.head[j]), cap = uni(L.cap[j]);
        const int64_t base = (int64_t)uni((uint64_t)L.base[j]);
        for (; at < upto; ++at) {
            int p = head + at;
            p = p > cap ? p - (cap + 1) : p;
            const int32_t x = coherent(gptr(st->e) + base + p), y = coherent(gptr(st->s) + base + p);
            lds_sorted_insert(L.pe + off, L.ps + off, at, uni(x), uni(y));
        }
    }
    for (uint64_t m = here; m != 0; m &= m - 1, ++at) {
        const int p = first_lane(m);
        const int32_t eq = rdlane(lp, p) + tau, sq = rdlane(lin, p) - tau;
        if (DIAG) {
            with = wave_peak_insert(L.pe + off, L.ps + off, at, sq, eq);
            if (lane == 0) peak[p] = with;
        } else {
            lds_sorted_insert(L.pe + off, L.ps + off, at, eq, sq);
        }
    }
    if (lane == 0) L.have[j] = B;
    wave_sync();
    return with;
}

// This wave's share of the group's jobs (PeakLDS).
__device__ __forceinline__ void run_jobs(CommitLDS& L, PeakLDS& P, int wave, int32_t tau)
{
    const int lane = lane_id();
    const int32_t rl = P.rl[lane], rB = P.rB[lane], lin = P.lin[lane], lp = P.lp[lane];
    const uint64_t jobs = uni(P.jobs), fetch = uni(P.fetch);
    int i = 0;
    uint64_t mine = 0;
    for (uint64_t m = jobs; m != 0; m &= m - 1, ++i)
        if (i % commit_waves(true) == wave) mine |= m & (0 - m);
    for (uint64_t m = mine & fetch; m != 0; m &= m - 1) copy_columns(L, first_lane(m));
    for (uint64_t m = mine; m != 0; m &= m - 1) {
        const int j = first_lane(m);
        const int32_t with = advance_columns<true>(L, P.peak, j, uni(P.B[j]), tau, rl, rB, lin, lp);
        if (lane == 0) P.last[j] = with;
    }
}

template <bool DIAG, bool USE_D>
__global__ __launch_bounds__(COMMIT_THREADS * commit_waves(DIAG)) void k_commit(State)
{
    constexpr int NT = COMMIT_THREADS;  // the deciding wave
    constexpr int NWV = commit_waves(DIAG);
    const int lane = lane_id();
    const int wave = uni(wave_id());
    Ctl* const cp = gptr(state_arg()->ctl) + blockIdx.x;
    const Ctl c = *cp;
    {
        const StateArg st = state_arg();
        if (c.call != st->call) {  // another call's control block: this call was blocked
            if (st->status != nullptr && threadIdx.x == 0) *gptr(st->status) = ALD_EBLOCKED;
            return;
        }
        const bool qbad = gptr(st->qbad) != nullptr && *gptr(st->qbad) != 0;
        if (qbad || c.err || c.start >= c.Q) {
            if (threadIdx.x == 0) {
                Ctl o = c;
                if (qbad) {  // an invalid query length: nothing is written
                    o.err = DEV_EINVAL;
                    cp->err = DEV_EINVAL;
                }
                publish_ctl(o);
            }
            return;
        }
    }
    const int32_t start = c.start, end = tile_end(c.start, c.Q, c.T, c.H, c.since_hb, c.hb_next);
    const int32_t fpc = min(gptr(state_arg()->tinfo)[blockIdx.x].first_pc, end);
    const int32_t empty_rank = gptr(state_arg()->tinfo)[blockIdx.x].empty_rank;
    const int32_t tau = c.tau, hb = c.hb_index;
    const int W = scen_arg()->W;
    const int groups = (end - start + 63) >> 6;
    const bool sorted = gptr(state_arg()->qpos) != nullptr;

    __shared__ CommitLDS L;
    __shared__ std::conditional_t<DIAG, PeakLDS, char> peak_lds;
    PeakLDS& P = reinterpret_cast<PeakLDS&>(peak_lds);  // (only touched with diagnostics)
    const bool lds_order = W <= ORDER_W;
    if (fpc < end) {
        if (W <= DBITS_W * 32)
            for (int k = threadIdx.x; k < (W + 31) / 32; k += NT * NWV) L.dbits[k] = 0u;
        if (lds_order) {
            const int32_t* const order = gptr(state_arg()->order) + scen_arg()->wbase;
            for (int k0 = 0; k0 < W; k0 += 4 * NT * NWV) {
                int32_t v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = order[min(k0 + u * NT * NWV + (int)threadIdx.x, W - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int k = k0 + u * NT * NWV + threadIdx.x;
                    if (k < W) L.order[k] = v[u];
                }
            }
        }
    }
    // short tiles with diagnostics: the commit merges the worker blocks' results
    // per query itself and writes every query's diagnostics (else the selection
    // wrote those of the queries that no worker can take).  shares waves take a
    // group's blocks between them.
    const bool brief = DIAG && state_arg()->brief != 0;
    static_assert(SHORT_TILE <= 64 * commit_waves(true), "a wave per group at least");
    const int shares = NWV / max(min(groups, NWV), 1);
    if (brief && wave < groups * shares) {
        const int64_t stride = scen_arg()->pstride;
        const int t = wave / shares * 64 + lane;
        const ulonglong2* row = gptr(state_arg()->part) + scen_arg()->part_off + 2 * (int64_t)(t < end - start ? t : 0);
        PeakLDS::Two r{~0ull, ~0ull, 0, 0};
        const int nblk = scen_arg()->nblk;
#pragma unroll 8
        for (int b = wave % shares; b < nblk; b += shares) {
            const ulonglong2 x = row[2 * b * stride], y = row[2 * b * stride + 1];
            merge_two(r.a1, r.a2, x.x, x.y);
            r.nfeas += (int32_t)y.x;
            r.ntcnt += (int32_t)y.y;
        }
        P.two[wave][lane] = r;
    }
    if (wave == 0) L.dsc[lane] = L.dsr[lane] = 0;
    if (NWV > 1) {
        __syncthreads();
        if (wave != 0) {
            for (;;) {  // the deciding wave posts jobs until the tile is done
                __syncthreads();
                if (uni(P.jobs) == 0) return;
                run_jobs(L, P, wave, tau);
                __syncthreads();
            }
        }
    }
    wave_sync();

    uint64_t dm = 0;      // lanes holding changed workers
    uint64_t cached = 0;  // lanes whose worker's columns are in the pool
    int pool_at = 0;
    Slot a;
    a.w = -1;
    a.B = a.room = a.M = a.slack = a.flo = 0;
    a.loe = INT32_MAX;
    a.key = 0;
    a.lead = 0;
    a.DS = a.S1 = a.S2 = a.rhs = 0.0;
    a.dlim = INFINITY;
    // the model's coefficients, in vector registers (the decision loop has no
    // scalar registers to spare)
    const double k2 = in_vgpr(scen_arg()->k2), c1 = in_vgpr(scen_arg()->c1), k1 = in_vgpr(scen_arg()->k1);
    const double k1q = in_vgpr(scen_arg()->k1q), ttft = in_vgpr(scen_arg()->ttft);
    const double theta = in_vgpr(scen_arg()->theta), c2 = in_vgpr(scen_arg()->c2), c3 = in_vgpr(scen_arg()->c3);
    const double dmax = in_vgpr(scen_arg()->tdec - scen_arg()->c3);
    const double up = in_vgpr(ldexp(1.0, scen_arg()->gs)), down = in_vgpr(ldexp(1.0, -scen_arg()->gs));
    const uint32_t gs = in_vgpr(scen_arg()->gs);

    auto rhs_of = [&](int B) { return theta * (dmax - c2 * (double)(B + 1)); };
    // the lanes where `in` holds take worker w (any valid index elsewhere) as at
    // tile start (its columns and sums are as built)
    auto load_slot = [&](bool in, int w, int rk) ALD_INLINE {
        const StateArg st = state_arg();
        const int gw = scen_arg()->wbase + w;
        const int32_t n = gptr(st->n)[gw], head = gptr(st->head)[gw], cap = gptr(st->cap)[gw];
        const int32_t M = gptr(st->M)[gw], peak = gptr(st->peak)[gw], loe = gptr(st->peake)[gw];
        const int64_t base = gptr(st->slot_base)[gw];
        const uint64_t key = gptr(st->key)[gw];
        const int64_t ds = gptr(st->DS)[gw], s1 = gptr(st->S1)[gw], s2 = gptr(st->S2)[gw];
        const bool cur = gptr(st->hbs)[gw] == hb;
        double dlim = INFINITY, phi = 0.0;
        int32_t lgn = 0;
        if (USE_D) {
            dlim = gptr(st->dlim)[gw];
            phi = gptr(st->phi)[gw];
            lgn = gptr(st->lgn)[gw];
        }
        a.w = in ? w : a.w;
        a.B = in ? n - head : a.B;
        a.room = in ? cap - (n - head) : a.room;
        a.M = in ? M : a.M;
        a.slack = in ? M - peak : a.slack;
        a.loe = in ? loe : a.loe;
        a.flo = in ? (int32_t)((uint32_t)(M - peak) - (uint32_t)loe) : a.flo;
        a.key = in ? key : a.key;
        a.lead = in ? key_lead(key) : a.lead;
        a.DS = in ? (double)ds * down : a.DS;
        a.S1 = in ? (cur ? (double)s1 : 0.0) : a.S1;
        a.S2 = in ? (cur ? (double)s2 : 0.0) : a.S2;
        a.rhs = in ? rhs_of(n - head) : a.rhs;
        if (USE_D) a.dlim = in ? dlim : a.dlim;
        if (in) {
            L.base[lane] = base;
            L.rk[lane] = rk;
            L.head[lane] = head;
            L.n[lane] = n;
            L.cap[lane] = cap;
            if (USE_D) {
                L.lgn[lane] = lgn;
                L.phi[lane] = phi;
            }
        }
    };
    // (per lane, within a group) the lane that this lane's query was committed to
    // (-1: none yet), and the requests its worker held before
    int32_t rl = -1, rB = 0;
    // room in the pool for lane j's columns: false if it has to be cleared first
    auto reserve = [&](int j) ALD_INLINE -> bool {
        const int room = rdlane(a.B, j) + POOL_SLACK;
        if (pool_at + room > POOL) return false;
        if (lane == 0) {
            L.off[j] = pool_at;
            L.room[j] = room;
        }
        pool_at += room;
        cached |= 1ull << j;
        return true;
    };
    // exact KV demand of lane j's worker with the query; the lane's bounds become
    // exact (lin, lp: the group's queries)
    auto scan = [&](int j, int32_t sq, int32_t eq, int32_t lin, int32_t lp) ALD_INLINE -> int32_t {
        cached = uni(cached);
        pool_at = uni(pool_at);
        wave_sync();
        const int B = rdlane(a.B, j);
        if (ALD_RARELY(!((cached >> j) & 1) || B > uni(L.room[j]))) {
            if (!reserve(j)) {  // full: every copy is dropped (HBM holds what they were made from)
                cached = 0;
                pool_at = 0;
                reserve(j);
            }
            wave_sync();
            copy_columns(L, j);
        }
        if (uni(L.have[j]) < B) {
            __builtin_amdgcn_s_waitcnt(0);  // earlier groups' appends have left
            advance_columns<DIAG>(L, P.peak, j, B, tau, rl, rB, lin, lp);
        }
        const int off = uni(L.off[j]);
        const Peak r = wave_kv_peak(L.pe + off, L.ps + off, B, sq, eq);
        const int32_t slack = rdlane(a.M, j) - r.without;
        a.slack = ald_writelane(slack, j, a.slack);
        a.loe = ald_writelane(r.at, j, a.loe);
        a.flo = ald_writelane(slack - r.at, j, a.flo);
        return r.with;
    };
    // (a changed worker's mark is set when someone looks: a decision only adds its
    // lane to dm)
    uint64_t noted = 0;
    auto note_dirty = [&]() ALD_INLINE {
        const uint64_t fresh = dm & ~noted;
        if (fresh != 0) {
            if (W <= DBITS_W * 32) {
                if (in_mask(fresh)) atomicOr(&L.dbits[a.w >> 5], 1u << (a.w & 31));
            } else if (in_mask(dm)) {
                L.dw[rank_in(dm)] = a.w;
            }
            noted = dm;
            wave_sync();
        }
    };

    int pos = brief ? start : fpc;
    // why the tile was cut (0: not)
    constexpr int CUT_STALE = 1, CUT_SLOTS = 2, CUT_PAIR = 3, CUT_LANES = 4;
    int cut = 0;
    int32_t full_w = -1;  // (CUT_SLOTS) the worker without one
    int commits = 0;
    int nrej = pos - start;  // the rejected prefix
    int firstrej = pos > start ? start : INT32_MAX;
    // its outputs (with diagnostics the selection wrote them)
    int32_t* out = gptr(state_arg()->out_worker);
    if (out != nullptr) out += scen_arg()->out_off;
    if (!DIAG && out != nullptr)
        for (int i = start + lane; i < fpc; i += NT) out[q_index(i)] = -1;
    // Work that only a fresh tile would have spared: changed workers that took
    // an exact scan and turned out full, and queries that every changed worker
    // turned away.  Past a budget a fresh tile is the cheaper way on, and the
    // tile is cut before the next decision.
    int stale = 0;
    int gany = -64;       // (arrival layout) lane l holds the word of group gany + l
    uint64_t anyv = 0;
    while (uni(pos) < end && uni(cut) == 0) {
        pos = uni(pos);
        dm = uni(dm);
        // one group of 64 queries; those before pos are decided
        const int g = (pos - start) >> 6;
        const int w0 = start + g * 64;
        const int i = w0 + lane;
        const bool act = i >= pos && i < end;
        const uint64_t actm = ballot(act);
        // the tile position of this lane's query: its own offset, or in the
        // sorted layout where the pair evaluation put it (the bit words are kept
        // by position)
        int tp = i - start;
        uint64_t potm;  // queries with a feasible worker at tile start
        {
            const uint64_t* const any = gptr(state_arg()->any) + scen_arg()->any_off;
            if (sorted) {
                tp = act ? gptr(state_arg()->qpos)[i - start] : 0;
                potm = ballot(act && ((any[tp >> 6] >> (tp & 63)) & 1));
            } else {
                if (g - gany >= 64) {
                    gany = g;
                    anyv = g + lane < groups ? any[g + lane] : 0;
                }
                potm = rdlane64(anyv, g - gany) & actm;
            }
        }
        if (potm == 0 && !brief && (!DIAG || dm == 0)) {  // all rejected, whatever the tile committed
            if (!DIAG && act && out != nullptr) out[q_index(i)] = -1;
            if (firstrej == INT32_MAX) firstrej = w0 + first_lane(actm);
            nrej += __popcll(actm);
            pos = min(end, w0 + NT);
            continue;
        }
        int32_t lin = 1, lp = 1;
        QSum q;
        q.nfeas = q.ntcnt = 0;
        q.ex1 = q.ex2 = INT32_MAX;
        q.w1 = q.w2 = -1;
        if (act) {
            const int64_t k = q_index(i);
            lin = gptr(state_arg()->q_lin)[k];
            lp = gptr(state_arg()->q_lpred)[k];
            if (DIAG && !brief) q = gptr(state_arg()->qsum)[scen_arg()->qsum_off + (i - start)];
        }
        if (brief) {
            uint64_t a1 = ~0ull, a2 = ~0ull;
            for (int v = g * shares; v < (g + 1) * shares; ++v) {
                const PeakLDS::Two x = P.two[v][lane];
                merge_two(a1, a2, x.a1, x.a2);
                q.nfeas += x.nfeas;
                q.ntcnt += x.ntcnt;
            }
            ex_unpack(a1, q.ex1, q.w1);
            ex_unpack(a2, q.ex2, q.w2);
            if (!act) q.nfeas = q.ntcnt = 0;
        }
        const double qd = (double)(((int64_t)lin << gs) + (int64_t)scen_arg()->gn * lp) * down;

        // the group's bit word of this lane's worker w (all lanes call it)
        auto word_of = [&](const uint64_t* bits, int w) ALD_INLINE -> uint64_t {
            const uint64_t* col = bits + scen_arg()->bits_off + w;
            if (!sorted) return col[(int64_t)g * W];
            uint64_t r = 0;
            for (int q0 = 0; q0 < 64; q0 += 8) {
                uint64_t v[8];
                int t[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    t[u] = rdlane(tp, q0 + u);
                    v[u] = col[(int64_t)(t[u] >> 6) * W];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) r |= ((v[u] >> (t[u] & 63)) & 1) << (q0 + u);
            }
            return r & actm;
        };
        // (of the workers from rank empty_rank on, which hold no request, the first
        // one's words are every one's)
        auto bits_at = [&](int r) {
            r = DIAG ? r : min(r, empty_rank);
            return lds_order ? L.order[r] : (gptr(state_arg()->order) + scen_arg()->wbase)[r];
        };
        auto worker_at = [&](int r) {
            return lds_order ? L.order[r] : (gptr(state_arg()->order) + scen_arg()->wbase)[r];
        };
        // the first untouched worker at or after rank r0 whose bit for query t's
        // position is set (-1: none), and its rank
        auto first_untouched = [&](const uint64_t* bits, int t, int r0, int& fr) ALD_INLINE -> int {
            const uint64_t* row = bits + scen_arg()->bits_off + (int64_t)(t >> 6) * W;
            note_dirty();
            const int nd = __popcll(dm);
            constexpr int U = 4;  // reads in flight
            for (; r0 < W; r0 += NT * U) {
                int32_t w[U];
                uint64_t v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    w[u] = worker_at(min(r0 + u * NT + lane, W - 1));
                    v[u] = row[bits_at(min(r0 + u * NT + lane, W - 1))];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool in = r0 + u * NT + lane < W;
                    const uint64_t hit = ballot(in && ((v[u] >> (t & 63)) & 1) && !dirty_w(L, W, nd, w[u]));
                    if (hit) {
                        const int l = first_lane(hit);
                        fr = r0 + u * NT + l;
                        return rdlane(w[u], l);
                    }
                }
            }
            return -1;
        };

        // ---- the lanes of this group
        uint64_t wbf = 0, wbn = 0;  // bit words of this lane's worker: feasibility, near ties
        bool over = false;          // untouched feasible workers are left beyond the lanes:
        int over_w = -1, over_r = 0;  // the best-ranked one
        uint64_t over_key = 0;
        if (potm != 0) {
            const uint64_t* const bits = gptr(state_arg()->bits_feas);
            note_dirty();
            const int nd = __popcll(dm), nfree = NT - nd;
            int cnt = 0;
            constexpr int U = 4;
            for (int r0 = 0; r0 < W && uni(cnt) <= nfree; r0 += NT * U) {
                int32_t wl[U];
                uint64_t wd[U];
#pragma unroll
                for (int u = 0; u < U; ++u) wl[u] = worker_at(min(r0 + u * NT + lane, W - 1));
#pragma unroll
                for (int u = 0; u < U; ++u)
                    wd[u] = r0 + u * NT < W ? word_of(bits, bits_at(min(r0 + u * NT + lane, W - 1))) : 0;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (r0 + u * NT >= W) break;
                    bool ok = r0 + u * NT + lane < W && (wd[u] & potm) != 0;
                    if (dm != 0) ok = ok && !dirty_w(L, W, nd, wl[u]);
                    const uint64_t nz = ballot(ok);
                    const int k = cnt + rank_in(nz);
                    if (ok && k < nfree) {
                        L.cw[k] = wl[u];
                        L.cr[k] = r0 + u * NT + lane;
                        L.cword[k] = wd[u];
                    } else if (ok && k == nfree) {
                        L.over_w = wl[u];
                        L.over_r = r0 + u * NT + lane;
                    }
                    cnt += __popcll(nz);
                }
            }
            wave_sync();
            cnt = uni(cnt);
            over = cnt > nfree;
            if (over) {
                over_w = __builtin_amdgcn_readfirstlane(L.over_w);
                over_r = __builtin_amdgcn_readfirstlane(L.over_r);
                over_key = gptr(state_arg()->key)[scen_arg()->wbase + over_w];
            }
            cached &= dm;  // (an untouched worker's columns go with its lane)
            const int k = rank_in(~dm);
            const bool pick = in_mask(~dm) && k < min(cnt, nfree);
            a.w = in_mask(~dm) ? -1 : a.w;
            load_slot(pick, pick ? L.cw[k] : 0, pick ? L.cr[k] : 0);
            wbf = pick ? L.cword[k] : 0;
            if (dm != 0) {
                const uint64_t v = word_of(bits, bits_at(in_mask(dm) ? L.rk[lane] : 0));
                if (in_mask(dm)) wbf = v;
            }
        }
        const bool ties = DIAG && ballot(act && q.ntcnt > 0) != 0;  // some query of the group has near ties
        if (ties) {
            const uint64_t v = word_of(gptr(state_arg()->bits_nt), max(a.w, 0));
            wbn = a.w >= 0 ? v : 0;
        }
        // (diagnostics) this lane's query's results: as at tile start until its turn
        int32_t d_feas = q.nfeas, d_near = q.ntcnt > 0 ? 1 : 0, d_ex = q.ex1;
        // and whether the workers of its two smallest excesses have changed
        int32_t hit1 = 0, hit2 = 0;
        if (DIAG && dm != 0) {
            note_dirty();
            hit1 = q.w1 >= 0 && dirty_w(L, W, __popcll(dm), q.w1) ? 1 : 0;
            hit2 = q.w2 >= 0 && dirty_w(L, W, __popcll(dm), q.w2) ? 1 : 0;
        }
        // the smallest excess of query p, whose best worker has changed but not the
        // second best
        auto excess = [&](int p, int32_t sq, int32_t eq) ALD_INLINE -> int32_t {
            const int32_t x2 = rdlane(q.ex2, p), w2 = rdlane(q.w2, p);
            const int j = first_lane(dm & ballot(a.w == rdlane(q.w1, p)));
            // (commits only raise a demand: a floor at or above the second smallest
            // leaves that one)
            if (w2 >= 0 && rdlane(a.loe, j) <= eq && (int64_t)sq - rdlane(a.flo, j) >= x2) return x2;
            const int32_t now = scan(j, sq, eq, lin, lp) - rdlane(a.M, j);
            stale += 1;
            return (w2 < 0 || now < x2) ? now : x2;
        };

        rl = -1;
        int lim = NT;      // queries of lanes below lim are decided when the group ends (the tile is cut there)
        // queries left to decide (with diagnostics, once a worker has changed,
        // the rejected ones too)
        uint64_t todo = (DIAG && dm != 0) ? actm : potm;
        const uint64_t nearm = DIAG ? ballot(q.ntcnt > 0) : 0;
        while (uni(todo) != 0) {
            todo = uni(todo);
            dm = uni(dm);
            cached = uni(cached);
            stale = uni(stale);
            // ---- the decisions that need no scan, no look at the workers beyond the
            // lanes and no tie rule: one straight block per decision, left at the
            // first query that does
            if (ALD_LIKELY(stale < STALE_CUT) && (!DIAG || dm != 0)) {
                const uint32_t over_lead = key_lead(over_key);
                uint64_t t = todo;
                uint64_t hitm = DIAG ? ballot(hit1 != 0) | nearm : 0;
                do {
                    const int p = first_lane(t);
                    const int32_t plin = rdlane(lin, p), plp = rdlane(lp, p);
                    const double pqd = rdlane_f64(qd, p), dlin = (double)plin;
                    const int32_t eq = plp + tau, sq = plin - tau;
                    // this lane's worker with the query added: (b), then (c) and (d)
                    const double DS = a.DS + pqd, S1 = a.S1 + dlin, S2 = a.S2 + dlin * dlin;
                    const double lhs = k2 * DS, tt = (c1 + k1 * S1) + k1q * S2;
                    const uint64_t fsm = ballot((wbf >> p) & 1);
                    uint64_t cand = fsm & ballot(lhs <= a.rhs) & ballot(tt <= ttft);
                    if (USE_D) cand &= ballot(a.dlim == INFINITY || tt <= a.dlim);
                    // (changed workers: surely feasible, surely not, or to be scanned)
                    cand &= ~(dm & ballot(a.loe <= eq) & ballot(sq > a.flo));
                    const uint64_t unsure = dm & ~ballot(plin + plp <= a.slack);
                    // the best rank by the keys' leading bits; among equal ones the first
                    // lane if all are untouched (these are in rank order)
                    const uint32_t top = wave_max_u32(in_mask(cand) ? a.lead : 0u);
                    const uint64_t m = cand & ballot(a.lead == top);
                    const uint64_t bit = m & (0 - m);
                    bool rare = (m == 0) | (((m ^ bit) != 0) & ((m & dm) != 0)) | (over & (top <= over_lead));
                    rare = rare | (((DIAG ? cand : bit) & unsure) != 0) | ((bit & ballot(a.room <= 0)) != 0);
                    if (DIAG) {
                        uint64_t tied = ballot(near_tie(lhs, a.rhs)) | (ballot(ttft != INFINITY) & ballot(near_tie(tt, ttft)));
                        if (USE_D) tied |= ballot(a.dlim != INFINITY) & ballot(near_tie(tt, a.dlim));
                        // (a rejected query is looked at in the slow path too)
                        rare = rare | ((tied & dm) != 0) | (((hitm >> p) & 1) != 0);
                    }
                    if (ALD_RARELY(rare)) break;
                    const int bl = first_lane(bit);
                    const int32_t B0 = rdlane(a.B, bl);
                    const bool sel = in_mask(bit);
                    if (DIAG) {
                        const int more = __popcll(dm & cand) - __popcll(dm & fsm);
                        d_feas = ald_writelane(rdlane(d_feas, p) + more, p, d_feas);
                        const double td = (c3 + c2 * (double)(B0 + 1)) + lhs;
                        if (sel) {
                            P.tt[p] = tt;
                            P.td[p] = td;
                        }
                        const int32_t bw = rdlane(a.w, bl);
                        hitm |= ballot(q.w1 == bw);
                        hit1 |= q.w1 == bw ? 1 : 0;
                        hit2 |= q.w2 == bw ? 1 : 0;
                    }
                    dm |= bit;
                    rl = ald_writelane(bl, p, rl);
                    rB = ald_writelane(B0, p, rB);
                    // (B <= 8192, gs <= 8; a sum beyond the range fails the call)
                    const uint32_t X = (uint32_t)(B0 + 1) << gs, D = (uint32_t)(DS * up);
                    a.B += sel ? 1 : 0;
                    a.room -= sel ? 1 : 0;
                    a.slack -= sel ? plin + plp : 0;
                    a.flo -= sel && a.loe <= eq ? sq + a.loe : 0;
                    a.DS = sel ? DS : a.DS;
                    const uint64_t key = (uint64_t)X * X + (uint64_t)D * D;
                    a.key = sel ? key : a.key;
                    a.lead = sel ? key_lead(key) : a.lead;
                    a.rhs = sel ? rhs_of(B0 + 1) : a.rhs;
                    a.S1 = sel ? S1 : a.S1;
                    a.S2 = sel ? S2 : a.S2;
                    t = uni(t & (t - 1));
                    if (ALD_RARELY(dm == ~0ull)) break;
                } while (t != 0);
                todo = uni(t);
                dm = uni(dm);
                if (ALD_RARELY(dm == ~0ull)) {  // every lane holds a changed worker
                    const int past = 64 - __builtin_clzll(ballot(rl >= 0));  // the last one placed made it so
                    if (w0 + past < end) {
                        cut = CUT_LANES;
                        lim = past;
                        todo = 0;
                    }
                }
                if (todo == 0) continue;
            }
            const int p = first_lane(todo);
            if (ALD_RARELY(stale >= STALE_CUT)) {
                lim = p;
                cut = CUT_STALE;
                todo = 0;
                continue;
            }
            if (DIAG && ALD_LIKELY(dm != 0)) {
                // queries rejected at tile start, up to the next that is not: nothing
                // commits between them, so a lane takes its own query against each
                // changed worker, unless they are few for that
                const uint64_t pots = todo & potm;
                uint64_t seg = todo & ~potm & (pots != 0 ? (pots & (0 - pots)) - 1 : ~0ull);
                if (ALD_RARELY(seg != 0) && __popcll(dm) <= 2 * __popcll(seg)) {
                    // (both smallest excesses' workers changed: the tile-start pair cannot decide)
                    const uint64_t pair = seg & ballot(hit1 != 0) & ballot(hit2 != 0);
                    if (pair != 0) seg &= (pair & (0 - pair)) - 1;
                    const double dl = (double)lin;
                    int32_t nt = 0, clean = q.ntcnt;
                    for (uint64_t m = dm; m != 0; m &= m - 1) {
                        const int j = first_lane(m);
                        const double lhs = k2 * (rdlane_f64(a.DS, j) + qd), rhs = rdlane_f64(a.rhs, j);
                        const double tt = (c1 + k1 * (rdlane_f64(a.S1, j) + dl)) + k1q * (rdlane_f64(a.S2, j) + dl * dl);
                        nt |= (int32_t)near_tie(lhs, rhs) | ((int32_t)(ttft != INFINITY) & (int32_t)near_tie(tt, ttft));
                        if (USE_D) {
                            const double dlim = rdlane_f64(a.dlim, j);
                            nt |= (int32_t)(dlim != INFINITY) & (int32_t)near_tie(tt, dlim);
                        }
                        if (ties) clean -= in_mask(rdlane64(wbn, j)) ? 1 : 0;
                    }
                    d_near = in_mask(seg) ? ((nt != 0 || clean > 0) ? 1 : 0) : d_near;
                    for (uint64_t m = seg & ballot(hit1 != 0); m != 0; m &= m - 1) {
                        const int p1 = first_lane(m);
                        d_ex = ald_writelane(excess(p1, rdlane(lin, p1) - tau, rdlane(lp, p1) + tau), p1, d_ex);
                    }
                    todo &= ~seg;
                    if (pair != 0) {
                        lim = first_lane(pair);
                        cut = CUT_PAIR;
                        todo = 0;
                    }
                    continue;
                }
            }
            todo &= todo - 1;
            const int32_t plin = rdlane(lin, p), plp = rdlane(lp, p);
            const double pqd = rdlane_f64(qd, p);
            const int32_t eq = plp + tau, sq = plin - tau;
            const double dlin = (double)plin;
            // this lane's worker with the query added: (b), then (c) and (d)
            double lhs = k2 * (a.DS + pqd);
            double tt = (c1 + k1 * (a.S1 + dlin)) + k1q * (a.S2 + dlin * dlin);
            const bool has_d = USE_D && a.dlim != INFINITY;
            const uint64_t fsm = ballot((wbf >> p) & 1);
            uint64_t cand = fsm & ballot(lhs <= a.rhs) & ballot(tt <= ttft);
            if (USE_D) cand &= ballot(!has_d || tt <= a.dlim);
            // changed workers: surely feasible, surely not, or to be scanned
            const uint64_t full = ballot(a.loe <= eq) & ballot(sq > a.flo);
            const uint64_t sure = ~dm | ballot(plin + plp <= a.slack);
            cand = uni(cand & ~(dm & full));
            int bl = -1;
            int32_t pk = -1;  // the chosen worker's KV peak with the query (-1: only bounded)
            if (!DIAG) {
                while (ALD_LIKELY(uni(cand) != 0)) {
                    cand = uni(cand);
                    const int j = best_lane(cand, a.lead, a.key, a.w);
                    if (ALD_LIKELY((sure >> j) & 1)) {
                        bl = j;
                        break;
                    }
                    const int32_t v = scan(j, sq, eq, lin, lp);
                    if (v <= rdlane(a.M, j)) {
                        bl = j;
                        pk = v;
                        break;
                    }
                    cand &= ~(1ull << j);
                    stale += 1;
                }
            } else {
                for (uint64_t u = cand & ~sure; u != 0; u &= u - 1) {
                    const int j = first_lane(u);
                    if (scan(j, sq, eq, lin, lp) > rdlane(a.M, j)) {
                        cand &= ~(1ull << j);
                        stale += 1;
                    }
                }
                if (cand != 0) bl = best_lane(cand, a.lead, a.key, a.w);
            }
            bl = uni(bl);
            pk = uni(pk);
            int32_t bw = bl >= 0 ? rdlane(a.w, bl) : -1;
            // untouched workers beyond the lanes
            if (ALD_RARELY(over) && (bl < 0 || !ranks_before(rdlane64(a.key, bl), bw, over_key, over_w))) {
                int fr = 0;
                const int fw = first_untouched(gptr(state_arg()->bits_feas), rdlane(tp, p), over_r, fr);
                if (fw >= 0 && (bl < 0 || ranks_before(gptr(state_arg()->key)[scen_arg()->wbase + fw], fw,
                                                       rdlane64(a.key, bl), bw))) {
                    // it takes the lane of the last-ranked untouched worker, which
                    // is then the best one beyond the lanes
                    const int l = 63 - __builtin_clzll(~dm);
                    over_w = rdlane(a.w, l);
                    over_r = uni(L.rk[l]);
                    over_key = rdlane64(a.key, l);
                    cached &= ~(1ull << l);
                    const uint64_t vf = word_of(gptr(state_arg()->bits_feas), bits_at(fr));
                    const uint64_t vn = DIAG ? word_of(gptr(state_arg()->bits_nt), fw) : 0;
                    load_slot(lane == l, fw, fr);
                    wbf = lane == l ? vf : wbf;
                    if (DIAG) wbn = lane == l ? vn : wbn;
                    if (DIAG) {
                        lhs = k2 * (a.DS + pqd);
                        tt = (c1 + k1 * (a.S1 + dlin)) + k1q * (a.S2 + dlin * dlin);
                    }
                    bl = l;
                    bw = fw;
                    pk = -1;
                }
            }
            bl = uni(bl);
            bw = uni(bw);
            pk = uni(pk);
            if (DIAG) {
                // smallest KV excess
                if (ALD_RARELY((ballot(hit1 != 0) >> p) & 1)) {
                    if ((ballot(hit2 != 0) >> p) & 1) {  // both changed: the tile-start pair cannot decide
                        lim = p;
                        cut = CUT_PAIR;
                        todo = 0;
                        continue;
                    }
                    d_ex = ald_writelane(excess(p, sq, eq), p, d_ex);
                }
                const int more = __popcll(dm & cand) - __popcll(dm & fsm);
                if (more != 0) d_feas = ald_writelane(rdlane(d_feas, p) + more, p, d_feas);
                // near tie among workers ranked at or above the choice (all when rejected)
                uint64_t tied = ballot(near_tie(lhs, a.rhs)) | (ballot(ttft != INFINITY) & ballot(near_tie(tt, ttft)));
                if (USE_D) tied |= ballot(a.dlim != INFINITY) & ballot(near_tie(tt, a.dlim));
                tied &= dm;
                const int clean = ties ? rdlane(q.ntcnt, p) - __popcll(dm & ballot((wbn >> p) & 1)) : 0;
                bool nt = false;
                if (ALD_RARELY(tied != 0 || clean > 0)) {
                    const uint64_t bk = bl >= 0 ? rdlane64(a.key, bl) : 0;
                    nt = bl < 0 || (tied & ballot(!ranks_before(bk, bw, a.key, a.w))) != 0;
                    if (!nt && clean > 0) {  // the best-ranked untouched worker with a near tie
                        int fr = 0;
                        const int fw = first_untouched(gptr(state_arg()->bits_nt), rdlane(tp, p), 0, fr);
                        nt = fw >= 0 && !ranks_before(bk, bw, gptr(state_arg()->key)[scen_arg()->wbase + fw], fw);
                    }
                }
                d_near = ald_writelane(nt ? 1 : 0, p, d_near);
                if (bl >= 0) {
                    const double td = (c3 + c2 * (double)(a.B + 1)) + lhs;
                    if (lane == bl) {
                        P.tt[p] = tt;
                        P.td[p] = td;
                    }
                }
            }
            if (ALD_RARELY(bl < 0)) {
                stale += DIAG ? 0 : 1;
                continue;
            }

            // ---- commit the query to lane bl's worker (its request and the sums of c
            // and r are stored when the group ends: a store here would be waited
            // for at the next decision's first load)
            const int32_t B0 = rdlane(a.B, bl);
            if (ALD_RARELY(rdlane(a.room, bl) <= 0)) {  // no slot left for one more live request
                full_w = bw;
                cut = CUT_SLOTS;
                lim = p + 1;
                todo = 0;
                continue;
            }
            if (DIAG) {
                // once a worker has changed the rejected queries are looked at too
                if (dm == 0) todo = actm & (~0ull << p) & ~(1ull << p);
                hit1 |= q.w1 == bw ? 1 : 0;
                hit2 |= q.w2 == bw ? 1 : 0;
            }
            dm |= 1ull << bl;
            rl = ald_writelane(bl, p, rl);
            rB = ald_writelane(B0, p, rB);
            {
                const bool sel = lane == bl;
                const double DS = a.DS + pqd;
                // (B <= 8192, gs <= 8; a sum beyond the range fails the call)
                const uint32_t X = (uint32_t)(B0 + 1) << gs, D = (uint32_t)(DS * up);
                a.B += sel ? 1 : 0;
                a.room -= sel ? 1 : 0;
                a.slack = sel ? (pk >= 0 ? a.M - pk : a.slack - (plin + plp)) : a.slack;
                a.flo -= sel && a.loe <= eq ? sq + a.loe : 0;
                a.DS = sel ? DS : a.DS;
                const uint64_t key = (uint64_t)X * X + (uint64_t)D * D;
                a.key = sel ? key : a.key;
                a.lead = sel ? key_lead(key) : a.lead;
                a.rhs = sel ? rhs_of(B0 + 1) : a.rhs;
                a.S1 = sel ? a.S1 + dlin : a.S1;
                a.S2 = sel ? a.S2 + dlin * dlin : a.S2;
            }
            if (ALD_RARELY(dm == ~0ull) && w0 + p + 1 < end) {  // every lane holds a changed worker
                cut = CUT_LANES;
                lim = p + 1;
                todo = 0;
            }
        }
        lim = uni(lim);
        cut = uni(cut);
        // the group's outputs and rejections
        const uint64_t donem = actm & (lim >= NT ? ~0ull : ((1ull << lim) - 1));
        if (DIAG) {
            // the peaks of the placements that no scan computed on its way
            uint64_t left = 0;
            for (uint64_t m = ballot(rl >= 0); m != 0; m &= ~ballot(rl == rdlane(rl, first_lane(m))))
                left |= 1ull << rdlane(rl, first_lane(m));
            wave_sync();
            left &= ~(cached & ballot(L.have[lane] >= a.B));
            if (left != 0) {
                P.rl[lane] = rl;
                P.rB[lane] = rB;
                P.lin[lane] = lin;
                P.lp[lane] = lp;
                P.B[lane] = a.B;
            }
            while (uni(left) != 0) {
                left = uni(left);
                cached = uni(cached);
                pool_at = uni(pool_at);
                uint64_t jobs = left & cached & ballot(a.B <= L.room[lane]), fetch = 0;
                for (uint64_t m = left & ~jobs; m != 0; m &= m - 1) {
                    const int j = first_lane(m);
                    if (!reserve(j)) break;
                    fetch |= 1ull << j;
                }
                jobs |= fetch;
                if (jobs == 0) {  // full: every copy is dropped (HBM holds what they were made from)
                    cached = 0;
                    pool_at = 0;
                    continue;
                }
                if (lane == 0) {
                    P.jobs = jobs;
                    P.fetch = fetch;
                }
                __syncthreads();
                run_jobs(L, P, 0, tau);
                __syncthreads();
                if (in_mask(jobs)) a.slack = a.M - P.last[lane];
                left &= ~jobs;
            }
        }
        const int32_t on = __shfl(a.w, max(rl, 0), 64);
        const int32_t res = rl >= 0 ? on : (cut == CUT_SLOTS && lane == lim - 1 ? full_w : -1);
        if (rl >= 0) {
            // the request goes behind the worker's sorted columns (in the room of
            // finished requests where the slot range ends)
            const StateArg st = state_arg();
            const int64_t base = L.base[rl];
            const int32_t cap = L.cap[rl], head = L.head[rl];
            int at = head + rB;
            at = at > cap ? at - (cap + 1) : at;
            gptr(st->e)[base + at] = lp + tau;
            gptr(st->s)[base + at] = lin - tau;
            atomicAdd((unsigned long long*)&L.dsc[rl], (unsigned long long)lin);
            atomicAdd((unsigned long long*)&L.dsr[rl], (unsigned long long)lp);
            if (USE_D) {
                // it decodes from the end of this heartbeat with zero slack
                const int64_t lpos = base + L.lgn[rl] + (rB - (L.n[rl] - head));
                gptr(st->lge)[lpos] = lp + tau;
                gptr(st->lgw)[lpos] = hb;
                gptr(st->lgs)[lpos] = -L.phi[rl];
            }
        }
        if (in_mask(donem)) {
            const int64_t k = q_index(i);
            if (out != nullptr) out[k] = res < 0 ? res : res + scen_arg()->out_add;
            if (DIAG) {
                Diag d;
                d.n_feasible = d_feas;
                d.near_tie = d_near;
                d.kv_peak_chosen = rl >= 0 ? P.peak[lane] : 0;
                d.kv_excess_min = d_ex;
                d.ttft_chosen = rl >= 0 ? P.tt[lane] : 0.0;
                d.tdec_chosen = rl >= 0 ? P.td[lane] : 0.0;
                gptr(state_arg()->out_diag)[k] = d;
            }
        }
        const uint64_t rm = donem & ballot(res < 0);
        nrej += __popcll(rm);
        commits += __popcll(donem & ~rm);
        if (rm && firstrej == INT32_MAX) firstrej = w0 + first_lane(rm);
        pos = min(end, w0 + lim);
    }
    if (NWV > 1) {
        if (lane == 0) P.jobs = 0;
        __syncthreads();  // the other waves are done
    }
    // write back the changed workers' sums and list the workers whose summaries
    // the next round must rebuild
    const StateArg st = state_arg();
    bool range = false;  // a sum left the exactly representable range (they only grow)
    wave_sync();
    if (in_mask(dm)) {
        const int gw = scen_arg()->wbase + a.w;
        range = a.DS * up >= 0x1p31 || a.S2 >= 0x1p53;
        const int tn = a.B - (L.n[lane] - L.head[lane]);
        const int64_t SC = gptr(st->SC)[gw] + (int64_t)L.dsc[lane], SR = gptr(st->SR)[gw] + (int64_t)L.dsr[lane];
        gptr(st->tn)[gw] = tn;
        gptr(st->B)[gw] = a.B;
        gptr(st->SC)[gw] = SC;
        gptr(st->SR)[gw] = SR;
        gptr(st->DS)[gw] = (SC << gs) + (int64_t)scen_arg()->gn * SR;
        gptr(st->key)[gw] = a.key;
        gptr(st->rhs)[gw] = a.rhs;
        gptr(st->S1)[gw] = (int64_t)a.S1;
        gptr(st->S2)[gw] = (int64_t)a.S2;
        gptr(st->hbs)[gw] = hb;
        if (USE_D) gptr(st->lgn)[gw] = L.lgn[lane] + tn;
        gptr(st->built)[gw] = 0;
        gptr(st->dlist)[blockIdx.x * MAX_DIRTY + rank_in(dm)] = gw;
    }
    // the words of this tile are used up
    for (int k = lane; k < groups; k += NT) (gptr(st->any) + scen_arg()->any_off)[k] = 0;
    // per-query heartbeats: the tile ended at a query that heartbeats precede;
    // they run now, and the whole wave finds the next such query
    const int32_t* const hbq = gptr(scen_arg()->hb);
    const bool hb_here = hbq != nullptr && pos == end && pos == c.hb_next && pos < c.Q;
    int32_t hb_n = 0, hb_after = c.Q;
    if (hb_here) {
        hb_n = hbq[pos];
        for (int32_t b = pos + 1; b < c.Q; b += NT) {
            const uint64_t m = ballot(b + lane < c.Q && hbq[b + lane] > 0);
            if (m) {
                hb_after = b + first_lane(m);
                break;
            }
        }
    }
    const bool ranged = ballot(range) != 0;
    const int nd = __popcll(dm);
    if (lane == 0) {
        Ctl o = c;
        o.rebuild = 0;
        o.n_rej = c.n_rej + nrej;
        o.first_rej = min(c.first_rej, firstrej);
        gptr(st->dcount)[blockIdx.x] = nd;
        o.ndirty = nd;
        o.since_hb = c.since_hb + (pos - c.start);
        if (pos == end && c.H > 0 && o.since_hb >= c.H) {
            o.tau = c.tau + 1;
            o.hb_index = c.hb_index + 1;
            o.since_hb = 0;
            o.rebuild = 1;
        } else if (hb_here) {  // hb_n decode iterations, each its own heartbeat
            o.tau = c.tau + hb_n;
            o.hb_index = c.hb_index + hb_n;
            o.since_hb = 0;
            o.rebuild = 1;
            o.hb_next = hb_after;
        }
        o.start = pos;
        o.aborts = c.aborts + (cut != 0 ? 1 : 0);
        // choices of an untouched worker, by its bit words, after the first
        o.fallbacks = c.fallbacks + max(nd - 1, 0);
        o.stale_cuts = c.stale_cuts + (cut == CUT_STALE ? 1 : 0);
        o.commits = c.commits + commits;
        o.round = c.round + 1;
        o.err = ranged ? DEV_EOVERFLOW : (cut == CUT_SLOTS ? DEV_ESLOTS : 0);
        *cp = o;
        gptr(st->tinfo)[blockIdx.x].first_pc = INT32_MAX;
        gptr(st->tinfo)[blockIdx.x].empty_rank = INT32_MAX;
        publish_ctl(o);
    }
}

// The variants checking constraint (d), in a unit of their own.
hipError_t launch_commit_d(const State& st, int32_t blocks, hipStream_t stream);

}  // namespace ald
