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
// What bounds it: the chain of decisions (one wave, no parallelism over
// queries), so instructions and round trips per decision.  Measured per
// placed query, 256-scenario sweep (tiles of 1,024, no diagnostics): see the
// figures beside the launch.

constexpr int DBITS_W = 2048;   // changed-worker bitmap words in LDS: scenarios of up to 65536 workers
constexpr int ORDER_W = 4096;   // workers whose rank order is kept in LDS
constexpr int POOL = 14336;     // pool entries (8 B each) for changed workers' columns
constexpr int POOL_SLACK = 48;  // entries a copied worker may grow by before it is copied again
static_assert(POOL >= HOT + POOL_SLACK, "the largest worker fits the pool");

// Orders LDS traffic between the lanes of the (single-wave) commit block
// without waiting for outstanding global memory operations.
__device__ __forceinline__ void wave_sync() { __builtin_amdgcn_wave_barrier(); }

// Branch hints: the decision loop is one wave's instruction stream, and every
// taken branch over a block that hardly ever runs stalls it.
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

// The lane of the non-empty mask m whose (key, worker) ranks first by Algorithm
// 1's order.  The keys' high words nearly always decide.
__device__ __forceinline__ int best_lane(uint64_t m, uint64_t key, int32_t w)
{
    if ((m & (m - 1)) == 0) return first_lane(m);
    const uint32_t hi = (uint32_t)(key >> 32);
    const uint32_t hm = wave_max_u32(in_mask(m) ? hi : 0u);
    m &= ballot(hi == hm);
    if (ALD_RARELY((m & (m - 1)) != 0)) {
        const uint32_t lo = (uint32_t)key;
        const uint32_t lm = wave_max_u32(in_mask(m) ? lo : 0u);
        m &= ballot(lo == lm);
        if (m & (m - 1)) {
            const int32_t wm = wave_min32(in_mask(m) ? w : INT32_MAX);
            m &= ballot(w == wm);
        }
    }
    return first_lane(m);
}

// The worker a lane holds.
struct Slot {
    int32_t w;       // scenario-local index, -1 = none
    int32_t rk;      // its place in the tile-start rank order
    int32_t B;       // live requests, appended ones included
    int32_t tn;      // requests appended in this tile
    int32_t head, n, M, cap;
    // Bounds of its KV peak without a new query: at most M - slack; its demand at
    // end iteration loe is at least M - loe - flo (so with a query that is alive
    // then, sq + loe more).
    int32_t slack, flo, loe;
    int32_t lgn;     // entries in its constraint-(d) log
    int32_t off, room;  // its columns in the LDS pool (when copied): first entry, entries reserved
    int64_t base;    // first slot
    int32_t *ep, *sp;  // the slot range's columns
    int64_t SC, SR;
    uint64_t key;
    // sums as fp64 (integers below 2^53 and multiples of 2^-8 below 2^31: exact)
    double DS;       // sum of D = 2^-gs * State::DS
    double S1, S2;   // TTFT sums of this heartbeat
    double rhs;
    double dlim;     // constraint (d)'s limit, fixed within a heartbeat (no ongoing request joins or leaves)
    double phi;      // its slack gain: a request placed now logs slack - phi = -phi
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

struct CommitLDS {
    int32_t cw[64], cr[64];  // untouched workers picked for the free lanes: index, rank
    uint64_t cword[64];      // and bit word
    int32_t over_w, over_r;  // the first one there was no lane for
    int32_t dw[MAX_DIRTY];
    uint32_t dbits[DBITS_W];
    int32_t order[ORDER_W];
    int32_t pe[POOL], ps[POOL];
};

// Has worker w (scenario-local) changed in this tile?  (any lane, any w)
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

template <bool DIAG, bool USE_D>
__global__ __launch_bounds__(COMMIT_THREADS) void k_commit(State)
{
    constexpr int NT = COMMIT_THREADS;
    const int lane = threadIdx.x;
    Ctl* const cp = gptr(state_arg()->ctl) + blockIdx.x;
    const Ctl c = *cp;
    {
        const StateArg st = state_arg();
        if (c.call != st->call) {  // another call's control block: this call was blocked
            if (st->status != nullptr && lane == 0) *gptr(st->status) = ALD_EBLOCKED;
            return;
        }
        const bool qbad = gptr(st->qbad) != nullptr && *gptr(st->qbad) != 0;
        if (qbad || c.err || c.start >= c.Q) {
            if (lane == 0) {
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
    const bool lds_order = W <= ORDER_W;
    if (fpc < end) {
        if (W <= DBITS_W * 32)
            for (int k = lane; k < (W + 31) / 32; k += NT) L.dbits[k] = 0u;
        if (lds_order) {
            const int32_t* const order = gptr(state_arg()->order) + scen_arg()->wbase;
            for (int k0 = 0; k0 < W; k0 += 4 * NT) {
                int32_t v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = order[min(k0 + u * NT + lane, W - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (k0 + u * NT + lane < W) L.order[k0 + u * NT + lane] = v[u];
            }
        }
    }
    wave_sync();

    uint64_t dm = 0;      // lanes holding changed workers
    uint64_t cached = 0;  // lanes whose worker's columns are in the pool
    int pool_at = 0;
    Slot a;
    a.w = -1;
    a.rk = a.B = a.tn = a.head = a.n = a.M = a.cap = a.slack = a.flo = a.lgn = a.off = a.room = 0;
    a.loe = INT32_MAX;
    a.base = a.SC = a.SR = 0;
    a.ep = a.sp = nullptr;
    a.key = 0;
    a.DS = a.S1 = a.S2 = a.rhs = a.phi = 0.0;
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
    // this lane's worker at tile start (its columns and sums are as built)
    auto load_slot = [&](int w, int rk) {
        const StateArg st = state_arg();
        const int gw = scen_arg()->wbase + w;
        a.w = w;
        a.rk = rk;
        a.tn = 0;
        a.n = gptr(st->n)[gw];
        a.head = gptr(st->head)[gw];
        a.M = gptr(st->M)[gw];
        a.cap = gptr(st->cap)[gw];
        const int32_t peak = gptr(st->peak)[gw];
        a.loe = gptr(st->peake)[gw];
        a.base = gptr(st->slot_base)[gw];
        a.ep = gptr(st->e) + a.base;
        a.sp = gptr(st->s) + a.base;
        a.SC = gptr(st->SC)[gw];
        a.SR = gptr(st->SR)[gw];
        a.key = gptr(st->key)[gw];
        const int64_t ds = gptr(st->DS)[gw], s1 = gptr(st->S1)[gw], s2 = gptr(st->S2)[gw];
        const bool cur = gptr(st->hbs)[gw] == hb;
        if (USE_D) {
            a.dlim = gptr(st->dlim)[gw];
            a.phi = gptr(st->phi)[gw];
            a.lgn = gptr(st->lgn)[gw];
        }
        a.B = a.n - a.head;
        a.slack = a.M - peak;
        a.flo = (int32_t)((uint32_t)a.slack - (uint32_t)a.loe);
        a.DS = (double)ds * down;
        a.S1 = cur ? (double)s1 : 0.0;
        a.S2 = cur ? (double)s2 : 0.0;
        a.rhs = rhs_of(a.B);
    };
    // make sure lane j's columns are in the pool
    auto fetch_columns = [&](int j) {
        cached = uni(cached);
        pool_at = uni(pool_at);
        if (ALD_LIKELY((cached >> j) & 1)) return;
        const StateArg st = state_arg();
        const int B = rdlane(a.B, j), tn = rdlane(a.tn, j), head = rdlane(a.head, j), n = rdlane(a.n, j);
        const int cap = rdlane(a.cap, j);
        const int64_t base = rdlane64s(a.base, j);
        const int room = B + POOL_SLACK;
        if (pool_at + room > POOL) {  // full: every copy is dropped (HBM holds what they were made from)
            cached = 0;
            pool_at = 0;
        }
        const int off = pool_at;
        pool_at += room;
        cached |= 1ull << j;
        if (lane == j) {
            a.off = off;
            a.room = room;
        }
        const int B0 = n - head;
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
        wave_sync();
        if (ALD_RARELY(tn > 0)) {
            __builtin_amdgcn_s_waitcnt(0);  // this wave's appends have left
            for (int t = 0; t < tn; ++t) {
                int p = n + t;
                p = p > cap ? p - (cap + 1) : p;
                const int32_t x = coherent(gptr(st->e) + base + p), y = coherent(gptr(st->s) + base + p);
                lds_sorted_insert(L.pe + off, L.ps + off, B0 + t, x, y);
            }
        }
    };
    // exact KV demand of lane j's worker with the query; the lane's bounds become exact
    auto scan = [&](int j, int32_t sq, int32_t eq) -> int32_t {
        fetch_columns(j);
        const int off = rdlane(a.off, j);
        const Peak r = wave_kv_peak(L.pe + off, L.ps + off, rdlane(a.B, j), sq, eq);
        if (lane == j) {
            a.slack = a.M - r.without;
            a.loe = r.at;
            a.flo = a.slack - r.at;
        }
        return r.with;
    };

    // short tiles with diagnostics: the commit merges the worker blocks' results
    // per query itself and writes every query's diagnostics (else the selection
    // wrote those of the queries that no worker can take)
    const bool brief = DIAG && state_arg()->brief != 0;
    int pos = brief ? start : fpc;
    // why the tile was cut (0: not)
    constexpr int CUT_STALE = 1, CUT_SLOTS = 2, CUT_PAIR = 3, CUT_LANES = 4;
    int cut = 0;
    int32_t range = 0;  // (per lane) nonzero: a sum left the exactly representable range
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
            const int64_t stride = scen_arg()->pstride;
            const ulonglong2* row = gptr(state_arg()->part) + scen_arg()->part_off + 2 * (int64_t)(act ? i - start : 0);
            uint64_t a1 = ~0ull, a2 = ~0ull;
            const int nblk = scen_arg()->nblk;
#pragma unroll 16
            for (int b = 0; b < nblk; ++b) {
                const ulonglong2 x = row[2 * b * stride], y = row[2 * b * stride + 1];
                merge_two(a1, a2, x.x, x.y);
                q.nfeas += (int32_t)y.x;
                q.ntcnt += (int32_t)y.y;
            }
            ex_unpack(a1, q.ex1, q.w1);
            ex_unpack(a2, q.ex2, q.w2);
        }
        const double qd = (double)(((int64_t)lin << gs) + (int64_t)scen_arg()->gn * lp) * down;

        // the group's bit word of this lane's worker w (all lanes call it)
        auto word_of = [&](const uint64_t* bits, int w) -> uint64_t {
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
        auto first_untouched = [&](const uint64_t* bits, int t, int r0, int& fr) -> int {
            const uint64_t* row = bits + scen_arg()->bits_off + (int64_t)(t >> 6) * W;
            const int nd = __popcll(dm);
            for (; r0 < W; r0 += NT) {
                const int w = worker_at(min(r0 + lane, W - 1));
                const uint64_t v = row[bits_at(min(r0 + lane, W - 1))];
                const uint64_t hit = ballot(r0 + lane < W && ((v >> (t & 63)) & 1) && !dirty_w(L, W, nd, w));
                if (hit) {
                    const int l = first_lane(hit);
                    fr = r0 + l;
                    return rdlane(w, l);
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
            if (in_mask(~dm)) {
                const int k = rank_in(~dm);
                a.w = -1;
                if (k < min(cnt, nfree)) {
                    load_slot(L.cw[k], L.cr[k]);
                    wbf = L.cword[k];
                }
            }
            if (dm != 0) {
                const uint64_t v = word_of(bits, bits_at(a.rk));
                if (in_mask(dm)) wbf = v;
            }
        }
        const bool ties = DIAG && ballot(act && q.ntcnt > 0) != 0;  // some query of the group has near ties
        if (ties) {
            const uint64_t v = word_of(gptr(state_arg()->bits_nt), max(a.w, 0));
            wbn = a.w >= 0 ? v : 0;
        }
        // With diagnostics every chosen worker is scanned: the columns of the
        // best-ranked untouched ones, one per query that can be placed, are read
        // together (a scan that has to fetch them waits a round trip; without
        // diagnostics so few are scanned that reading ahead cost more: 72 -> 83 us
        // per tile of 50 queries over 257 workers whose capacity binds)
        if (DIAG && potm != 0) {
            uint64_t want = ~dm & ~cached & ballot(a.w >= 0 && a.B <= 128);
            for (int k = __popcll(want) - __popcll(potm); k > 0; --k) want &= ~(1ull << (63 - __builtin_clzll(want)));
            while (want != 0) {
                constexpr int U = 8;
                int j[U], off[U];
                int32_t ve[U][2], vs[U][2];
                int n = 0;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    j[u] = want != 0 ? first_lane(want) : j[u > 0 ? u - 1 : 0];
                    const int room = rdlane(a.B, j[u]) + POOL_SLACK;
                    const bool fits = want != 0 && pool_at + room <= POOL;
                    off[u] = pool_at;
                    if (fits) {
                        pool_at += room;
                        cached |= 1ull << j[u];
                        if (lane == j[u]) {
                            a.off = off[u];
                            a.room = room;
                        }
                        n = u + 1;
                    }
                    want = fits ? want & (want - 1) : 0;
                    const int B = rdlane(a.B, j[u]), head = rdlane(a.head, j[u]);
                    const int32_t* ge = (const int32_t*)rdlane64((uint64_t)a.ep, j[u]) + head;
                    const int32_t* gs_ = (const int32_t*)rdlane64((uint64_t)a.sp, j[u]) + head;
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const int k = max(min(c * 64 + lane, B - 1), 0);
                        ve[u][c] = gptr(ge)[k];
                        vs[u][c] = gptr(gs_)[k];
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int B = rdlane(a.B, j[u]);
#pragma unroll
                    for (int c = 0; c < 2; ++c)
                        if (u < n && c * 64 + lane < B) {
                            L.pe[off[u] + c * 64 + lane] = ve[u][c];
                            L.ps[off[u] + c * 64 + lane] = vs[u][c];
                        }
                }
            }
            wave_sync();
        }
        // (diagnostics) this lane's query's results: as at tile start until its turn
        int32_t d_feas = q.nfeas, d_near = q.ntcnt > 0 ? 1 : 0, d_peak = 0, d_ex = q.ex1;
        int32_t d_t0 = 0, d_t1 = 0, d_d0 = 0, d_d1 = 0;  // ttft and tdec of the choice (low and high words)
        // and whether the workers of its two smallest excesses have changed
        int32_t hit1 = 0, hit2 = 0;
        if (DIAG && dm != 0) {
            hit1 = q.w1 >= 0 && dirty_w(L, W, __popcll(dm), q.w1) ? 1 : 0;
            hit2 = q.w2 >= 0 && dirty_w(L, W, __popcll(dm), q.w2) ? 1 : 0;
        }
        // the smallest excess of query p, whose best worker has changed but not the
        // second best
        auto excess = [&](int p, int32_t sq, int32_t eq) -> int32_t {
            const int32_t x2 = rdlane(q.ex2, p), w2 = rdlane(q.w2, p);
            const int j = first_lane(dm & ballot(a.w == rdlane(q.w1, p)));
            // (commits only raise a demand: a floor at or above the second smallest
            // leaves that one)
            if (w2 >= 0 && rdlane(a.loe, j) <= eq && (int64_t)sq - rdlane(a.flo, j) >= x2) return x2;
            const int32_t now = scan(j, sq, eq) - rdlane(a.M, j);
            stale += 1;
            return (w2 < 0 || now < x2) ? now : x2;
        };

        int32_t res = -1;  // this lane's query's worker
        int lim = NT;      // queries of lanes below lim are decided when the group ends (the tile is cut there)
        // queries left to decide (with diagnostics, once a worker has changed,
        // the rejected ones too)
        uint64_t todo = (DIAG && dm != 0) ? actm : potm;
        while (uni(todo) != 0) {
            todo = uni(todo);
            dm = uni(dm);
            cached = uni(cached);
            stale = uni(stale);
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
                    const int j = best_lane(cand, a.key, a.w);
                    if (ALD_LIKELY((sure >> j) & 1)) {
                        bl = j;
                        break;
                    }
                    const int32_t v = scan(j, sq, eq);
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
                    if (scan(j, sq, eq) > rdlane(a.M, j)) {
                        cand &= ~(1ull << j);
                        stale += 1;
                    }
                }
                if (cand != 0) bl = best_lane(cand, a.key, a.w);
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
                    over_r = rdlane(a.rk, l);
                    over_key = rdlane64(a.key, l);
                    cached &= ~(1ull << l);
                    const uint64_t vf = word_of(gptr(state_arg()->bits_feas), bits_at(fr));
                    const uint64_t vn = DIAG ? word_of(gptr(state_arg()->bits_nt), fw) : 0;
                    if (lane == l) {
                        load_slot(fw, fr);
                        wbf = vf;
                        wbn = vn;
                    }
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
                    pk = scan(bl, sq, eq);
                    d_peak = ald_writelane(pk, p, d_peak);
                    const double td = (c3 + c2 * (double)(a.B + 1)) + lhs;
                    const uint64_t t = rdlane64(__builtin_bit_cast(uint64_t, tt), bl);
                    const uint64_t d = rdlane64(__builtin_bit_cast(uint64_t, td), bl);
                    d_t0 = ald_writelane((int32_t)(uint32_t)t, p, d_t0);
                    d_t1 = ald_writelane((int32_t)(uint32_t)(t >> 32), p, d_t1);
                    d_d0 = ald_writelane((int32_t)(uint32_t)d, p, d_d0);
                    d_d1 = ald_writelane((int32_t)(uint32_t)(d >> 32), p, d_d1);
                }
            }
            if (ALD_RARELY(bl < 0)) {
                stale += DIAG ? 0 : 1;
                continue;
            }

            // ---- commit the query to lane bl's worker
            if (lane == p) res = bw;
            if (ALD_RARELY(!((ballot(a.B < a.cap) >> bl) & 1))) {  // no slot left for one more live request
                cut = CUT_SLOTS;
                lim = p + 1;
                todo = 0;
                continue;
            }
            if (ALD_RARELY(!((dm >> bl) & 1))) {  // untouched so far
                if (lane == 0) {
                    L.dw[__popcll(dm)] = bw;
                    if (W <= DBITS_W * 32) L.dbits[bw >> 5] |= 1u << (bw & 31);
                }
                dm |= 1ull << bl;
                wave_sync();
                if (DIAG) {  // from here on the rejected queries are looked at too
                    todo = actm & (~0ull << p) & ~(1ull << p);
                    hit1 |= q.w1 == bw ? 1 : 0;
                    hit2 |= q.w2 == bw ? 1 : 0;
                }
            }
            if (DIAG ? ALD_LIKELY((cached >> bl) & 1) : ALD_RARELY((cached >> bl) & 1)) {
                const int B0 = rdlane(a.B, bl);
                if (ALD_LIKELY(B0 < rdlane(a.room, bl))) {
                    const int off = rdlane(a.off, bl);
                    lds_sorted_insert(L.pe + off, L.ps + off, B0, eq, sq);
                } else {
                    cached &= ~(1ull << bl);
                }
            }
            if (lane == bl) {
                // behind the sorted columns (in the room of finished requests
                // where the slot range ends)
                int at = a.n + a.tn;
                at = at > a.cap ? at - (a.cap + 1) : at;
                a.ep[at] = eq;
                a.sp[at] = sq;
                a.tn += 1;
                a.B += 1;
                a.SC += plin;
                a.SR += plp;
                a.DS += pqd;
                const double DS = a.DS * up;
                range |= DS >= 0x1p31 ? 1 : 0;
                const uint32_t X = (uint32_t)a.B << gs, D = (uint32_t)DS;  // (B <= 8192, gs <= 8)
                a.key = (uint64_t)X * X + (uint64_t)D * D;
                a.rhs = rhs_of(a.B);
                a.S1 += dlin;
                a.S2 += dlin * dlin;
                range |= a.S2 >= 0x1p53 ? 1 : 0;
                a.slack = pk >= 0 ? a.M - pk : a.slack - (plin + plp);
                if (a.loe <= eq) a.flo -= sq + a.loe;
                if (USE_D) {
                    // the new request decodes from the end of this heartbeat with zero slack
                    const StateArg st = state_arg();
                    const int64_t lpos = a.base + a.lgn;
                    gptr(st->lge)[lpos] = eq;
                    gptr(st->lgw)[lpos] = hb;
                    gptr(st->lgs)[lpos] = -a.phi;
                    a.lgn += 1;
                }
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
        if (in_mask(donem)) {
            const int64_t k = q_index(i);
            if (out != nullptr) out[k] = res < 0 ? res : res + scen_arg()->out_add;
            if (DIAG) {
                Diag d;
                d.n_feasible = d_feas;
                d.near_tie = d_near;
                d.kv_peak_chosen = d_peak;
                d.kv_excess_min = d_ex;
                d.ttft_chosen = __builtin_bit_cast(double, ((uint64_t)(uint32_t)d_t1 << 32) | (uint32_t)d_t0);
                d.tdec_chosen = __builtin_bit_cast(double, ((uint64_t)(uint32_t)d_d1 << 32) | (uint32_t)d_d0);
                gptr(state_arg()->out_diag)[k] = d;
            }
        }
        const uint64_t rm = donem & ballot(res < 0);
        nrej += __popcll(rm);
        commits += __popcll(donem & ~rm);
        if (rm && firstrej == INT32_MAX) firstrej = w0 + first_lane(rm);
        pos = min(end, w0 + lim);
    }
    // write back the changed workers' sums and list the workers whose summaries
    // the next round must rebuild
    const StateArg st = state_arg();
    if (in_mask(dm)) {
        const int gw = scen_arg()->wbase + a.w;
        gptr(st->tn)[gw] = a.tn;
        gptr(st->B)[gw] = a.B;
        gptr(st->SC)[gw] = a.SC;
        gptr(st->SR)[gw] = a.SR;
        gptr(st->DS)[gw] = (a.SC << gs) + (int64_t)scen_arg()->gn * a.SR;
        gptr(st->key)[gw] = a.key;
        gptr(st->rhs)[gw] = a.rhs;
        gptr(st->S1)[gw] = (int64_t)a.S1;
        gptr(st->S2)[gw] = (int64_t)a.S2;
        gptr(st->hbs)[gw] = hb;
        if (USE_D) gptr(st->lgn)[gw] = a.lgn;
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
    const bool ranged = ballot(range != 0) != 0;
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
