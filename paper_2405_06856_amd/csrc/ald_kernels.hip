// HIP kernels of libaladdin for gfx950 (MI355X): wave64, no matrix cores --
// the placement evaluator is integer/fp64 scan-and-reduce work.
//
// Per tile of T consecutive queries (one heartbeat segment at most):
//   k_build   rebuild the breakpoint summaries of workers whose live set moved
//   k_eval    (k_eval_short where the tile is short) every (query, worker) pair of the tile against the tile-start
//             state: KV peak (constraint (e)), decode (b), TTFT (c), near-tie
//             margins; feasibility / near-tie bits, per-block KV-excess minima,
//             the workers' rank order
//   k_select  (diagnostics, long tiles) per query: feasible and near-tie counts, the
//             two smallest KV excesses, the outputs of queries no worker can take
//   k_commit  arrival-order commit: one wave per scenario walks the tile,
//             re-evaluating only workers changed earlier in the same tile, and
//             cuts the tile when the tile-start results cannot decide exactly
//             (ald_commit.h; launched from ald_commit.hip and ald_commit_d.hip).
#include "ald_device.h"

#include <type_traits>

namespace ald {

// ---------------------------------------------------------------------------------------------
// Sort the requests a commit appended behind a worker's slots [head, n) into
// them, and move the whole to the start of the slot range (whole block): each
// request's place is counted (a sorted one moves up by the appended ones ending
// strictly before it; an appended one goes behind every sorted one ending no
// later and every earlier appended one ending no later).  The worker's summary
// slots, which are rebuilt afterwards, hold the result in between.
constexpr int TAIL_LDS = 1024;  // appended requests whose ends are kept in LDS (more are read from memory)
__device__ void merge_tail(int32_t* e, int32_t* s, int4* tmp, int head, int n, int cap, int m, int32_t* te)
{
    constexpr int NT = BUILD_THREADS;
    const int tid = threadIdx.x;
    const int L = n - head;
    auto at = [&](int t) { return n + t > cap ? n + t - (cap + 1) : n + t; };
    for (int t = tid; t < min(m, TAIL_LDS); t += NT) te[t] = e[at(t)];
    __syncthreads();
    auto tail = [&](int t) { return t < TAIL_LDS ? te[t] : e[at(t)]; };
    for (int k = tid; k < L; k += NT) {
        const int32_t x = e[head + k];
        int up = 0;
        for (int t = 0; t < m; ++t) up += tail(t) < x ? 1 : 0;
        tmp[k + up].x = x;
        tmp[k + up].y = s[head + k];
    }
    for (int t = tid; t < m; t += NT) {
        const int32_t x = tail(t);
        int to = lower_bound_i32(e, head, n, x + 1) - head;
        for (int j = 0; j < m; ++j) {
            const int32_t v = tail(j);
            to += (v < x || (v == x && j < t)) ? 1 : 0;
        }
        tmp[to].x = x;
        tmp[to].y = s[at(t)];
    }
    __syncthreads();
    for (int k = tid; k < L + m; k += NT) {
        e[k] = tmp[k].x;
        s[k] = tmp[k].y;
    }
    __syncthreads();
}

// Integer forms of a built worker's latency checks.  Both left sides are rounded
// fp64 expressions that never decrease as DS + qD (resp. l_in) grows -- each step
// is an exact conversion, a product with a non-negative constant or a sum,
// and rounding is monotone -- so each check holds exactly up to a threshold,
// found by searching with the very expression the pair check evaluates.
// Queries have qD <= 2^33 and l_in <= 2^24; DS < 2^31.
struct Sums {
    int64_t DS, S1, S2;
    double rhs, dlim;
};
constexpr int64_t XMAX = (int64_t)1 << 36;
constexpr int64_t LMAX = (int64_t)1 << 24;

// An estimate of the largest l with c1 + k1 (S1 + l) + k1q (S2 + l^2) <= t.
__device__ __forceinline__ double ttft_root(const Scen& sc, const Sums& u, double t)
{
    const double c = t - ((sc.c1 + sc.k1 * (double)u.S1) + sc.k1q * (double)u.S2);
    return 2.0 * c / (sc.k1 + sqrt(fmax(0.0, sc.k1 * sc.k1 + 4.0 * sc.k1q * c)));
}

// The thresholds of (b) and of (c) with (d) (one whole wave).
__device__ void build_limits(const State& st, const Scen& sc, int gw, const Sums& u)
{
    const double per = ldexp(1.0, sc.gs) / sc.k2;
    const int64_t x = wave_last_true_near(u.rhs * per, 0, XMAX, [&](int64_t v) { return dec_lhs(sc, v) <= u.rhs; });
    // (c) and (d) bound the same prefill time
    const int64_t l = wave_last_true_near(ttft_root(sc, u, fmin(sc.ttft, u.dlim)), 1, LMAX, [&](int64_t v) {
        const double t = ttft_of(sc, u.S1 + v, u.S2 + v * v);
        return t <= sc.ttft && t <= u.dlim;
    });
    if (lane_id() == 0) {
        st.dq_max[gw] = x - u.DS;
        st.lthr[gw] = (int32_t)l;
    }
}

// The near-tie bands of (b) (`decode`) or of (c) and (d) (one whole wave).
// Inside a band of at most 64 values the margin test itself is run once per
// value (one per lane), giving the exact near-tie set as a bit mask.
__device__ void build_ties(const State& st, const Scen& sc, int gw, const Sums& u, bool decode, int32_t* err)
{
    const bool l0 = lane_id() == 0;
    if (decode) {
        const double per = ldexp(1.0, sc.gs) / sc.k2;
        const double band = tie_band(u.rhs);
        const double lo = u.rhs - band, hi = u.rhs + band;
        const int64_t xl = wave_last_true_near(lo * per, 0, XMAX, [&](int64_t v) { return dec_lhs(sc, v) < lo; }) + 1;
        const int64_t xh = wave_last_true_near(hi * per, 0, XMAX, [&](int64_t v) { return dec_lhs(sc, v) <= hi; });
        const int64_t width = xh - xl + 1;
        const uint64_t mask = ballot(lane_id() < width && near_tie(dec_lhs(sc, xl + lane_id()), u.rhs));
        if (l0) {
            st.ntd_lo[gw] = xl - u.DS;
            st.ntd_hi[gw] = xh - u.DS;
            st.ntd_mask[gw] = width <= 64 ? mask : 0;
            if (width > 64 && sc.ntint) raise_error(err, DEV_EOVERFLOW);
        }
        return;
    }
    auto tt = [&](int64_t l) { return ttft_of(sc, u.S1 + l, u.S2 + l * l); };
    // the TTFT band (empty on a decode worker, whose T_pre is +inf)
    int64_t ll = 1, lh = 0;
    if (sc.ttft != INFINITY) {
        const double band = tie_band(sc.ttft);
        const double lo = sc.ttft - band, hi = sc.ttft + band;
        ll = wave_last_true_near(ttft_root(sc, u, lo), 1, LMAX, [&](int64_t v) { return tt(v) < lo; }) + 1;
        lh = wave_last_true_near(ttft_root(sc, u, hi), 1, LMAX, [&](int64_t v) { return tt(v) <= hi; });
    }
    const int64_t width = lh - ll + 1;
    const uint64_t mask = ballot(lane_id() < width && near_tie(tt(ll + lane_id()), sc.ttft));
    if (l0) {
        st.ntt_lo[gw] = (int32_t)ll;
        st.ntt_hi[gw] = (int32_t)lh;
        st.ntt_mask[gw] = width <= 64 ? mask : 0;
        if (width > 64 && sc.ntint) raise_error(err, DEV_EOVERFLOW);
    }
    // the band of (d)'s limit (empty without one)
    int64_t pl = 1, ph = 0;
    if (u.dlim != INFINITY) {
        const double band = tie_band(u.dlim);
        const double lo = u.dlim - band, hi = u.dlim + band;
        pl = wave_last_true_near(ttft_root(sc, u, lo), 1, LMAX, [&](int64_t v) { return tt(v) < lo; }) + 1;
        ph = wave_last_true_near(ttft_root(sc, u, hi), 1, LMAX, [&](int64_t v) { return tt(v) <= hi; });
    }
    if (l0) {
        st.ntp_lo[gw] = (int32_t)pl;
        st.ntp_hi[gw] = (int32_t)ph;
    }
}

// Breakpoint summaries of one worker (whole block).  Drops finished requests
// (e < tau), recomputes ss / pme / sm over the live slots and the worker's
// aggregates.  Called with every thread of a BUILD_THREADS block.
__device__ void build_worker(const State& st, const Scen& sc, int gw, int32_t tau, int32_t hb, int need, int32_t* err)
{
    constexpr int NT = BUILD_THREADS;
    __shared__ int64_t red[NT / 64];
    const int tid = threadIdx.x;
    const int64_t base = st.slot_base[gw];
    int32_t* e = st.e + base;
    int32_t* s = st.s + base;
    int4* pms = st.pms + base;
    __shared__ int32_t hist[LB_MAX];  // (first the appended requests' ends)
    static_assert(TAIL_LDS <= LB_MAX, "the ends fit");
    int n = st.n[gw];
    int head = st.head[gw];
    const int tn = st.tn[gw];
    if (tn > 0) {
        merge_tail(e, s, pms, head, n, st.cap[gw], tn, hist);
        n = n - head + tn;
        head = 0;
        if (tid == 0) {
            st.n[gw] = n;
            st.tn[gw] = 0;
        }
    }

    // Constraint (d): bring the worker's slack gain phi up to the current
    // heartbeat.  Each heartbeat since the last update ran one decode iteration
    // over the requests live at its start (e >= that iteration's tau; nothing
    // is placed between heartbeats without a build), taking Eq. 3's time.
    double phi = 0.0;
    if (sc.use_d) {
        phi = st.phi[gw];
        const int pending = hb - st.phi_hb[gw];
        if (pending < 0) {
            if (tid == 0) raise_error(err, DEV_EINVAL);
        } else {
            for (int p = 0; p < pending; ++p) {
                const int32_t tk = tau - pending + p;
                int64_t cnt = 0, ssum = 0;
                for (int k = head + tid; k < n; k += NT) {
                    const bool in = e[k] >= tk;
                    cnt += in ? 1 : 0;
                    ssum += in ? s[k] : 0;
                }
                cnt = block_reduce<NT>(cnt, 0, OpAdd(), red);
                ssum = block_reduce<NT>(ssum, 0, OpAdd(), red);
                if (cnt == 0) break;  // the live set only shrinks: no later iteration runs a batch
                const int64_t ctx = ssum + cnt * (int64_t)tk;  // sum of the contexts c = s + tau
                const double t_iter = (sc.c3 + sc.c2 * (double)cnt) + sc.k2 * (double)ctx;
                phi = phi + (sc.tdec - t_iter);
            }
            if (tid == 0) {
                st.phi[gw] = phi;
                st.phi_hb[gw] = hb;
            }
        }
    }

    // finished requests form a prefix of the live range (sorted by e)
    int64_t fin = 0;
    for (int k = head + tid; k < n; k += NT) fin += (e[k] < tau) ? 1 : 0;
    head += (int)block_reduce<NT>(fin, 0, OpAdd(), red);

    const int B = n - head;
    const int CH = (B + NT - 1) / NT;
    const int k0 = head + tid * CH;
    const int k1 = min(n, k0 + CH);

    int64_t ls = 0, le = 0;
    for (int k = k0; k < k1; ++k) { ls += s[k]; le += e[k]; }
    int64_t tot_s, tot_e;
    const int64_t soff = block_scan_excl<NT, true>(ls, 0, OpAdd(), &tot_s, red);
    block_scan_excl<NT, true>(le, 0, OpAdd(), &tot_e, red);

    int64_t run = soff, lmaxP = INT64_MIN, lmaxPe = INT64_MIN;
    int32_t peake = INT32_MAX;  // the end at which this thread's largest P falls
    for (int k = k1 - 1; k >= k0; --k) {
        run += s[k];
        pms[k].z = (int32_t)run;
        const int64_t P = run + (int64_t)(n - k) * e[k];
        peake = P >= lmaxP ? e[k] : peake;
        lmaxP = P > lmaxP ? P : lmaxP;
        const int64_t Pe = P + e[k];
        lmaxPe = Pe > lmaxPe ? Pe : lmaxPe;
    }
    int64_t totP, totPe;
    const int64_t smoff = block_scan_excl<NT, true>(lmaxP, INT64_MIN, OpMax(), &totP, red);
    const int64_t pmoff = block_scan_excl<NT, false>(lmaxPe, INT64_MIN, OpMax(), &totPe, red);
    // the earliest end at which the worker's peak falls
    __shared__ int32_t first_peak;
    if (tid == 0) first_peak = INT32_MAX;
    __syncthreads();
    if (lmaxP == totP && k0 < k1) atomicMin(&first_peak, peake);

    int64_t runmax = smoff;
    for (int k = k1 - 1; k >= k0; --k) {
        const int64_t P = (int64_t)pms[k].z + (int64_t)(n - k) * e[k];
        runmax = P > runmax ? P : runmax;
        pms[k].y = (int32_t)runmax;
    }
    int64_t runpm = pmoff;
    for (int k = k0; k < k1; ++k) {
        pms[k].x = runpm == INT64_MIN ? PME_NONE : (int32_t)runpm;
        pms[k].w = n - k;
        const int64_t P = (int64_t)pms[k].z + (int64_t)(n - k) * e[k];
        const int64_t Pe = P + e[k];
        runpm = Pe > runpm ? Pe : runpm;
    }
    // Constraint (d)'s limit: drop finished requests from the worker's log and
    // take theta * the smallest slack of the ongoing ones (placed before this
    // heartbeat).  In place, 256 entries at a time: every entry of a chunk is
    // read before any kept one is written, and kept entries only move down.
    double dl = INFINITY;
    if (sc.use_d) {
        int32_t* lge = st.lge + base;
        int32_t* lgw = st.lgw + base;
        double* lgs = st.lgs + base;
        const int L0 = st.lgn[gw];
        int wpos = 0;
        double mn = INFINITY;
        for (int c0 = 0; c0 < L0; c0 += NT) {
            const int k = c0 + tid;
            const bool in = k < L0;
            const int32_t ek = in ? lge[k] : 0, wk = in ? lgw[k] : 0;
            const double sk = in ? lgs[k] : 0.0;
            const bool keep = in && ek >= tau;
            if (keep && wk < hb) mn = fmin(mn, sk);
            int64_t kept;
            const int pos = (int)block_scan_excl<NT, false>(keep ? 1 : 0, 0, OpAdd(), &kept, red);
            if (keep) {
                lge[wpos + pos] = ek;
                lgw[wpos + pos] = wk;
                lgs[wpos + pos] = sk;
            }
            wpos += (int)kept;
            __syncthreads();
        }
        mn = double_of(block_reduce<NT>(ord_of(mn), ord_of(INFINITY), OpMin(), red));
        if (mn != INFINITY) dl = sc.theta * (mn + phi);
        if (tid == 0) st.lgn[gw] = wpos;
    }
    if (tid == 0) st.dlim[gw] = dl;

    __syncthreads();  // first_peak
    const int64_t SC = tot_s + (int64_t)B * tau;
    const int64_t SR = tot_e - (int64_t)B * tau;
    const int64_t DS = (SC << sc.gs) + (int64_t)sc.gn * SR;
    const double rhs = sc.theta * ((sc.tdec - sc.c3) - sc.c2 * (double)(B + 1));
    if (tid == 0) {
        pms[n] = make_int4(totPe == INT64_MIN ? PME_NONE : (int32_t)totPe, NEG, 0, 0);
        const int64_t X = (int64_t)B << sc.gs;
        if (DS >= ((int64_t)1 << 31) || X >= ((int64_t)1 << 31) || DS < 0) raise_error(err, DEV_EOVERFLOW);
        const uint64_t key = (uint64_t)(X * X) + (uint64_t)(DS * DS);
        st.head[gw] = head;
        st.B[gw] = B;
        st.SC[gw] = SC;
        st.SR[gw] = SR;
        st.DS[gw] = DS;
        st.key[gw] = key;
        st.peak[gw] = B > 0 ? (int32_t)totP : 0;
        st.peake[gw] = B > 0 ? first_peak : INT32_MAX;
        st.rhs[gw] = rhs;
    }
    // Breakpoint table (has_table): a histogram of the
    // remaining lengths r = e - tau of the live requests (those below LB_MAX),
    // then an exclusive scan, so that entry v - 1 = the byte offset, from the
    // first live slot's summaries, of the first live slot with r >= v (16
    // bytes per slot before it).
    if (has_table(B, need)) {
        for (int v = tid; v < LB_MAX; v += NT) hist[v] = 0;
        __syncthreads();
        for (int k = head + tid; k < n; k += NT) {
            const int32_t r = e[k] - tau;
            if ((uint32_t)r < (uint32_t)LB_MAX) atomicAdd(&hist[r], 1);
        }
        __syncthreads();
        static_assert((LB_SLOTS - 1) * sizeof(int4) <= 0xFFFF && STAGE_MAX <= LB_SLOTS,
                      "byte offsets of the slots fit 16 bits; every staged worker has a table");
        constexpr int CHV = LB_MAX / NT;  // entries per thread
        int32_t loc = 0;
#pragma unroll
        for (int j = 0; j < CHV; ++j) loc += hist[tid * CHV + j];
        int64_t tot;
        int32_t run = (int32_t)block_scan_excl<NT, false>(loc, 0, OpAdd(), &tot, red);
        uint16_t* out = st.lbt + (int64_t)gw * LB_MAX;
#pragma unroll
        for (int j = 0; j < CHV; ++j) {
            run += hist[tid * CHV + j];  // now: requests with r <= tid * CHV + j
            out[tid * CHV + j] = (uint16_t)(run * (int32_t)sizeof(int4));  // entry v - 1, v = tid * CHV + j + 1
        }
    }
    const bool cur = st.hbs[gw] == hb;
    const Sums u{DS, cur ? st.S1[gw] : 0, cur ? st.S2[gw] : 0, rhs, dl};
    const int wv = wave_id();
    if (wv == 0) {
        build_limits(st, sc, gw, u);
    } else if (wv <= 2 && (need & BUILT_TIES)) {
        build_ties(st, sc, gw, u, wv == 1, err);
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------------------------
// Ingest: validate residents, convert to (e, s) at tau = 0 and sort each worker by e.
constexpr int SORT_MAX = 4096;

__global__ __launch_bounds__(BUILD_THREADS) void k_ingest(State st, const int64_t* res_off,
                                                          const int32_t* lin, const int32_t* lpred,
                                                          const int32_t* gen, const double* tdec)
{
    constexpr int NT = BUILD_THREADS;
    __shared__ uint64_t keys[SORT_MAX];
    __shared__ int64_t red[NT / 64];
    const int gw = blockIdx.x;
    const int tid = threadIdx.x;
    const int64_t r0 = res_off[gw];
    const int R = (int)(res_off[gw + 1] - r0);
    const int64_t base = st.slot_base[gw];
    int32_t* e = st.e + base;
    int32_t* s = st.s + base;
    const int32_t LIM = 1 << 24;

    int64_t bad = 0, tot = 0;
    for (int k = tid; k < R; k += NT) {
        const int32_t a = lin[r0 + k], p = lpred[r0 + k], g = gen[r0 + k];
        const bool ok = a >= 1 && p >= 1 && a <= LIM && p <= LIM && g >= 0 && g < p &&
                        (tdec == nullptr || (isfinite(tdec[r0 + k]) && tdec[r0 + k] >= 0.0));
        bad += ok ? 0 : 1;
        tot += ok ? ((int64_t)a + p) : 0;  // sum of (c + r), an upper bound of the KV peak
    }
    bad = block_reduce<NT>(bad, 0, OpAdd(), red);
    tot = block_reduce<NT>(tot, 0, OpAdd(), red);
    if (bad) {
        if (tid == 0) raise_error(st.err_word, DEV_EINVAL);
        return;
    }
    if (tot > ((int64_t)1 << 30) || R > st.cap[gw]) {
        if (tid == 0) raise_error(st.err_word, R > st.cap[gw] ? DEV_ESLOTS : DEV_EOVERFLOW);
        return;
    }
    auto make_key = [&](int k) -> uint64_t {
        const int32_t a = lin[r0 + k], p = lpred[r0 + k], g = gen[r0 + k];
        const uint32_t ek = (uint32_t)(p - g);  // r at tau = 0
        const uint32_t sk = (uint32_t)(a + g);  // c at tau = 0
        return ((uint64_t)ek << 32) | sk;
    };
    if (R <= SORT_MAX) {
        int P2 = 1;
        while (P2 < R) P2 <<= 1;
        for (int k = tid; k < P2; k += NT) keys[k] = k < R ? make_key(k) : ~(uint64_t)0;
        __syncthreads();
        for (int size = 2; size <= P2; size <<= 1) {
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
                for (int k = tid; k < P2; k += NT) {
                    const int j = k ^ stride;
                    if (j > k) {
                        const bool up = (k & size) == 0;
                        const uint64_t x = keys[k], y = keys[j];
                        if ((x > y) == up) { keys[k] = y; keys[j] = x; }
                    }
                }
                __syncthreads();
            }
        }
        for (int k = tid; k < R; k += NT) {
            e[k] = (int32_t)(keys[k] >> 32);
            s[k] = (int32_t)(keys[k] & 0xffffffffu);
        }
    } else {
        // rank sort: position = number of keys smaller, ties by input index
        for (int k = tid; k < R; k += NT) {
            const uint64_t x = make_key(k);
            int pos = 0;
            for (int j = 0; j < R; ++j) {
                const uint64_t y = make_key(j);
                pos += (y < x || (y == x && j < k)) ? 1 : 0;
            }
            e[pos] = (int32_t)(x >> 32);
            s[pos] = (int32_t)(x & 0xffffffffu);
        }
    }
    // constraint (d)'s log exists only where (d) is checked (a decode worker's
    // model ignores the decode history, and its log arrays hold no slots)
    const bool keep_log = tdec != nullptr && st.scen[0].use_d;
    if (keep_log) {
        // the log, in input order: phi = 0 at load, so each resident's entry
        // holds its slack T_dec * g - t_dec
        const Scen& sc = st.scen[0];
        for (int k = tid; k < R; k += NT) {
            const int32_t p = lpred[r0 + k], g = gen[r0 + k];
            st.lge[base + k] = p - g;  // e at tau = 0
            st.lgw[base + k] = -1;
            st.lgs[base + k] = sc.tdec * (double)g - tdec[r0 + k];
        }
    }
    if (tid == 0) {
        st.n[gw] = R;
        st.head[gw] = 0;
        st.tn[gw] = 0;
        st.built[gw] = 0;
        st.S1[gw] = 0;
        st.S2[gw] = 0;
        st.hbs[gw] = -1;
        st.lgn[gw] = keep_log ? R : 0;
    }
}

// ---------------------------------------------------------------------------------------------
// Does worker gw of scenario s have to be built now?
__device__ __forceinline__ bool must_build(const State& st, int mode, int need, int gw, int s)
{
    const Ctl* c = st.ctl + s;
    if (mode == 2) return true;
    if (c->call != st.call) return false;  // another call's control block
    if (mode == 0) {
        if (c->err || c->start >= c->Q) return false;
        const int32_t built = st.built[gw];
        if ((built & need) == need) {
            if (!c->rebuild) return false;
            // A worker that held no live request at its last build and has taken
            // none since (a placement clears `built`), with no prefill sum, has
            // the same summaries and thresholds at any tau: only the slack clock
            // of constraint (d) moves on (its gain is zero without a batch).
            if (st.B[gw] == 0 && st.S1[gw] == 0) {
                if (lane_id() == 0 && st.scen[s].use_d) st.phi_hb[gw] = c->hb_index;
                return false;
            }
        }
    }
    return true;
}

// mode 1: the workers the last commit round listed; modes 0 and 2: every
// worker (one block each).
__global__ __launch_bounds__(BUILD_THREADS) void k_build(State st, int mode, int need)
{
    int s, gw;
    if (mode == 1) {
        s = blockIdx.x / MAX_DIRTY;
        const int j = blockIdx.x % MAX_DIRTY;
        if (s >= st.S || j >= st.dcount[s]) return;
        gw = st.dlist[s * MAX_DIRTY + j];
        if ((st.built[gw] & need) == need) return;
    } else {
        gw = blockIdx.x;
        s = find_scen_by_worker(st, gw);
    }
    if (!must_build(st, mode, need, gw, s)) return;
    const Scen sc = st.scen[s];
    build_worker(st, sc, gw, st.ctl[s].tau, st.ctl[s].hb_index, need, &st.ctl[s].err);
    if (threadIdx.x == 0) st.built[gw] = need;
}

// The same build by one wave per worker, for workers of at most SMALL_SLOTS
// slots: a block barrier per scan costs such a worker more than the scan.  Lane l
// holds slots 64 c + l in registers; scans are cross-lane, with a carry over
// the chunks c, and everything is 32-bit (a demand is below 2^31, a sum of
// s = c - tau within 2^30 + 2^27); only the sum of the ends is not.
constexpr int SMALL_CH = SMALL_SLOTS / 64;
constexpr int SMALL_WAVES = 4;  // workers per block

struct SmallLDS {
    union {
        struct {
            int32_t e[SMALL_SLOTS], s[SMALL_SLOTS];
        };
        uint16_t mark[LB_MAX];
    };
};

__device__ void build_small(const State& st, const Scen& sc, int gw, int32_t tau, int32_t hb, int need, int32_t* err,
                            SmallLDS& L)
{
    const int lane = lane_id();
    const int64_t base = st.slot_base[gw];
    int n = st.n[gw], head = st.head[gw];
    const int tn = st.tn[gw];
    int32_t e[SMALL_CH], s[SMALL_CH];
    {
        const int N = n - head;
#pragma unroll
        for (int c = 0; c < SMALL_CH; ++c) {
            const int k = c * 64 + lane;
            const bool in = k < N;
            e[c] = in ? st.e[base + head + k] : 0;
            s[c] = in ? st.s[base + head + k] : 0;
        }
        if (tn > 0) {
            // sort the appended requests in: every request's place is counted (see
            // merge_tail), in LDS, and the whole moves to the start of the slot range
            const int cap = st.cap[gw];
            int32_t up[SMALL_CH];
#pragma unroll
            for (int c = 0; c < SMALL_CH; ++c) up[c] = 0;
            for (int t0 = 0; t0 < tn; t0 += 64) {
                auto at = [&](int t) { return n + t > cap ? n + t - (cap + 1) : n + t; };
                const int mt = min(64, tn - t0);
                const int p = at(t0 + min(lane, mt - 1));
                const int32_t x = st.e[base + p], y = st.s[base + p];
                int to = 0;
                for (int j = 0; j < tn; j += 64) {  // against the other appended requests
                    const int mj = min(64, tn - j);
                    const int32_t v = j == t0 ? x : st.e[base + at(j + min(lane, mj - 1))];
                    for (int q = 0; q < mj; ++q) {
                        const int32_t xq = rdlane(v, q);
                        to += (xq < x || (xq == x && j + q < t0 + lane)) ? 1 : 0;
                    }
                }
                for (int q = 0; q < mt; ++q) {  // against the sorted ones
                    const int32_t xq = rdlane(x, q);
                    int above = 0;
#pragma unroll
                    for (int c = 0; c < SMALL_CH; ++c) {
                        if (c * 64 >= N) break;
                        const uint64_t m = ballot(c * 64 + lane < N) & ballot(e[c] > xq);
                        up[c] += __builtin_amdgcn_inverse_ballot_w64(m) ? 1 : 0;
                        above += __popcll(m);
                    }
                    to += lane == q ? N - above : 0;
                }
                if (lane < mt) {
                    L.e[to] = x;
                    L.s[to] = y;
                }
            }
#pragma unroll
            for (int c = 0; c < SMALL_CH; ++c) {
                const int k = c * 64 + lane;
                if (k < N) {
                    L.e[k + up[c]] = e[c];
                    L.s[k + up[c]] = s[c];
                }
            }
            __builtin_amdgcn_wave_barrier();
            n = N + tn;
            head = 0;
#pragma unroll
            for (int c = 0; c < SMALL_CH; ++c) {
                const int k = c * 64 + lane;
                const bool in = k < n;
                e[c] = in ? L.e[min(k, SMALL_SLOTS - 1)] : 0;
                s[c] = in ? L.s[min(k, SMALL_SLOTS - 1)] : 0;
                if (in) {
                    st.e[base + k] = e[c];
                    st.s[base + k] = s[c];
                }
            }
            if (lane == 0) {
                st.n[gw] = n;
                st.tn[gw] = 0;
            }
        }
    }
    const int N = n - head;
    // Constraint (d): the worker's slack gain up to the current heartbeat (see
    // build_worker)
    double phi = 0.0;
    if (sc.use_d) {
        phi = st.phi[gw];
        const int pending = hb - st.phi_hb[gw];
        if (pending < 0) {
            if (lane == 0) raise_error(err, DEV_EINVAL);
        } else {
            for (int p = 0; p < pending; ++p) {
                const int32_t tk = tau - pending + p;
                int cnt = 0;
                int32_t part = 0;
#pragma unroll
                for (int c = 0; c < SMALL_CH; ++c) {
                    const bool in = c * 64 + lane < N && e[c] >= tk;
                    cnt += __popcll(ballot(in));
                    part += in ? s[c] : 0;
                }
                if (cnt == 0) break;  // the live set only shrinks: no later iteration runs a batch
                const int64_t ctx = (int64_t)wave_sum32(part) + (int64_t)cnt * tk;  // sum of the contexts c = s + tau
                const double t_iter = (sc.c3 + sc.c2 * (double)cnt) + sc.k2 * (double)ctx;
                phi = phi + (sc.tdec - t_iter);
            }
            if (lane == 0) {
                st.phi[gw] = phi;
                st.phi_hb[gw] = hb;
            }
        }
    }
    // finished requests form a prefix of the live range (sorted by e)
    int fin = 0;
#pragma unroll
    for (int c = 0; c < SMALL_CH; ++c) fin += __popcll(ballot(c * 64 + lane < N && e[c] < tau));
    const int B = N - fin;
    head += fin;
    // from the last slot down: sums of s, the demands P at the end points, their
    // running maximum
    int32_t P[SMALL_CH], ss[SMALL_CH], sm[SMALL_CH];
    int32_t sum = 0, top = NEG, at = INT32_MAX;
    int64_t se = 0;
#pragma unroll
    for (int c = SMALL_CH - 1; c >= 0; --c) {
        P[c] = NEG;
        ss[c] = sm[c] = 0;
        if (c * 64 >= N) continue;
        const int k = c * 64 + lane;
        const bool in = k >= fin && k < N;
        const int32_t sv = in ? s[c] : 0;
        se += in ? e[c] : 0;
        // (an inclusive scan from lane 0 up; the suffix is what it leaves)
        const int32_t inc = wave_incl_scan(sv, 0, Add32());
        const int32_t all = rdlane(inc, 63);
        ss[c] = sum + all - inc + sv;
        sum += all;
        // (wrap-around arithmetic: the demand itself is below 2^31)
        P[c] = in ? (int32_t)((uint32_t)ss[c] + (uint32_t)(N - k) * (uint32_t)e[c]) : NEG;
        const int32_t chunk = wave_max32(P[c]);
        sm[c] = max(wave_suffix_max(P[c]), top);
        if (chunk >= top && chunk != NEG) at = rdlane(e[c], __builtin_ctzll(ballot(P[c] == chunk)));  // the earliest end
        top = max(top, chunk);
    }
    int32_t pm = NEG;
#pragma unroll
    for (int c = 0; c < SMALL_CH; ++c) {
        if (c * 64 >= N) break;
        const int k = c * 64 + lane;
        const bool in = k >= fin && k < N;
        const int32_t Pe = in ? P[c] + e[c] : NEG;
        const int32_t inc = wave_incl_scan(Pe, NEG, Max32());
        const int32_t below = __shfl_up(inc, 1, 64);  // (every lane takes part)
        const int32_t before = max(pm, lane == 0 ? NEG : below);
        pm = max(pm, rdlane(inc, 63));
        if (in) st.pms[base + head - fin + k] = make_int4(before == NEG ? PME_NONE : before, sm[c], ss[c], N - k);
    }
    double dl = INFINITY;
    if (sc.use_d) {  // constraint (d)'s limit (see build_worker), 64 log entries at a time
        int32_t* lge = st.lge + base;
        int32_t* lgw = st.lgw + base;
        double* lgs = st.lgs + base;
        const int L0 = st.lgn[gw];
        int wpos = 0;
        double mn = INFINITY;
        for (int c0 = 0; c0 < L0; c0 += 64) {
            const int k = c0 + lane;
            const bool in = k < L0;
            const int32_t ek = in ? lge[k] : 0, wk = in ? lgw[k] : 0;
            const double sk = in ? lgs[k] : 0.0;
            const bool keep = in && ek >= tau;
            if (keep && wk < hb) mn = fmin(mn, sk);
            const uint64_t m = ballot(keep);
            if (keep) {  // (kept entries only move down, to places already read)
                const int to = wpos + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
                lge[to] = ek;
                lgw[to] = wk;
                lgs[to] = sk;
            }
            wpos += __popcll(m);
        }
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) mn = fmin(mn, __shfl_xor(mn, d, 64));
        if (mn != INFINITY) dl = sc.theta * (mn + phi);
        if (lane == 0) st.lgn[gw] = wpos;
    }
    const int64_t SC = (int64_t)sum + (int64_t)B * tau;
    const int64_t SR = wave_sum64(se) - (int64_t)B * tau;
    const int64_t DS = (SC << sc.gs) + (int64_t)sc.gn * SR;
    const double rhs = sc.theta * ((sc.tdec - sc.c3) - sc.c2 * (double)(B + 1));
    if (lane == 0) {
        st.pms[base + n] = make_int4(pm == NEG ? PME_NONE : pm, NEG, 0, 0);
        const int64_t X = (int64_t)B << sc.gs;
        if (DS >= ((int64_t)1 << 31) || X >= ((int64_t)1 << 31) || DS < 0) raise_error(err, DEV_EOVERFLOW);
        st.head[gw] = head;
        st.B[gw] = B;
        st.SC[gw] = SC;
        st.SR[gw] = SR;
        st.DS[gw] = DS;
        st.key[gw] = (uint64_t)(X * X) + (uint64_t)(DS * DS);
        st.peak[gw] = B > 0 ? top : 0;
        st.peake[gw] = B > 0 ? at : INT32_MAX;
        st.rhs[gw] = rhs;
        st.dlim[gw] = dl;
    }
    if (has_table(B, need)) {
        // breakpoint table (see build_worker): the requests are sorted, so the last
        // one of each remaining length r marks entry r with the number ending no
        // later, and a running maximum fills the entries between
        for (int v = lane; v < LB_MAX / 8; v += 64) reinterpret_cast<uint4*>(L.mark)[v] = make_uint4(0, 0, 0, 0);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int c = 0; c < SMALL_CH; ++c) {
            if (c * 64 >= N) break;
            const int k = c * 64 + lane;
            const int32_t ahead = c + 1 < SMALL_CH ? rdlane(e[c + 1 < SMALL_CH ? c + 1 : c], 0) : 0;
            const int32_t down = __shfl_down(e[c], 1, 64);
            const int32_t next = lane == 63 ? ahead : down;
            const int32_t r = e[c] - tau;
            if (k >= fin && k < N && r < LB_MAX && (k == N - 1 || next != e[c])) L.mark[r] = (uint16_t)(k - fin + 1);
        }
        __builtin_amdgcn_wave_barrier();
        int32_t run = 0;
        uint4* out = reinterpret_cast<uint4*>(st.lbt + (int64_t)gw * LB_MAX);
#pragma unroll
        for (int q = 0; q < LB_MAX / 512; ++q) {
            const uint4 v = reinterpret_cast<const uint4*>(L.mark)[q * 64 + lane];
            int32_t m[8] = {(int32_t)(v.x & 0xffff), (int32_t)(v.x >> 16), (int32_t)(v.y & 0xffff), (int32_t)(v.y >> 16),
                            (int32_t)(v.z & 0xffff), (int32_t)(v.z >> 16), (int32_t)(v.w & 0xffff), (int32_t)(v.w >> 16)};
#pragma unroll
            for (int u = 1; u < 8; ++u) m[u] = max(m[u], m[u - 1]);
            const int32_t inc = wave_incl_scan(m[7], 0, Max32());
            const int32_t prev = __shfl_up(inc, 1, 64);
            const int32_t carry = max(run, lane == 0 ? 0 : prev);
            run = max(run, rdlane(inc, 63));
            uint32_t o[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)  // byte offsets of the slots' summaries
                o[u] = (uint32_t)(max(m[2 * u], carry) * (int32_t)sizeof(int4)) |
                       ((uint32_t)(max(m[2 * u + 1], carry) * (int32_t)sizeof(int4)) << 16);
            out[q * 64 + lane] = make_uint4(o[0], o[1], o[2], o[3]);
        }
    }
    const bool cur = st.hbs[gw] == hb;
    const Sums u{DS, cur ? st.S1[gw] : 0, cur ? st.S2[gw] : 0, rhs, dl};
    build_limits(st, sc, gw, u);
    if (need & BUILT_TIES) {
        build_ties(st, sc, gw, u, true, err);
        build_ties(st, sc, gw, u, false, err);
    }
}

__global__ __launch_bounds__(64 * SMALL_WAVES) void k_build_small(State st, int mode, int need)
{
    __shared__ SmallLDS L[SMALL_WAVES];
    const int id = blockIdx.x * SMALL_WAVES + __builtin_amdgcn_readfirstlane(wave_id());
    int s, gw;
    if (mode == 1) {
        s = id / MAX_DIRTY;
        const int j = id % MAX_DIRTY;
        if (s >= st.S || j >= st.dcount[s]) return;
        gw = st.dlist[s * MAX_DIRTY + j];
        if ((st.built[gw] & need) == need) return;
    } else {
        gw = id;
        if (gw >= st.NW) return;
        s = find_scen_by_worker(st, gw);
    }
    if (!must_build(st, mode, need, gw, s)) return;
    build_small(st, st.scen[s], gw, st.ctl[s].tau, st.ctl[s].hb_index, need, &st.ctl[s].err,
                L[__builtin_amdgcn_readfirstlane(wave_id())]);
    if (lane_id() == 0) st.built[gw] = need;
}

// ---------------------------------------------------------------------------------------------
// What the pair evaluation needs of one worker, gathered into LDS once per
// block so that the evaluation loop reads no per-worker global data.
struct WInfo {
    int64_t base;  // first live slot
    int64_t DS, S1, S2;
    double rhs;
    int64_t dq_max, ntd_lo, ntd_hi;
    uint64_t ntd_mask, ntt_mask;
    int32_t head, n, M, lthr;  // (one 16-byte read)
    int32_t dq32;    // dq_max - the block's smallest qD, clamped to [-1, 2^31 - 1]
    int32_t nt_any;  // some query of the block's chunk may have a near-tie margin with this worker
    int32_t ntt_lo, ntt_hi, ntp_lo, ntp_hi;
    double dlim;
};

__device__ __forceinline__ View winfo_view(const State& st, const WInfo& wi)
{
    View v;
    v.e = st.e + (wi.base - wi.head);
    v.pms = st.pms + (wi.base - wi.head);
    v.head = wi.head;
    v.n = wi.n;
    v.M = wi.M;
    v.DS = wi.DS;
    v.S1 = wi.S1;
    v.S2 = wi.S2;
    v.key = 0;
    v.rhs = wi.rhs;
    v.dlim = wi.dlim;
    return v;
}

// Block-wide reductions of one int64 per thread (all threads get the result).
template <int NT, typename Op>
__device__ __forceinline__ int64_t block_all(int64_t v, int64_t ident, Op op, int64_t* lds)
{
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v = op(v, __shfl_xor(v, d, 64));
    if (lane_id() == 0) lds[wave_id()] = v;
    __syncthreads();
    int64_t r = ident;
#pragma unroll
    for (int j = 0; j < NT / 64; ++j) r = op(r, lds[j]);
    __syncthreads();
    return r;
}

// v_mul_u32_u24: the product of the low 24 bits of each operand (full rate)
__device__ uint32_t ald_mul_u24(uint32_t a, uint32_t b) __asm("llvm.amdgcn.mul.u24");

// Word `acc` with lane J's value replaced by the wave-uniform `v` (one
// v_writelane_b32 per half, the lane an inline constant, J < 16).
template <int J>
__device__ __forceinline__ uint64_t put_lane_c(uint64_t acc, uint64_t v)
{
    const uint32_t lo = (uint32_t)ald_writelane((int)(uint32_t)v, J, (int)(uint32_t)acc);
    const uint32_t hi = (uint32_t)ald_writelane((int)(uint32_t)(v >> 32), J, (int)(uint32_t)(acc >> 32));
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t put_lane(uint64_t acc, uint64_t v, int j)
{
    switch (j) {
    case 0: return put_lane_c<0>(acc, v);
    case 1: return put_lane_c<1>(acc, v);
    case 2: return put_lane_c<2>(acc, v);
    case 3: return put_lane_c<3>(acc, v);
    case 4: return put_lane_c<4>(acc, v);
    case 5: return put_lane_c<5>(acc, v);
    case 6: return put_lane_c<6>(acc, v);
    case 7: return put_lane_c<7>(acc, v);
    case 8: return put_lane_c<8>(acc, v);
    case 9: return put_lane_c<9>(acc, v);
    case 10: return put_lane_c<10>(acc, v);
    case 11: return put_lane_c<11>(acc, v);
    case 12: return put_lane_c<12>(acc, v);
    case 13: return put_lane_c<13>(acc, v);
    case 14: return put_lane_c<14>(acc, v);
    default: return put_lane_c<15>(acc, v);
    }
}

// Keep a query's two smallest KV excesses as (excess, worker) pairs, smaller
// excess first, then the higher index; e1 = INT32_MAX, w1 = -1 when empty
// (every excess is below INT32_MAX).  IN_ORDER: w is above every index seen so
// far, so an equal excess replaces.
template <bool IN_ORDER>
__device__ __forceinline__ void keep_two(int32_t ex, int32_t w, int32_t& e1, int32_t& w1, int32_t& e2, int32_t& w2)
{
    const bool b1 = IN_ORDER ? ex <= e1 : ((ex < e1) | ((ex == e1) & (w > w1)));
    const bool b2 = IN_ORDER ? ex <= e2 : ((ex < e2) | ((ex == e2) & (w > w2)));
    e2 = b1 ? e1 : (b2 ? ex : e2);
    w2 = b1 ? w1 : (b2 ? w : w2);
    e1 = b1 ? ex : e1;
    w1 = b1 ? w : w1;
}

// One thread's share of a staged worker: slots tid + j * EVAL_THREADS of the
// summaries (clamped to slot B, which exists) and LBV entries of its table.
constexpr int PF_N = (STAGE_MAX + EVAL_THREADS - 1) / EVAL_THREADS;
constexpr int LBV = LB_MAX / EVAL_THREADS;  // table entries per thread (8 or 4)
static_assert(LBV == 8 || LBV == 4, "one 16- or 8-byte table load per thread");
using LBVec = std::conditional_t<LBV == 8, uint4, uint2>;
struct Prefetch {
    int4 p[PF_N];
    LBVec lb;  // LBV entries of the worker's breakpoint table (zeros for an empty worker)
};

__device__ __forceinline__ Prefetch prefetch_worker(const State& st, const WInfo& x, int gw, int tid)
{
    Prefetch f;
    const int B = x.n - x.head;
#pragma unroll
    for (int j = 0; j < PF_N; ++j) f.p[j] = st.pms[x.base + min(tid + j * EVAL_THREADS, B)];
    f.lb = LBVec{};
    if (B > 0) f.lb = reinterpret_cast<const LBVec*>(st.lbt + (int64_t)gw * LB_MAX)[tid];
    return f;
}

// Write one thread's share of a staged worker into LDS: the summaries of
// slots 0 .. B and the table entries below L (the chunk's largest l_pred).
__device__ __forceinline__ void stage_put(uint16_t* LBs, int4* Ss, const Prefetch& pf, int tid, int B, int L)
{
#pragma unroll
    for (int j = 0; j < PF_N; ++j)
        if (tid + j * EVAL_THREADS <= B) Ss[tid + j * EVAL_THREADS] = pf.p[j];
    if (LBV * tid < L) reinterpret_cast<LBVec*>(LBs)[tid] = pf.lb;
}

// First worker at or after j (block-local index) that is evaluated from LDS.
// skip: workers that share another's bit words.
__device__ __forceinline__ int next_staged(const WInfo* Wi, int nw, bool use_lb, uint64_t skip, int j)
{
    if (!use_lb) return nw;
    while (j < nw && (Wi[j].n - Wi[j].head >= STAGE_MAX || ((skip >> j) & 1))) ++j;
    return j;
}

// Ranges of a chunk's query figures, for skipping near-tie work per worker.
struct QRange {
    int64_t qdmin, qdmax, lnmin, lnmax;
};

// Evaluate this thread's queries against one worker and store the wave's bit
// words (lane j < 2 EVAL_QPT stores word j).  STAGED: breakpoint slot from the block's
// table and summaries in LDS; else binary search over global memory.  MODE as
// for launch_eval.  STAGED requires every l_pred + tau of the block below 2^24
// (the count-times-end product takes the full-rate 24-bit multiply).  TAB: an
// unstaged worker with a table is read through it from global memory for the
// queries the table covers (l_pred <= LB_MAX), by a binary search for the rest.
template <int MODE, bool EX, bool STAGED, bool TAB>
__device__ __forceinline__ void eval_worker(const State& st, const Scen& sc, const WInfo& wi, int w, int32_t tau,
                                            const int32_t (&lin)[EVAL_QPT], const int32_t (&lp)[EVAL_QPT],
                                            const bool (&act)[EVAL_QPT], const uint64_t (&am)[EVAL_QPT],
                                            const int32_t (&qd)[EVAL_QPT], int32_t (&e1)[EVAL_QPT],
                                            int32_t (&w1)[EVAL_QPT], int32_t (&e2)[EVAL_QPT],
                                            int32_t (&w2)[EVAL_QPT], uint64_t (&anyb)[EVAL_QPT],
                                            const uint16_t* LBs, const int4* Ss, uint64_t* bdst)
{
    constexpr bool MONO = MODE >= 1;
    const int lane = lane_id();
    const int B = wi.n - wi.head;
    const View v = winfo_view(st, wi);
    // KV peaks first: the table reads of all queries, then their summary reads,
    // so that the LDS latencies overlap
    int32_t peak[EVAL_QPT];
    if (STAGED) {
        int ofs[EVAL_QPT];
        int4 t[EVAL_QPT];
#pragma unroll
        for (int m = 0; m < EVAL_QPT; ++m) ofs[m] = LBs[lp[m] - 1];  // byte offset of the first slot ending at or after the query
#pragma unroll
        for (int m = 0; m < EVAL_QPT; ++m) t[m] = *reinterpret_cast<const int4*>(reinterpret_cast<const char*>(Ss) + ofs[m]);
#pragma unroll
        for (int m = 0; m < EVAL_QPT; ++m) {
            // every candidate below is a KV demand with the query added, so it
            // lies under the worker's peak (<= 2^30) plus l_in + l_pred: 32-bit
            // wrap-around arithmetic gives it exactly (t.w = live slots from
            // the breakpoint on, below STAGE_MAX)
            const uint32_t sq = (uint32_t)(lin[m] - tau), eq = (uint32_t)(lp[m] + tau);
            const uint32_t ne = ald_mul_u24((uint32_t)t[m].w, eq);
            const int32_t a = (int32_t)((uint32_t)t[m].x + sq);
            const int32_t c = (int32_t)((uint32_t)t[m].z + ne + sq + eq);
            const int32_t p = a > t[m].y ? a : t[m].y;
            peak[m] = p > c ? p : c;
        }
    } else if (TAB && B < LB_SLOTS) {
        // two dependent reads per query, table entry then summaries (32-bit
        // wrap-around arithmetic as above, with a full 32-bit multiply); a
        // query past the table's range searches
        const uint16_t* tb = st.lbt + (int64_t)(sc.wbase + w) * LB_MAX;
        int kq[EVAL_QPT];
#pragma unroll
        for (int m = 0; m < EVAL_QPT; ++m) kq[m] = (B > 0 && lp[m] <= LB_MAX) ? tb[lp[m] - 1] / (int)sizeof(int4) : 0;
        int4 t[EVAL_QPT];
#pragma unroll
        for (int m = 0; m < EVAL_QPT; ++m) t[m] = v.pms[v.head + kq[m]];
#pragma unroll
        for (int m = 0; m < EVAL_QPT; ++m) {
            const uint32_t sq = (uint32_t)(lin[m] - tau), eq = (uint32_t)(lp[m] + tau);
            const int32_t a = (int32_t)((uint32_t)t[m].x + sq);
            const int32_t c = (int32_t)((uint32_t)t[m].z + (uint32_t)t[m].w * eq + sq + eq);
            const int32_t p = a > t[m].y ? a : t[m].y;
            peak[m] = p > c ? p : c;
            if (lp[m] > LB_MAX) peak[m] = (int32_t)kv_peak_with(v, lin[m] - tau, lp[m] + tau);
        }
    } else {
#pragma unroll
        for (int m = 0; m < EVAL_QPT; ++m) peak[m] = (int32_t)kv_peak_with(v, lin[m] - tau, lp[m] + tau);
    }
    uint64_t bits = 0;  // lane j < 2 EVAL_QPT: the word it stores
    if (MONO) {
        // feasibility from the integer thresholds (the worker's figures read
        // once; no short-circuit, so no branch per query)
        const int32_t M = wi.M, lthr = wi.lthr;
#pragma unroll
        for (int m = 0; m < EVAL_QPT; ++m) {
            // constraint (b) as qD <= dq_max: staged, relative to the block's
            // smallest qD in 32 bits (the block's qD span is below 2^31)
            const bool bok = STAGED ? qd[m] <= wi.dq32
                                    : ((int64_t)lin[m] << sc.gs) + (int64_t)sc.gn * lp[m] <= wi.dq_max;
            // one ballot per compare: each compare's lane mask is its ballot
            const uint64_t bf = am[m] & ballot(peak[m] <= M) & ballot(bok) & ballot(lin[m] <= lthr);
            bits = put_lane(bits, bf, m);
            anyb[EX ? 0 : m] |= bf;
            if (EX) keep_two<STAGED>(peak[m] - M, w, e1[m], w1[m], e2[m], w2[m]);
        }
        // near-tie words (lanes EVAL_QPT .. 2 EVAL_QPT - 1) stay zero here: near_tie_words fills
        // them in for the workers with nt_any
    } else {
#pragma unroll
        for (int m = 0; m < EVAL_QPT; ++m) {
            const Latency Lt = latency(sc, v, lin[m], lp[m], B + 1);
            const uint64_t bf = ballot(act[m] && peak[m] <= wi.M && Lt.dec_ok && Lt.ttft_ok);
            const uint64_t bn = ballot(act[m] && Lt.nt);
            bits = put_lane(bits, bf, m);
            anyb[EX ? 0 : m] |= bf;
            bits = put_lane(bits, bn, m + EVAL_QPT);
            if (EX) keep_two<STAGED>(peak[m] - wi.M, w, e1[m], w1[m], e2[m], w2[m]);
        }
    }
    if (lane < 2 * EVAL_QPT) bdst[w] = bits;
}

// Near-tie words of one worker (lanes EVAL_QPT .. 2 EVAL_QPT - 1 store the
// wave's words for its queries m = lane - EVAL_QPT), with the integer thresholds (MODE >= 1): from the
// worker's exact near-tie sets (MODE 2) or by the fp64 margin tests of the
// queries inside a tie band (MODE 1).  Independent of the KV peak, so it runs
// after the staged loop, apart from its registers.
template <int MODE>
__device__ __forceinline__ void near_tie_words(const State& st, const Scen& sc, const WInfo& wi, int w,
                                               const int32_t (&lin)[EVAL_QPT], const int32_t (&lp)[EVAL_QPT],
                                               const bool (&act)[EVAL_QPT], uint64_t* bdst)
{
    const int lane = lane_id();
    const View v = winfo_view(st, wi);
    const int B = wi.n - wi.head;
    uint64_t bits = 0;
#pragma unroll
    for (int m = 0; m < EVAL_QPT; ++m) {
        const int64_t qD = ((int64_t)lin[m] << sc.gs) + (int64_t)sc.gn * lp[m];
        bool nt;
        if (MODE == 2) {
            const uint64_t dd = (uint64_t)(qD - wi.ntd_lo);
            const uint32_t dl = (uint32_t)(lin[m] - wi.ntt_lo);
            nt = (dd < 64 && ((wi.ntd_mask >> dd) & 1)) || (dl < 64 && ((wi.ntt_mask >> dl) & 1));
        } else {
            const bool maybe = (qD >= wi.ntd_lo && qD <= wi.ntd_hi) || (lin[m] >= wi.ntt_lo && lin[m] <= wi.ntt_hi) ||
                               (lin[m] >= wi.ntp_lo && lin[m] <= wi.ntp_hi);
            nt = maybe && latency(sc, v, lin[m], lp[m], B + 1).nt;
        }
        const uint64_t bn = ballot(act[m] && nt);
        bits = put_lane(bits, bn, m + EVAL_QPT);
    }
    if (lane >= EVAL_QPT && lane < 2 * EVAL_QPT) bdst[w] = bits;
}

// Sorted layout (a one-scenario tile with State::qorig): the order in which
// the block evaluates its chunk of EVAL_Q queries, by l_pred in buckets of 8
// (the last bucket also takes every l_pred above 2032), ties by arrival, the
// chunk's missing queries (offsets >= nact) last, so that the lanes of a wave
// read neighbouring breakpoint entries and summaries.  Every worker block of
// the chunk computes the same order.  A stable counting sort: the lanes of a
// wave with the same bucket find each other by eight ballots (one per key
// bit); a histogram per (segment of 64 offsets, bucket) and one scan over the
// buckets give each query its position.  On return o[m] is the chunk offset
// of the query at position m * NT + tid (its lengths are then read again:
// passing them through LDS, or holding them through the sort, measured
// slower); the chunk's first worker block writes the tile's permutation
// (qorig, qpos).  `sh`: 10 KB of scratch (histogram, then the permutation);
// `red` that of block_scan_excl.
template <int QPT>
__device__ __forceinline__ void sort_chunk(const State& st, const Scen& sc, int start, int q0, int nact, bool writer,
                                           int (&o)[QPT], uint16_t* sh, int64_t* red)
{
    constexpr int NT = EVAL_THREADS;
    constexpr int NB = 256;                 // buckets (one per thread for the scan)
    constexpr int NS = QPT * (NT / 64);     // segments of 64 offsets: segment m * 4 + wave
    static_assert(NT == NB, "one bucket per thread");
    uint16_t* H = sh;                       // [NS][NB] counts, then positions
    uint16_t* perm = sh + NS * NB;          // sorted position -> chunk offset
    const int tid = threadIdx.x, lane = lane_id(), wv = wave_id();
    const uint64_t below = (1ull << lane) - 1;
    for (int k = tid; k < NS * NB / 4; k += NT) reinterpret_cast<uint64_t*>(H)[k] = 0;
    int key[QPT];
#pragma unroll
    for (int m = 0; m < QPT; ++m) {
        const int off = m * NT + tid;
        const bool in = off < nact;
        const int32_t l = in ? st.q_lpred[q_at(sc, q0 + off)] : 1;
        // (an invalid length, which fails the call, still gets a bucket)
        key[m] = in ? min(max(l - 1, 0) >> 3, NB - 2) : NB - 1;
    }
    __syncthreads();
    int rank[QPT];
#pragma unroll
    for (int m = 0; m < QPT; ++m) {
        uint64_t peers = ~0ull;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool kb = (key[m] >> b) & 1;
            const uint64_t bb = ballot(kb);
            peers &= kb ? bb : ~bb;
        }
        rank[m] = __popcll(peers & below);
        if (rank[m] == 0) H[(m * (NT / 64) + wv) * NB + key[m]] = (uint16_t)__popcll(peers);
    }
    __syncthreads();
    int64_t cnt = 0;
    for (int sg = 0; sg < NS; ++sg) cnt += H[sg * NB + tid];
    int64_t all;
    int64_t at = block_scan_excl<NT, false>(cnt, 0, OpAdd(), &all, red);
    for (int sg = 0; sg < NS; ++sg) {
        const int n = H[sg * NB + tid];
        H[sg * NB + tid] = (uint16_t)at;
        at += n;
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < QPT; ++m) perm[H[(m * (NT / 64) + wv) * NB + key[m]] + rank[m]] = (uint16_t)(m * NT + tid);
    __syncthreads();
    const int t0 = q0 - start;  // the chunk's first tile offset
#pragma unroll
    for (int m = 0; m < QPT; ++m) {
        const int p = m * NT + tid;
        const int off = perm[p];
        o[m] = off;
        if (writer && p < nact) {
            st.qorig[t0 + p] = t0 + off;
            st.qpos[t0 + off] = t0 + p;
        }
    }
    __syncthreads();  // the scratch is the staging area of the evaluation
}

// Write the block's workers (those of this chunk's or group's share) into the
// rank order, and (empties) the place of the first one without a request.
// One wave; nw <= 64.
__device__ __forceinline__ void publish_ranks(const State& st, const Scen& sc, int s, int nw, int wbeg, int share,
                                              int mine, const int32_t* rk, const uint64_t* wkey, bool empties)
{
    const int j = lane_id();
    const bool in = j < nw && j % share == mine;
    if (in) st.order[sc.wbase + rk[j]] = wbeg + j;
    if (empties && sc.uniform_M) {
        const uint64_t m = ballot(in && wkey[min(j, nw - 1)] == 0);
        if (m != 0 && j == __builtin_ctzll(m)) atomicMin(&st.tinfo[s].empty_rank, rk[j]);
    }
}

// How many of the wave's keys (key kk of worker k, where k < W) rank before
// worker j of key kj: larger first, the lower index among equal ones.
__device__ __forceinline__ int count_before(uint64_t kk, int k, int W, uint64_t kj, int j)
{
    return __popcll(ballot(k < W) & (ballot(kk > kj) | (ballot(kk == kj) & ballot(k < j))));
}

// Pair evaluation: block = (scenario, worker block, chunk of EVAL_Q queries).
// Thread t holds queries t, t + 256, t + 512, t + 768 of the chunk.  For each
// worker of the block, its summaries and breakpoint table (built with the
// summaries) are staged in LDS; a query's breakpoint slot is then one table
// read, l = LB[l_pred - 1], and the summaries of slot l give the KV peak with the
// query added.  The next worker's data travels in registers while the current
// one is evaluated.  Workers with B >= STAGE_MAX, or chunks with an l_pred above
// LB_MAX, take the binary search over global memory instead.  MODE: how the
// latency checks are taken (launch_eval); EX: the two smallest KV excesses are
// tracked (diagnostics); TAB: unstaged workers are read through their tables.
template <int MODE, bool EX, bool TAB = false>
__global__ __launch_bounds__(EVAL_THREADS) __attribute__((amdgpu_waves_per_eu((MODE == 2 && !TAB) ? 5 : 4))) void
k_eval(State st)
{
    constexpr int NT = EVAL_THREADS;
    constexpr int QPT = EVAL_QPT;
    static_assert(2 * QPT <= 16, "lane words by put_lane");
    __shared__ uint16_t LBs[LB_MAX];               // the worker's breakpoint table
    __shared__ int4 Ss[PF_N * NT];                 // pms of live slot k, k = 0..B
    __shared__ WInfo Wi[EVAL_WPB_MAX];
    __shared__ int32_t rk[EVAL_WPB_MAX];           // the workers' ranks
    __shared__ uint64_t wkey[EVAL_WPB_MAX];        // and rank keys
    __shared__ uint16_t chunk_at[EVAL_Q];          // chunk offset of the query at each position
    __shared__ int64_t red[NT / 64];
    static_assert(sizeof(Ss) >= 10 * 1024, "the sort's scratch");

    const int s = find_scen<&Scen::eval_blk0>(st, blockIdx.x);
    const Scen sc = st.scen[s];
    const Ctl* cp = st.ctl + s;
    const int32_t start = cp->start, Q = cp->Q;
    const bool mine = cp->call == st.call;
    if (st.qbad != nullptr && start == 0 && mine) {
        // first round of a one-scenario call: check every query length of the
        // call before the first commit can run (grid-stride over all queries)
        bool bad = false;
        for (int64_t i = (int64_t)blockIdx.x * EVAL_THREADS + threadIdx.x; i < Q; i += (int64_t)gridDim.x * EVAL_THREADS) {
            const int32_t a = st.q_lin[i], p = st.q_lpred[i];
            bad = bad || !(a >= 1 && p >= 1 && a <= (1 << 24) && p <= (1 << 24));
        }
        if (ballot(bad) != 0 && lane_id() == 0) atomicOr(st.qbad, 1);
    }
    if (cp->err || start >= Q || !mine) return;
    const int32_t end = tile_end(start, Q, cp->T, cp->H, cp->since_hb, cp->hb_next);
    const int local = blockIdx.x - sc.eval_blk0;
    const int wb = local % sc.nblk;
    const int qc = local / sc.nblk;
    const int q0 = start + qc * EVAL_Q;
    if (q0 >= end) return;
    const int32_t tau = cp->tau, hb = cp->hb_index;
    const int tid = threadIdx.x;
    const int lane = lane_id();

    // Thread tid evaluates chunk positions m * NT + tid: the queries in
    // arrival order, or (sorted layout) in order of l_pred
    int o[QPT];  // chunk offset of the query at position m * NT + tid
#pragma unroll
    for (int m = 0; m < QPT; ++m) o[m] = m * NT + tid;
    if (st.qorig != nullptr)
        sort_chunk<QPT>(st, sc, start, q0, min(EVAL_Q, end - q0), wb == 0, o, reinterpret_cast<uint16_t*>(Ss), red);
    // (kept in LDS for the end: registers held over the loop cost a wave per SIMD)
#pragma unroll
    for (int m = 0; m < QPT; ++m) chunk_at[m * NT + tid] = (uint16_t)o[m];
    int32_t lin[QPT], lp[QPT];
    bool act[QPT];
    int32_t e1[QPT], w1[QPT], e2[QPT], w2[QPT];  // two smallest KV excesses per query
    int64_t lpmax = 0, qdmin = INT64_MAX, qdmax = INT64_MIN, lnmin = INT64_MAX, lnmax = INT64_MIN;
#pragma unroll
    for (int m = 0; m < QPT; ++m) {
        act[m] = q0 + m * NT + tid < end;
        lin[m] = act[m] ? st.q_lin[q_at(sc, q0 + o[m])] : 1;
        lp[m] = act[m] ? max(st.q_lpred[q_at(sc, q0 + o[m])], 1) : 1;  // (an invalid length fails the call)
        e1[m] = e2[m] = INT32_MAX;
        w1[m] = w2[m] = -1;
        const int64_t qD = ((int64_t)lin[m] << sc.gs) + (int64_t)sc.gn * lp[m];
        if (act[m]) {
            lpmax = lp[m] > lpmax ? lp[m] : lpmax;
            qdmin = qD < qdmin ? qD : qdmin;
            qdmax = qD > qdmax ? qD : qdmax;
            lnmin = lin[m] < lnmin ? lin[m] : lnmin;
            lnmax = lin[m] > lnmax ? lin[m] : lnmax;
        }
    }
    uint64_t am[QPT];  // the wave's lanes holding a query m
#pragma unroll
    for (int m = 0; m < QPT; ++m) am[m] = ballot(act[m]);
    lpmax = block_all<NT>(lpmax, 0, OpMax(), red);
    QRange qr;
    qr.qdmin = block_all<NT>(qdmin, INT64_MAX, OpMin(), red);
    qr.qdmax = block_all<NT>(qdmax, INT64_MIN, OpMax(), red);
    qr.lnmin = block_all<NT>(lnmin, INT64_MAX, OpMin(), red);
    qr.lnmax = block_all<NT>(lnmax, INT64_MIN, OpMax(), red);
    const int L = (int)lpmax;  // table covers v = 0 .. L
    // staging needs the table to cover every l_pred of the block, every
    // eq = l_pred + tau (idle lanes: 1 + tau) below 2^24 for the 24-bit
    // multiply, and the block's qD within a 2^31 span
    const bool use_lb = L <= LB_MAX && (int64_t)max(L, 1) + tau < ((int64_t)1 << 24) &&
                        qr.qdmax - qr.qdmin < ((int64_t)1 << 31);
    int32_t qd[QPT];  // qD - the block's smallest (idle lanes: anything; masked)
#pragma unroll
    for (int m = 0; m < QPT; ++m)
        qd[m] = (int32_t)(((int64_t)lin[m] << sc.gs) + (int64_t)sc.gn * lp[m] - qr.qdmin);

    const int wbeg = wb * sc.wpb;
    const int nw = min(sc.W, wbeg + sc.wpb) - wbeg;
    if (tid < nw) {
        const int gw = sc.wbase + wbeg + tid;
        WInfo x;
        x.head = st.head[gw];
        x.n = st.n[gw];
        x.base = st.slot_base[gw] + x.head;
        x.M = st.M[gw];
        x.DS = st.DS[gw];
        const bool cur = st.hbs[gw] == hb;
        x.S1 = cur ? st.S1[gw] : 0;
        x.S2 = cur ? st.S2[gw] : 0;
        x.rhs = st.rhs[gw];
        x.dq_max = st.dq_max[gw];
        const int64_t dqr = x.dq_max - qr.qdmin;
        x.dq32 = dqr < 0 ? -1 : (dqr > INT32_MAX ? INT32_MAX : (int32_t)dqr);
        x.ntd_lo = st.ntd_lo[gw];
        x.ntd_hi = st.ntd_hi[gw];
        x.lthr = st.lthr[gw];
        x.ntt_lo = st.ntt_lo[gw];
        x.ntt_hi = st.ntt_hi[gw];
        x.ntd_mask = st.ntd_mask[gw];
        x.ntt_mask = st.ntt_mask[gw];
        // constraint (d) never runs with the integer near-tie sets (mode 2)
        x.dlim = MODE == 2 ? INFINITY : st.dlim[gw];
        x.ntp_lo = MODE == 2 ? 1 : st.ntp_lo[gw];
        x.ntp_hi = MODE == 2 ? 0 : st.ntp_hi[gw];
        // a near-tie margin needs some query of the chunk inside a tie band
        x.nt_any = MODE == 0 || (qr.qdmax >= x.ntd_lo && qr.qdmin <= x.ntd_hi) ||
                   (qr.lnmax >= x.ntt_lo && qr.lnmin <= x.ntt_hi) || (qr.lnmax >= x.ntp_lo && qr.lnmin <= x.ntp_hi);
        Wi[tid] = x;
        rk[tid] = 0;
        wkey[tid] = st.key[gw];
    }
    __syncthreads();

    // Algorithm 1's rank of the block's workers at tile start, for the commit: a
    // worker's place is the number of workers that rank before it.  The chunks
    // of the tile share the block's workers out among them, so that a tile of
    // many chunks pays for it once.  Eight keys per thread at a time.  (With
    // diagnostics the selection does this: here it would cost a wave per SIMD.)
    const int nqc = (end - start + EVAL_Q - 1) / EVAL_Q;
    if (!EX && qc < nw) {
        for (int k0 = 0; k0 < sc.W; k0 += NT * 8) {
            uint64_t kk[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) kk[u] = st.key[sc.wbase + min(k0 + u * NT + tid, sc.W - 1)];
            for (int j = qc; j < nw; j += nqc) {
                const uint64_t kj = wkey[j];
                int cnt = 0;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (k0 + u * NT < sc.W) cnt += count_before(kk[u], k0 + u * NT + tid, sc.W, kj, wbeg + j);
                }
                if (lane == 0) atomicAdd(&rk[j], cnt);
            }
        }
    }

    // The next worker's e column and summaries travel in registers while the
    // current one is evaluated.  Plain loads of clamped (in-range) slots, masked
    // only where they are used, so nothing waits for them before then.
    Prefetch pf;
    // bit word of (query group, worker) for lane j < 2 QPT of each wave:
    // feasibility (j < QPT) or near-tie (j >= QPT) of the wave's queries m = j % QPT
    const int64_t brow = sc.bits_off + (int64_t)(((q0 - start) >> 6) + wave_id() + (lane % QPT) * (NT / 64)) * sc.W;
    uint64_t* const bdst = (lane < QPT ? st.bits_feas : st.bits_nt) + brow;

    // the wave's queries that some worker of the block can take (with EX only
    // whether there are any, in anyb[0])
    uint64_t anyb[QPT];
#pragma unroll
    for (int m = 0; m < QPT; ++m) anyb[m] = 0;
    // Workers without a request are all alike where the capacity is one (no
    // placement's prefill is counted on them either: its request would still be
    // there); the block's first stands for the others, and the scenario's first
    // is found by its rank.
    uint64_t empty = 0;
    if (!EX && sc.uniform_M) {
        empty = ballot(lane < nw && wkey[min(lane, nw - 1)] == 0);  // (an empty worker's rank key)
        empty &= empty - 1;
    }
    int cur = next_staged(Wi, nw, use_lb, empty, 0);
    if (cur < nw) pf = prefetch_worker(st, Wi[cur], sc.wbase + wbeg + cur, tid);
    while (cur < nw) {
        __syncthreads();  // the previous worker's readers of LBs / Ss are done
        stage_put(LBs, Ss, pf, tid, Wi[cur].n - Wi[cur].head, L);
        __syncthreads();
        const int nxt = next_staged(Wi, nw, use_lb, empty, cur + 1);
        if (nxt < nw) pf = prefetch_worker(st, Wi[nxt], sc.wbase + wbeg + nxt, tid);
        eval_worker<MODE, EX, true, false>(st, sc, Wi[cur], wbeg + cur, tau, lin, lp, act, am, qd, e1, w1, e2, w2,
                                           anyb, LBs, Ss, bdst);
        cur = nxt;
    }
    // workers too large to stage: binary search over global memory
    for (int j0 = 0; j0 < nw; ++j0) {
        const WInfo wi = Wi[j0];
        if ((use_lb && wi.n - wi.head < STAGE_MAX) || ((empty >> j0) & 1)) continue;
        eval_worker<MODE, EX, false, TAB>(st, sc, wi, wbeg + j0, tau, lin, lp, act, am, qd, e1, w1, e2, w2, anyb, LBs,
                                          Ss, bdst);
    }
    // the tile's queries with a feasible worker, and the first of them
    if (EX) {
        // (from the wave's own bit words: where the tile is long and the cluster
        // full, as in admission control, there are none, and the masks would cost
        // the loop a wave per SIMD in registers)
        if (anyb[0] != 0) {
            __builtin_amdgcn_s_waitcnt(0);  // they have left
            uint64_t v[QPT];
#pragma unroll
            for (int m = 0; m < QPT; ++m) {
                const int g = ((q0 - start) >> 6) + wave_id() + m * (NT / 64);
                const uint64_t* row = st.bits_feas + sc.bits_off + (int64_t)g * sc.W + wbeg;
                v[m] = lane < nw ? __hip_atomic_load(row + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
            }
#pragma unroll
            for (int m = 0; m < QPT; ++m) anyb[m] = wave_or64(v[m]);
        }
    }
    int32_t first = INT32_MAX;
#pragma unroll
    for (int m = 0; m < QPT; ++m) {
        if (anyb[m] == 0) continue;  // wave-uniform
        if (lane == 0)
            atomicOr((unsigned long long*)&st.any[sc.any_off + ((q0 - start) >> 6) + wave_id() + m * (NT / 64)],
                     (unsigned long long)anyb[m]);
        if ((anyb[m] >> lane) & 1) first = min(first, q0 + chunk_at[m * NT + tid]);
    }
    first = wave_min32(first);
    if (lane == 0 && first != INT32_MAX) atomicMin(&st.tinfo[s].first_pc, first);
    __syncthreads();
    if (!EX && wave_id() == 0) publish_ranks(st, sc, s, nw, wbeg, nqc, qc, rk, wkey, true);
    if (MODE >= 1 && EX) {  // near-tie margins feed only the diagnostics
        for (int j0 = 0; j0 < nw; ++j0)
            if (Wi[j0].nt_any) near_tie_words<MODE>(st, sc, Wi[j0], wbeg + j0, lin, lp, act, bdst);
    }
    if (!EX) return;
#pragma unroll
    for (int m = 0; m < QPT; ++m) {
        const int qi = q0 + m * NT + tid;
        const uint64_t k1 = w1[m] < 0 ? ~0ull : ex_key(e1[m], w1[m]);
        const uint64_t k2 = w2[m] < 0 ? ~0ull : ex_key(e2[m], w2[m]);
        if (act[m]) st.part[sc.part_off + (int64_t)wb * sc.pstride + (qi - start)] = make_ulonglong2(k1, k2);
    }
}

// ---------------------------------------------------------------------------------------------
// Pair evaluation of short tiles (at most SHORT_TILE queries: heartbeats cut the
// tiles of a serving stream to the queries of one decode iteration).  A block of
// k_eval is laid out for 1,024 queries and stages every worker's summaries
// through LDS; with 15 to 100 queries nearly all of its lanes idle and the
// staging is the cost.  Here a block takes one 64-query group and wpb workers, a
// wave a quarter of them: a lane holds one query, finds its breakpoint slot by a
// binary search of the worker's ends in LDS (workers below SHORT_STAGE requests,
// which then need no table; larger ones through their tables) and reads the
// slot's summaries from global memory, four workers at a time.  What bounds it:
// the dependent reads of one block, so few workers per wave and many blocks.  With diagnostics (EX) the block also leaves, per
// query, its two smallest KV excesses and its feasible and near-tie counts,
// which the commit merges itself.
constexpr int SHORT_SPAN = SHORT_WPB / (EVAL_THREADS / 64);  // workers per wave
static_assert(SHORT_SPAN <= 64, "one lane per worker");

// saturated to int32 (comparisons against other saturated values stay conservative)
__device__ __forceinline__ int32_t sat32(int64_t x)
{
    return x > INT32_MAX ? INT32_MAX : (x < INT32_MIN ? INT32_MIN : (int32_t)x);
}

template <int MODE, bool EX>
__global__ __launch_bounds__(EVAL_THREADS) void k_eval_short(State st)
{
    constexpr int NT = EVAL_THREADS, NWV = NT / 64;
    __shared__ int32_t rk[SHORT_WPB];
    __shared__ uint64_t wkey[SHORT_WPB];
    __shared__ uint64_t anyw[NWV];
    struct Two {
        uint64_t k1, k2;
        int32_t nfeas, ntcnt;
    };
    __shared__ Two two[NWV][64];
    constexpr int U = 4;  // workers in flight
    __shared__ int32_t ends[NWV][U][SHORT_STAGE];
    const int s = find_scen<&Scen::eval_blk0>(st, blockIdx.x);
    const Scen sc = st.scen[s];
    const Ctl* cp = st.ctl + s;
    const int32_t start = cp->start, Q = cp->Q;
    const bool mine = cp->call == st.call;
    if (st.qbad != nullptr && start == 0 && mine) {
        // first round of a one-scenario call: check every query length of the
        // call before the first commit can run (grid-stride over all queries)
        bool bad = false;
        for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < Q; i += (int64_t)gridDim.x * NT) {
            const int32_t a = st.q_lin[i], p = st.q_lpred[i];
            bad = bad || !(a >= 1 && p >= 1 && a <= (1 << 24) && p <= (1 << 24));
        }
        if (ballot(bad) != 0 && lane_id() == 0) atomicOr(st.qbad, 1);
    }
    if (cp->err || start >= Q || !mine) return;
    const int32_t end = tile_end(start, Q, cp->T, cp->H, cp->since_hb, cp->hb_next);
    const int local = blockIdx.x - sc.eval_blk0;
    const int wb = local % sc.nblk, g = local / sc.nblk;
    const int q0 = start + g * 64;
    if (q0 >= end) return;
    const int ngr = (end - start + 63) >> 6;
    const int32_t tau = cp->tau, hb = cp->hb_index;
    const int tid = threadIdx.x, lane = lane_id(), wv = wave_id();
    const int wbeg = wb * sc.wpb, nw = min(sc.W, wbeg + sc.wpb) - wbeg;
    // this wave's workers: w0 .. w0 + nk - 1, lane k holding worker k's figures
    const int span = (nw + NWV - 1) / NWV;
    const int w0 = wbeg + wv * span;
    const int nk = max(0, min(span, wbeg + nw - w0));
    const int gwk = sc.wbase + min(w0 + min(lane, max(nk - 1, 0)), sc.W - 1);
    const int32_t fhead = st.head[gwk], fn = st.n[gwk], fM = st.M[gwk], flthr = st.lthr[gwk];
    const int64_t fbase = st.slot_base[gwk] + fhead, fdq = st.dq_max[gwk];
    const int32_t fB = fn - fhead;
    if (tid < nw) {
        rk[tid] = 0;
        wkey[tid] = st.key[sc.wbase + wbeg + tid];
    }
    // the workers to evaluate (of those without a request, see k_eval, the wave's
    // first stands for the others)
    uint64_t left = nk > 0 ? ~0ull >> (64 - nk) : 0;
    if (!EX && sc.uniform_M) {
        const uint64_t empty = left & ballot(fB == 0);
        left &= ~(empty & (empty - 1));
    }
    // this lane's query
    const bool act = q0 + lane < end;
    const int64_t qi = q_at(sc, min(q0 + lane, end - 1));
    const int32_t lin = act ? st.q_lin[qi] : 1;
    const int32_t lp = act ? max(st.q_lpred[qi], 1) : 1;  // (an invalid length fails the call)
    const int64_t qD = ((int64_t)lin << sc.gs) + (int64_t)sc.gn * lp;
    const uint32_t sq = (uint32_t)(lin - tau), eq = (uint32_t)(lp + tau);
    const uint64_t am = ballot(act);
    // the next workers (the last one again where fewer are left) and their first
    // 64 ends, in flight early
    int kx[U], kn = 0;
    int32_t pre[U];
    auto prefetch = [&]() {
        kn = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            kn += left != 0 ? 1 : 0;
            kx[u] = left != 0 ? __builtin_ctzll(left) : (u > 0 ? kx[u > 0 ? u - 1 : 0] : 0);
            left &= left - 1;
            pre[u] = (st.e + rdlane64s(fbase, kx[u]))[max(min(lane, rdlane(fB, kx[u]) - 1), 0)];
        }
    };
    prefetch();
    __syncthreads();
    // Algorithm 1's rank of the block's workers at tile start (the number of
    // workers that rank before it), shared out over the tile's groups
    if (g < nw) {
        for (int k0 = 0; k0 < sc.W; k0 += NT * 8) {
            uint64_t kk[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) kk[u] = st.key[sc.wbase + min(k0 + u * NT + tid, sc.W - 1)];
            for (int j = g; j < nw; j += ngr) {
                const uint64_t kj = wkey[j];
                int cnt = 0;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (k0 + u * NT < sc.W) cnt += count_before(kk[u], k0 + u * NT + tid, sc.W, kj, wbeg + j);
                }
                if (lane == 0) atomicAdd(&rk[j], cnt);
            }
        }
    }
    // workers whose tie bands some query of the group may lie in
    uint64_t tied = 0;
    if (EX && MODE >= 1) {
        const int32_t qs = sat32(qD);
        const int32_t qmin = wave_min32(act ? qs : INT32_MAX), qmax = wave_max32(act ? qs : INT32_MIN);
        const int32_t lmin = wave_min32(act ? lin : INT32_MAX), lmax = wave_max32(act ? lin : INT32_MIN);
        bool t = (qmax >= sat32(st.ntd_lo[gwk]) && qmin <= sat32(st.ntd_hi[gwk])) ||
                 (lmax >= st.ntt_lo[gwk] && lmin <= st.ntt_hi[gwk]);
        // (constraint (d) never runs with the integer near-tie sets, mode 2)
        if (MODE == 1) t = t || (lmax >= st.ntp_lo[gwk] && lmin <= st.ntp_hi[gwk]);
        tied = ballot(lane < nk && t);
    }
    uint64_t wf = 0, wn = 0;  // lane k: worker k's bit words
    uint64_t anyf = 0;
    int32_t nfeas = 0, ntcnt = 0;
    int32_t e1 = INT32_MAX, w1 = -1, e2 = INT32_MAX, w2 = -1;
    while (kn > 0) {  // (an empty worker's first end is never compared)
        int k4[U];
        const int n4 = kn;
#pragma unroll
        for (int u = 0; u < U; ++u) k4[u] = kx[u];
        int at[U];  // first live slot ending at or after the query
        int4 t[U];
        int most = 0;  // of the workers staged
        bool tables = false;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k4[u];
            const int B = rdlane(fB, k);
            most = max(most, B < SHORT_STAGE ? B : 0);
            tables = tables || B >= SHORT_STAGE;
            ends[wv][u][lane] = pre[u];
        }
        for (int c = 64; c < most; c += 64) {
            int32_t v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k4[u];
                v[u] = (st.e + rdlane64s(fbase, k))[max(min(c + lane, rdlane(fB, k) - 1), 0)];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) ends[wv][u][c + lane] = v[u];
        }
        prefetch();
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < U; ++u) at[u] = 0;
        // a binary search in LDS, the four workers' side by side
        for (int step = most > 0 ? 1 << (31 - __builtin_clz(most)) : 0; step > 0; step >>= 1) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int B = rdlane(fB, k4[u]);
                const int to = at[u] + step;
                const int32_t v = ends[wv][u][min(to, SHORT_STAGE) - 1];
                at[u] = (to <= B && B < SHORT_STAGE && v < (int32_t)eq) ? to : at[u];
            }
        }
        if (tables) {
            // larger workers: through their tables; past a table (or without one) the
            // slot is searched from the table's last entry on
            int len[U];
            bool more = false;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k4[u];
                const int B = rdlane(fB, k);
                const uint16_t* tb = st.lbt + (int64_t)(sc.wbase + w0 + k) * LB_MAX;
                if (B >= SHORT_STAGE) at[u] = B < LB_SLOTS ? tb[min(lp, LB_MAX) - 1] / (int)sizeof(int4) : 0;
                len[u] = (B >= LB_SLOTS || (B >= SHORT_STAGE && lp > LB_MAX)) ? B - at[u] : 0;
                more = more || len[u] > 0;
            }
            while (ballot(more) != 0) {
                more = false;
                int32_t v[U];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    v[u] = (st.e + rdlane64s(fbase, k4[u]))[at[u] + (len[u] > 0 ? len[u] >> 1 : 0)];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int half = len[u] >> 1;
                    const bool right = len[u] > 0 && v[u] < (int32_t)eq;
                    at[u] = right ? at[u] + half + 1 : at[u];
                    len[u] = right ? len[u] - half - 1 : half;
                    more = more || len[u] > 0;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k4[u];
            const int64_t base = rdlane64s(fbase, k);
            t[u] = st.pms[base + at[u]];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u >= n4) break;
            const int k = k4[u];
            // every candidate is a KV demand with the query added, below 2^31:
            // 32-bit wrap-around arithmetic gives it exactly
            const int32_t a = (int32_t)((uint32_t)t[u].x + sq);
            const int32_t c = (int32_t)((uint32_t)t[u].z + (uint32_t)t[u].w * eq + sq + eq);
            int32_t peak = a > t[u].y ? a : t[u].y;
            peak = peak > c ? peak : c;
            const int32_t M = rdlane(fM, k);
            uint64_t bf, bn = 0;
            if (MODE >= 1) {
                bf = am & ballot(peak <= M) & ballot(qD <= rdlane64s(fdq, k)) & ballot(lin <= rdlane(flthr, k));
            } else {
                const View v = load_view(st, sc.wbase + w0 + k, hb);
                const Latency Lt = latency(sc, v, lin, lp, rdlane(fB, k) + 1);
                bf = am & ballot(peak <= M) & ballot(Lt.dec_ok && Lt.ttft_ok);
                bn = am & ballot(Lt.nt);
            }
            if (EX && MODE >= 1 && ((tied >> k) & 1)) {
                const int gw = sc.wbase + w0 + k;
                bool nt;
                if (MODE == 2) {
                    const uint64_t dd = (uint64_t)(qD - st.ntd_lo[gw]);
                    const uint32_t dl = (uint32_t)(lin - st.ntt_lo[gw]);
                    nt = (dd < 64 && ((st.ntd_mask[gw] >> dd) & 1)) || (dl < 64 && ((st.ntt_mask[gw] >> dl) & 1));
                } else {
                    const bool maybe = (qD >= st.ntd_lo[gw] && qD <= st.ntd_hi[gw]) ||
                                       (lin >= st.ntt_lo[gw] && lin <= st.ntt_hi[gw]) ||
                                       (lin >= st.ntp_lo[gw] && lin <= st.ntp_hi[gw]);
                    nt = maybe && latency(sc, load_view(st, gw, hb), lin, lp, rdlane(fB, k) + 1).nt;
                }
                bn = am & ballot(nt);
            }
            anyf |= bf;
            wf = lane == k ? bf : wf;
            if (EX) {
                wn = lane == k ? bn : wn;
                nfeas += __builtin_amdgcn_inverse_ballot_w64(bf) ? 1 : 0;
                ntcnt += __builtin_amdgcn_inverse_ballot_w64(bn) ? 1 : 0;
                keep_two<true>(peak - M, w0 + k, e1, w1, e2, w2);
            }
        }
    }
    const int64_t row = sc.bits_off + (int64_t)g * sc.W;
    if (lane < nk) {
        st.bits_feas[row + w0 + lane] = wf;
        if (EX) st.bits_nt[row + w0 + lane] = wn;
    }
    if (lane == 0) anyw[wv] = anyf;
    if (EX) two[wv][lane] = Two{w1 < 0 ? ~0ull : ex_key(e1, w1), w2 < 0 ? ~0ull : ex_key(e2, w2), nfeas, ntcnt};
    __syncthreads();
    if (wv == 0) publish_ranks(st, sc, s, nw, wbeg, ngr, g, rk, wkey, !EX);
    if (tid == 0) {
        const uint64_t f = anyw[0] | anyw[1] | anyw[2] | anyw[3];
        if (f != 0) {
            atomicOr((unsigned long long*)&st.any[sc.any_off + g], (unsigned long long)f);
            atomicMin(&st.tinfo[s].first_pc, q0 + __builtin_ctzll(f));
        }
    }
    if (EX && wv == NWV - 1 && act) {
        uint64_t a1 = ~0ull, a2 = ~0ull;
        int32_t nf = 0, nt = 0;
#pragma unroll
        for (int v = 0; v < NWV; ++v) {
            const Two x = two[v][lane];
            merge_two(a1, a2, x.k1, x.k2);
            nf += x.nfeas;
            nt += x.ntcnt;
        }
        ulonglong2* out = st.part + sc.part_off + 2 * ((int64_t)wb * sc.pstride + g * 64 + lane);
        out[0] = make_ulonglong2(a1, a2);
        out[1] = make_ulonglong2((uint32_t)nf, (uint32_t)nt);
    }
}

// ---------------------------------------------------------------------------------------------
// Per-query summary over all workers of the scenario, for the diagnostics: how
// many are feasible, how many have a near-tie margin, the two smallest KV
// excesses.  A lane holds one query of a 64-query group; the waves of the group
// share the workers.  Each non-zero bit word is added to the lanes' counts
// straight from its mask.
__global__ __launch_bounds__(SEL_THREADS) void k_select(State st)
{
    const int s = find_scen<&Scen::sel_blk0>(st, blockIdx.x);
    const Scen sc = st.scen[s];
    Ctl* cp = st.ctl + s;
    const int32_t start = cp->start, Q = cp->Q;
    const int local = blockIdx.x - sc.sel_blk0;
    if (cp->call != st.call) return;  // another call's control block
    if (cp->err || start >= Q) return;
    const int32_t end = tile_end(start, Q, cp->T, cp->H, cp->since_hb, cp->hb_next);
    // Algorithm 1's rank order at tile start, for the commit: a worker's place is
    // the number of workers that rank before it, counted by one wave per worker
    for (int j = local * (SEL_THREADS / 64) + wave_id(); j < sc.W; j += sc.sel_n * (SEL_THREADS / 64)) {
        const uint64_t kj = st.key[sc.wbase + j];
        int cnt = 0;
        for (int k0 = 0; k0 < sc.W; k0 += 64 * 8) {
            uint64_t kk[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) kk[u] = st.key[sc.wbase + min(k0 + u * 64 + lane_id(), sc.W - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u) cnt += count_before(kk[u], k0 + u * 64 + lane_id(), sc.W, kj, j);
        }
        if (lane_id() == 0) st.order[sc.wbase + cnt] = j;
    }
    // waves of the block: sel_g of them per 64-query group, each scanning its
    // share of the workers
    constexpr int NWV = SEL_THREADS / 64;
    const int G = sc.sel_g;
    const int wv = wave_id();
    const int group = local * (NWV / G) + wv / G;  // 64-query group of this wave
    const int slice = wv % G;                       // its share of the workers
    const int q0 = start + group * 64;
    const bool live = q0 < end;                     // wave-uniform
    const int lane = lane_id();
    // the group's words hold tile positions q0 - start + lane: the queries in
    // arrival order, or (sorted layout) the query qorig of each position
    const int slot = q0 - start + lane;
    const bool act = live && q0 + lane < end;
    const int qi = (act && st.qorig != nullptr) ? start + st.qorig[slot] : q0 + lane;

    int32_t nfeas = 0, ntcnt = 0;
    // the group's 64 queries share one bit word per worker; 64 workers' words
    // are read at once and only workers with a set bit are visited
    const int64_t row = sc.bits_off + (int64_t)group * sc.W;
    const int span = ((sc.W + G * 64 - 1) / (G * 64)) * 64;  // workers per wave, whole batches
    const int wlo = live ? min(sc.W, slice * span) : 0;
    const int whi = live ? min(sc.W, wlo + span) : 0;
    constexpr int UB = 8;  // 64-worker batches whose words are loaded together
    for (int g0 = wlo; g0 < whi; g0 += 64 * UB) {
        uint64_t fls[UB], nls[UB];
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            const int wl = g0 + u * 64 + lane;
            const bool in = wl < whi;
            fls[u] = in ? st.bits_feas[row + wl] : 0;
            nls[u] = in ? st.bits_nt[row + wl] : 0;
        }
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            for (uint64_t m = ballot(fls[u] != 0); m != 0; m &= m - 1)
                nfeas += __builtin_amdgcn_inverse_ballot_w64(rdlane64(fls[u], __ffsll((unsigned long long)m) - 1)) ? 1 : 0;
            for (uint64_t m = ballot(nls[u] != 0); m != 0; m &= m - 1)
                ntcnt += __builtin_amdgcn_inverse_ballot_w64(rdlane64(nls[u], __ffsll((unsigned long long)m) - 1)) ? 1 : 0;
        }
    }
    // each wave of the group merges its share of the worker blocks' two
    // smallest excess keys
    uint64_t a1 = ~0ull, a2 = ~0ull;
    auto merge = [&](ulonglong2 p) { merge_two(a1, a2, p.x, p.y); };
    if (act) {
        const ulonglong2* prow = st.part + sc.part_off + slot;
        if (sc.nblk > 64 * G) {  // many worker blocks (short tiles over many workers): more reads in flight
#pragma unroll 16
            for (int b = slice; b < sc.nblk; b += G) merge(prow[(int64_t)b * sc.pstride]);
        } else {
#pragma unroll 8
            for (int b = slice; b < sc.nblk; b += G) merge(prow[(int64_t)b * sc.pstride]);
        }
    }
    // merge the group's partial results into its first wave
    struct Part {
        uint64_t a1, a2;
        int32_t nfeas, ntcnt;
    };
    __shared__ Part parts[NWV][64];
    if (G > 1) {
        if (slice > 0) parts[wv][lane] = Part{a1, a2, nfeas, ntcnt};
        __syncthreads();
        if (slice > 0) return;
        for (int v = wv + 1; v < wv + G; ++v) {
            const Part pt = parts[v][lane];
            nfeas += pt.nfeas;
            ntcnt += pt.ntcnt;
            merge(ulonglong2{pt.a1, pt.a2});
        }
    }
    if (!act) return;
    QSum q;
    q.nfeas = nfeas;
    q.ntcnt = ntcnt;
    ex_unpack(a1, q.ex1, q.w1);
    ex_unpack(a2, q.ex2, q.w2);
    st.qsum[sc.qsum_off + (qi - start)] = q;
    if (nfeas == 0 && (st.qbad == nullptr || *st.qbad == 0)) {
        // no feasible worker at tile start: rejected whatever the tile commits
        // before it.  These tile-start diagnostics are exact for the queries
        // before the tile's first commit; the commit overwrites the ones after.
        if (st.out_worker) st.out_worker[sc.out_off + q_at(sc, qi)] = -1;
        Diag d;
        d.n_feasible = 0;
        d.near_tie = ntcnt > 0 ? 1 : 0;
        d.kv_peak_chosen = 0;
        d.kv_excess_min = q.ex1;
        d.ttft_chosen = 0.0;
        d.tdec_chosen = 0.0;
        st.out_diag[q_at(sc, qi)] = d;
    }
}

// ---------------------------------------------------------------------------------------------
// Query validation for one call: any length outside [1, 2^24] sets the error
// word of every scenario, which makes every later kernel of the call a no-op.
__global__ __launch_bounds__(256) void k_query_stats(const int32_t* lin, const int32_t* lpred, int32_t Q,
                                                     Ctl* ctl, int32_t S)
{
    __shared__ int64_t red[4];
    int64_t bad = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < Q; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t a = lin[i], p = lpred[i];
        bad += (a >= 1 && p >= 1 && a <= (1 << 24) && p <= (1 << 24)) ? 0 : 1;
    }
    bad = block_reduce<256>(bad, 0, OpAdd(), red);
    if (threadIdx.x == 0 && bad)
        for (int s = 0; s < S; ++s) atomicCAS(&ctl[s].err, 0, DEV_EINVAL);
}

// Start of an ald_place_stream call (one scenario, one block): the control
// block, the tile record, the group words and a cleared query-error word (the
// first round's pair evaluation checks the query lengths).  With gate >= 0 the
// call follows asynchronous call `gate` and starts only if that call finished
// without an error; otherwise the control block stays that call's, and every
// kernel of this call finds it foreign and does nothing.
__global__ __launch_bounds__(256) void k_begin(Ctl c, TileInfo ti, Ctl* ctl, TileInfo* tinfo, int32_t* qbad,
                                               int32_t gate, uint64_t* any, int64_t words)
{
    if (gate >= 0) {
        const Ctl o = *ctl;
        if (o.call != gate || o.err || o.start < o.Q) return;
        __syncthreads();  // every thread has read it
    }
    for (int64_t k = threadIdx.x; k < words; k += 256) any[k] = 0;
    if (threadIdx.x == 0) {
        *ctl = c;
        *tinfo = ti;
        *qbad = 0;
    }
}

__global__ __launch_bounds__(256) void k_clear(uint64_t* any, int64_t words)
{
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k < words) any[k] = 0;
}

// The outcome of an asynchronous call with no queries.
__global__ void k_status_ok(int32_t* status) { *status = ALD_OK; }

__global__ void k_summary(State st, int32_t W, int32_t* B, int64_t* sc, int64_t* sr, int64_t* peak)
{
    const int w = blockIdx.x * blockDim.x + threadIdx.x;
    if (w >= W) return;
    B[w] = st.B[w];
    sc[w] = st.SC[w];
    sr[w] = st.SR[w];
    peak[w] = st.peak[w];
}

__global__ void k_sweep_outputs(State st, int32_t* rejected, int32_t* first_reject)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= st.S) return;
    rejected[s] = st.ctl[s].n_rej;
    const int32_t f = st.ctl[s].first_rej;
    first_reject[s] = f == INT32_MAX ? -1 : f;
}

// The sweep's answer (Sec. 4.4, Sec. 6.4: the fewest GPUs that serve the
// stream with no violation): among scenarios with no rejection, the smallest
// n_workers * GPUs per worker, ties to the lowest scenario index.  One block;
// the (GPUs, index) pairs are ordered as one int64 key.
__global__ __launch_bounds__(256) void k_sweep_best(State st, int64_t* min_gpus)
{
    __shared__ int64_t red[4];
    int64_t best = INT64_MAX;
    for (int s = threadIdx.x; s < st.S; s += 256) {
        const Scen sc = st.scen[s];
        if (st.ctl[s].n_rej != 0 || st.ctl[s].err != 0) continue;
        // GPUs < 2^38 and s < 2^24 (checked on the host): the key fits in 62 bits
        const int64_t key = ((int64_t)sc.W * sc.gpw << 24) + s;
        best = key < best ? key : best;
    }
    best = block_reduce<256>(best, INT64_MAX, OpMin(), red);
    if (threadIdx.x == 0) {
        min_gpus[0] = best == INT64_MAX ? -1 : best >> 24;
        min_gpus[1] = best == INT64_MAX ? -1 : (best & ((1 << 24) - 1));
    }
}

// The outcome of an asynchronous sweep: the first scenario (by index) with a
// device error gives the code, as the synchronous sweep returns it; else
// ALD_EINCOMPLETE if a scenario has queries left, else ALD_OK.  One block.
__global__ __launch_bounds__(256) void k_sweep_status(State st, int32_t* status)
{
    __shared__ int64_t red[4];
    int64_t first_err = INT32_MAX, left = 0;
    for (int s = threadIdx.x; s < st.S; s += 256) {
        const Ctl c = st.ctl[s];
        if (c.err != 0 && s < first_err) first_err = s;
        left |= c.start < c.Q ? 1 : 0;
    }
    first_err = block_reduce<256>(first_err, (int64_t)INT32_MAX, OpMin(), red);
    left = block_reduce<256>(left, (int64_t)0, OpMax(), red);
    if (threadIdx.x == 0)
        *status = first_err != INT32_MAX ? ctl_status(st.ctl[first_err]) : (left ? ALD_EINCOMPLETE : ALD_OK);
}

// ---------------------------------------------------------------------------------------------
hipError_t launch_ingest(const State& st, int32_t W, const int64_t* res_off, const int32_t* lin,
                         const int32_t* lpred, const int32_t* gen, const double* tdec, hipStream_t stream)
{
    hipLaunchKernelGGL(k_ingest, dim3(W), dim3(BUILD_THREADS), 0, stream, st, res_off, lin, lpred, gen, tdec);
    return hipGetLastError();
}

hipError_t launch_build(const State& st, hipStream_t stream, int mode, int need, bool small)
{
    const int workers = mode == 1 ? st.S * MAX_DIRTY : st.NW;
    if (small)
        hipLaunchKernelGGL(k_build_small, dim3((workers + SMALL_WAVES - 1) / SMALL_WAVES), dim3(64 * SMALL_WAVES), 0,
                           stream, st, mode, need);
    else
        hipLaunchKernelGGL(k_build, dim3(workers), dim3(BUILD_THREADS), 0, stream, st, mode, need);
    return hipGetLastError();
}

hipError_t launch_eval(const State& st, int32_t blocks, int mode, hipStream_t stream)
{
    const bool ex = st.out_diag != nullptr;
    const dim3 g(blocks), b(EVAL_THREADS);
    if (st.brief) {
        if (mode >= 2) {
            if (ex) hipLaunchKernelGGL((k_eval_short<2, true>), g, b, 0, stream, st);
            else hipLaunchKernelGGL((k_eval_short<2, false>), g, b, 0, stream, st);
        } else if (mode == 1) {
            if (ex) hipLaunchKernelGGL((k_eval_short<1, true>), g, b, 0, stream, st);
            else hipLaunchKernelGGL((k_eval_short<1, false>), g, b, 0, stream, st);
        } else {
            if (ex) hipLaunchKernelGGL((k_eval_short<0, true>), g, b, 0, stream, st);
            else hipLaunchKernelGGL((k_eval_short<0, false>), g, b, 0, stream, st);
        }
        return hipGetLastError();
    }
    if (mode == 3) {
        if (ex) hipLaunchKernelGGL((k_eval<2, true, true>), g, b, 0, stream, st);
        else hipLaunchKernelGGL((k_eval<2, false, true>), g, b, 0, stream, st);
    } else if (mode == 2) {
        if (ex) hipLaunchKernelGGL((k_eval<2, true>), g, b, 0, stream, st);
        else hipLaunchKernelGGL((k_eval<2, false>), g, b, 0, stream, st);
    } else if (mode == 1) {
        if (ex) hipLaunchKernelGGL((k_eval<1, true>), g, b, 0, stream, st);
        else hipLaunchKernelGGL((k_eval<1, false>), g, b, 0, stream, st);
    } else {
        if (ex) hipLaunchKernelGGL((k_eval<0, true>), g, b, 0, stream, st);
        else hipLaunchKernelGGL((k_eval<0, false>), g, b, 0, stream, st);
    }
    return hipGetLastError();
}

int eval_blocks_per_cu(int mode, bool ex)
{
    const void* f = mode == 3 ? (ex ? (const void*)k_eval<2, true, true> : (const void*)k_eval<2, false, true>)
                  : mode == 2 ? (ex ? (const void*)k_eval<2, true> : (const void*)k_eval<2, false>)
                  : mode == 1 ? (ex ? (const void*)k_eval<1, true> : (const void*)k_eval<1, false>)
                              : (ex ? (const void*)k_eval<0, true> : (const void*)k_eval<0, false>);
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, EVAL_THREADS, 0) != hipSuccess) return 0;
    return n;
}

hipError_t launch_select(const State& st, int32_t blocks, hipStream_t stream)
{
    hipLaunchKernelGGL(k_select, dim3(blocks), dim3(SEL_THREADS), 0, stream, st);
    return hipGetLastError();
}

hipError_t launch_query_stats(const int32_t* lin, const int32_t* lpred, int32_t Q, Ctl* ctl, int32_t S,
                              hipStream_t stream)
{
    int blocks = (Q + 255) / 256;
    if (blocks > 256) blocks = 256;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_query_stats, dim3(blocks), dim3(256), 0, stream, lin, lpred, Q, ctl, S);
    return hipGetLastError();
}

hipError_t launch_begin(const Ctl& c, const TileInfo& ti, Ctl* ctl, TileInfo* tinfo, int32_t* qbad, int32_t gate,
                        uint64_t* any, int64_t words, hipStream_t stream)
{
    hipLaunchKernelGGL(k_begin, dim3(1), dim3(256), 0, stream, c, ti, ctl, tinfo, qbad, gate, any, words);
    return hipGetLastError();
}

hipError_t launch_clear(uint64_t* any, int64_t words, hipStream_t stream)
{
    if (words == 0) return hipSuccess;
    hipLaunchKernelGGL(k_clear, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, stream, any, words);
    return hipGetLastError();
}

hipError_t launch_status_ok(int32_t* status, hipStream_t stream)
{
    hipLaunchKernelGGL(k_status_ok, dim3(1), dim3(1), 0, stream, status);
    return hipGetLastError();
}

hipError_t launch_summary(const State& st, int32_t W, int32_t* B, int64_t* sc, int64_t* sr, int64_t* peak,
                          hipStream_t stream)
{
    hipLaunchKernelGGL(k_summary, dim3((W + 255) / 256), dim3(256), 0, stream, st, W, B, sc, sr, peak);
    return hipGetLastError();
}

hipError_t launch_sweep_outputs(const State& st, int32_t* rejected, int32_t* first_reject, int64_t* min_gpus,
                                hipStream_t stream)
{
    hipLaunchKernelGGL(k_sweep_outputs, dim3((st.S + 255) / 256), dim3(256), 0, stream, st, rejected,
                       first_reject);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || min_gpus == nullptr) return e;
    hipLaunchKernelGGL(k_sweep_best, dim3(1), dim3(256), 0, stream, st, min_gpus);
    return hipGetLastError();
}

hipError_t launch_sweep_status(const State& st, int32_t* status, hipStream_t stream)
{
    hipLaunchKernelGGL(k_sweep_status, dim3(1), dim3(256), 0, stream, st, status);
    return hipGetLastError();
}

}  // namespace ald
