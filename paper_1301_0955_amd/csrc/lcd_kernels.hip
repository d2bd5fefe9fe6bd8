// Kernels of the multi-scale local community sweep for gfx950 (CDNA4, wave64).
//
// One wavefront grows one community through every scale (paper Sec. 2,
// Algorithm 1, chained over scales as in Algorithm 2).  Per community the
// wave keeps a table of every node it has touched:
//   open-addressing hash  node id -> dense index   (int32 slots, 2^hbits >= 2 cap)
//   dense arrays          node id, d_in | flags, weighted degree k, rank R
// held in LDS (tier 0) or, for communities that outgrow the LDS table, in a
// per-wave slab of global memory (tiers 1 and 2, same code).
//
// The sequential priority queue of Algorithm 1 is emulated exactly:
//   * every live (queued) entry is tested against the current (K, V); the
//     highest-ranked improving entry e* is the one the queue would add next,
//     and every live entry ranked above e* would have been popped and
//     rejected against the same state first.  Those pops are applied lazily:
//     the next pass drops a live entry ranked above the previous e* unless
//     the addition of e* touched it (flag FRESH), which is exactly the
//     queue update that Algorithm 1 applies to the neighbours of an added
//     node.
//   * the number of pops G is counted where entries enter the queue (every
//     entry that enters is popped exactly once before the queue empties).
//   * a removal pass visits members in ascending id: each step finds the
//     smallest removable id above the cursor with a wave min-reduction.
// Decisions use only exact integer sums and the integer log L below, in
// the same IEEE operation order as the specification, so the result is
// bit-identical to a sequential evaluation.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "lcd_internal.h"

namespace lcd {

namespace {

constexpr double kMargin = 0x1p-40;   // improvement threshold on the log-fitness gain
constexpr double kCert = 1e-10;       // certified comparisons' margin (see improves_add)
constexpr uint32_t kDMask = (1u << 27) - 1;   // d (weighted degrees stay below 2^27)
constexpr uint32_t kMember = 1u << 31;
constexpr uint32_t kLive = 1u << 30;
constexpr uint32_t kFresh = 1u << 29;
// delta output: member at the set's last emitted record
constexpr uint32_t kWas = 1u << 28;
// bucketed queue: re-ranked by the latest addition, not yet seen by a
// fresh-list scan
constexpr uint32_t kTouch = 1u << 27;

// ---------------------------------------------------------------------------
// L(x): natural log of an integer 1 <= x < 2^53.  x = m 2^e with m in
// (sqrt(2)/2, sqrt(2)]; ln m = 2 atanh(s), s = (m-1)/(m+1), by the series
// 2 s (1 + z/3 + ... + z^11/23) with z = s^2; ln 2 as a Cody-Waite pair so
// that e * ln2_hi is exact.  Plain IEEE operations, no contraction.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double ilog(uint64_t x) {
    int e = 63 - __builtin_clzll(x);
    double m = (double)x * __longlong_as_double((long long)(1023 - e) << 52);
    if (m > 0x1.6a09e667f3bcdp+0) {
        m = m * 0.5;
        e = e + 1;
    }
    double s = (m - 1.0) / (m + 1.0);
    double z = s * s;
    double p = 1.0 / 23.0;
    p = p * z + 1.0 / 21.0;
    p = p * z + 1.0 / 19.0;
    p = p * z + 1.0 / 17.0;
    p = p * z + 1.0 / 15.0;
    p = p * z + 1.0 / 13.0;
    p = p * z + 1.0 / 11.0;
    p = p * z + 1.0 / 9.0;
    p = p * z + 1.0 / 7.0;
    p = p * z + 1.0 / 5.0;
    p = p * z + 1.0 / 3.0;
    p = p * z + 1.0;
    double h = s * p;
    double lnm = h + h;
    double de = (double)e;
    return de * 6.93147180369123816490e-01 + (de * 1.90821492927058770002e-10 + lnm);
}

__device__ __forceinline__ uint64_t lanes_below(int lane) {
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// Ordering point between table phases of one wave.  LDS operations of a
// wave execute in order, so only the compiler must be fenced; global
// tables additionally wait for outstanding memory operations.
template <bool GLOBAL>
__device__ __forceinline__ void wsync() {
    if constexpr (GLOBAL)
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    else
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint32_t hash_of(int32_t u, int hbits) {
    return ((uint32_t)u * 2654435761u) >> (32 - hbits);
}

// true when (r, u) pops before (pr, pu): higher rank, then smaller id
__device__ __forceinline__ bool before(double r, int32_t u, double pr, int32_t pu) {
    return r > pr || (r == pr && u < pu);
}

// A wave's community table: one array per field (a scan reads one field of
// consecutive entries).
struct Tab {
    double *rk;
    int32_t *node;
    uint32_t *dv;
    int32_t *kv;
    __device__ __forceinline__ double &RK(int32_t i) const { return rk[i]; }
    __device__ __forceinline__ int32_t &NODE(int32_t i) const { return node[i]; }
    __device__ __forceinline__ uint32_t &DV(int32_t i) const { return dv[i]; }
    __device__ __forceinline__ int32_t &KV(int32_t i) const { return kv[i]; }
    int32_t *scr;
    int32_t *hs;      // hash slots: entry index
    uint32_t hmask;
    int hbits;
    int cap;
};

// Rank f64[cap], node i32[cap], d|flags u32[cap], degree i32[cap], scratch
// i32[cap], hash slots i32[2^hbits], in LDS or global memory.
__device__ __forceinline__ Tab carve(char *base, int cap, int hbits) {
    Tab t;
    t.rk = (double *)base;
    t.node = (int32_t *)(t.rk + cap);
    t.dv = (uint32_t *)(t.node + cap);
    t.kv = t.node + 2 * (size_t)cap;
    t.scr = t.node + 3 * (size_t)cap;
    t.hs = t.node + 4 * (size_t)cap;
    t.hbits = hbits;
    t.hmask = (1u << hbits) - 1;
    t.cap = cap;
    return t;
}

template <bool GLOBAL>
__device__ __forceinline__ int32_t hs_load(const int32_t *p) {
    if constexpr (GLOBAL)
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        return *p;
}

template <bool GLOBAL>
__device__ __forceinline__ void hs_store(int32_t *p, int32_t v) {
    if constexpr (GLOBAL)
        __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        *p = v;
}

// Per-wave state.  Every field except the lane partial counters holds the
// same value in all lanes.
struct St {
    int32_t count;     // dense entries in use
    int32_t nmem;      // members
    int64_t K, V;      // k_in and volume of the community
    double rK2, rV;    // 2 / K and 1 / V when positive, for the certified comparisons
    double alpha;
    double pr;         // rank and id of the entry added last in this call
    int32_t pu;
    uint32_t Gl, Rl;   // lane partial counts of pops and rank computations
    uint64_t Gu;       // wave-uniform part of G (removal-pass visits)
    uint64_t M;        // moves in this (set, scale)
    bool ovf;          // the table ran out of entries
    uint32_t err;
    int64_t move_limit; // guard against a runaway loop in one (set, scale)
    uint64_t t0;        // wall clock when the set started
    uint64_t budget;    // wall-clock ticks the set may take
    uint64_t rows;      // CSR rows gathered (moves and initial members)
    uint64_t row_len;   // ... and their total length
    uint64_t inserted;  // table entries created (one degree read each)
    uint64_t written;   // member ids written to the pool
    uint64_t scanned;   // table entries visited by the growth scans
    // algorithmic work, committed when a scale's record is written (work of
    // a scale that overflows is redone in the next tier and not counted)
    uint64_t mrows, mrow_len;       // rows gathered by moves, running totals
    uint64_t c_mrows, c_mrow_len;   // ... at the last record written
    uint64_t ins_mark, c_ins;       // entries created: not counted before ins_mark;
                                    // committed count at the last record written
    uint64_t srows, srow_len;       // seed-set rows of a set in its first tier
    double qtop, qscale;            // workgroup tables: rank range of the queue's buckets
    double qhi, qlo, qalpha;        // the ranks' range at the last build, and its scale
    int32_t flen;                   // ... entries on the fresh list
    int32_t nadd, nrem;             // ... additions and removals at the scale being grown
    bool emitted;                   // a record was written in this tier
};

// Watchdog: a seed set that runs past its budget stops with ERR_TIMEOUT, so
// a logic error ends the sweep with an error instead of running on.
__device__ __forceinline__ bool over_budget(St &st) {
    if (wall_clock64() - st.t0 > st.budget) {
        st.err |= ERR_TIMEOUT;
        return true;
    }
    return false;
}

struct Ctx {
    const int32_t *row_ptr;
    const int32_t *col;
    const uint8_t *w;
    const int32_t *kdeg;
    const double *logtab;
    int32_t logtab_last;   // largest valid index of logtab
    int32_t n;             // nodes
    int64_t nnz;           // directed entries
    const int2 *info;      // per node: row start, weighted degree
    const int4 *adj;       // per directed entry: neighbour, its degree, its row start, weight; or null
    const double *adjl;    // ... and the log of its degree
};

__device__ __forceinline__ Ctx make_ctx(const GraphDev &g) {
    Ctx c;
    c.row_ptr = g.row_ptr;
    c.col = g.col;
    c.w = g.w;
    c.kdeg = g.kdeg;
    c.logtab = g.logtab;
    c.logtab_last = g.logtab_n - 1;
    c.n = g.n;
    c.nnz = g.nnz;
    c.info = g.info;
    c.adj = g.adj;
    c.adjl = g.adjl;
    return c;
}

// queue rank R(d, k) = L(2d) - alpha L(k); 2d <= 2k <= 2 max degree, so both
// logs come from the table (the clamp only keeps a broken table in bounds)
__device__ __forceinline__ double rank_of(const Ctx &c, int32_t d, int32_t k, double alpha) {
    const int32_t i2 = min(2 * d, c.logtab_last);
    const int32_t ik = min(k, c.logtab_last);
    return c.logtab[i2] - alpha * c.logtab[ik];
}

template <bool GLOBAL>
__device__ __forceinline__ int32_t tab_find(const Tab &t, int32_t u, uint32_t &err) {
    uint32_t p = hash_of(u, t.hbits);
    for (uint32_t it = 0; it <= t.hmask; ++it) {
        int32_t i = hs_load<GLOBAL>(&t.hs[p]);
        if (i < 0)
            return -1;
        if (t.NODE(i) == u)
            return i;
        p = (p + 1) & t.hmask;
    }
    err |= ERR_PROBE;
    return -1;
}

// Put entry idx of node u into its hash slot (linear probing).
template <bool GLOBAL>
__device__ __forceinline__ void tab_slot_insert(const Tab &t, int32_t u, int32_t idx, uint32_t &err) {
    uint32_t p = hash_of(u, t.hbits);
    uint32_t it = 0;
    for (; it <= t.hmask; ++it) {
        if (atomicCAS(&t.hs[p], -1, idx) == -1)
            break;
        p = (p + 1) & t.hmask;
    }
    if (it > t.hmask)
        err |= ERR_PROBE;
}

// Empty the hash slot of entry i (global tables, before the slab's next
// community).
template <bool GLOBAL>
__device__ __forceinline__ void tab_slot_clear(const Tab &t, int32_t i) {
    uint32_t p = hash_of(t.NODE(i), t.hbits);
    for (uint32_t it = 0; it <= t.hmask; ++it) {
        if (hs_load<GLOBAL>(&t.hs[p]) == i) {
            hs_store<GLOBAL>(&t.hs[p], -1);
            return;
        }
        p = (p + 1) & t.hmask;
    }
}

// A directed entry: neighbour, its degree, its row start, the edge's weight,
// the log of the degree.
struct Edge {
    int4 e;
    double lk;
};

__device__ __forceinline__ Edge edge_at(const Ctx &c, int32_t j) {
    Edge x;
    if (c.adj) {
        x.e = c.adj[j];
        x.lk = c.adjl[j];
        return x;
    }
    const int32_t u = c.col[j];
    const int2 in = c.info[u];
    x.e = make_int4(u, in.y, in.x, c.w ? (int32_t)c.w[j] : 1);
    x.lk = c.logtab[min(in.y, c.logtab_last)];
    return x;
}

__device__ __forceinline__ Edge no_edge() {
    Edge x;
    x.e = make_int4(0, 0, 0, 0);
    x.lk = 0.0;
    return x;
}

// Dense index of u (of degree k) for every active lane, inserting absent ids.  All active
// ids of one call are distinct.  Returns -1 for inactive lanes, and for all
// lanes when the table would overflow (st.ovf is then set).
template <bool GLOBAL>
__device__ int32_t tab_ensure(const Tab &t, St &st, bool act, int32_t u, int32_t k, int lane) {
    int32_t idx = act ? tab_find<GLOBAL>(t, u, st.err) : -1;
    bool need = act && idx < 0;
    uint64_t m = __ballot(need);
    if (m == 0)
        return idx;
    int nn = __popcll(m);
    if (st.count + nn > t.cap) {
        st.ovf = true;
        return -1;
    }
    st.inserted += (uint64_t)nn;
    if (need) {
        idx = st.count + __popcll(m & lanes_below(lane));
        t.NODE(idx) = u;
        t.KV(idx) = k;
        t.DV(idx) = 0u;
        tab_slot_insert<GLOBAL>(t, u, idx, st.err);
    }
    st.count += nn;
    wsync<GLOBAL>();
    return idx;
}

enum { ROW_INIT = 0, ROW_ADD = 1, ROW_REMOVE = 2 };

// Apply the edges of node n to the table: d_in += w for INIT and ADD,
// d_in -= w for REMOVE.  For ADD, every non-member neighbour is (re)queued
// with its new rank (the queue update of Algorithm 1).
template <bool GLOBAL, int MODE>
__device__ void row_update(const Tab &t, St &st, const Ctx &c, int32_t n, int lane) {
    const int32_t beg = c.row_ptr[n];
    const int32_t len = c.row_ptr[n + 1] - beg;
    st.rows += 1;
    st.row_len += (uint64_t)len;
    if constexpr (MODE != ROW_INIT) {
        st.mrows += 1;
        st.mrow_len += (uint64_t)len;
    }
    for (int32_t base = 0; base < len; base += 64) {
        const bool act = base + lane < len;
        const Edge x = act ? edge_at(c, beg + base + lane) : no_edge();
        const int32_t u = x.e.x, wt = x.e.w;
        int32_t idx;
        if constexpr (MODE == ROW_REMOVE) {
            idx = act ? tab_find<GLOBAL>(t, u, st.err) : -1;
            if (act && idx < 0)
                st.err |= ERR_MISSING;
        } else {
            idx = tab_ensure<GLOBAL>(t, st, act, u, x.e.y, lane);
            if (st.ovf)
                return;
        }
        if (act && idx >= 0) {
            const uint32_t v = t.DV(idx);
            int32_t d = (int32_t)(v & kDMask);
            if constexpr (MODE == ROW_REMOVE) {
                d -= wt;
                t.DV(idx) = (v & ~kDMask) | (uint32_t)d;
            } else if constexpr (MODE == ROW_INIT) {
                d += wt;
                t.DV(idx) = (v & ~kDMask) | (uint32_t)d;
            } else {
                d += wt;
                if (v & kMember) {
                    t.DV(idx) = (v & ~kDMask) | (uint32_t)d;
                } else {
                    // still queued unless popped and rejected above the node just added
                    const bool queued = (v & kLive) && !before(t.RK(idx), u, st.pr, st.pu);
                    if (!queued)
                        st.Gl += 1;
                    t.RK(idx) = c.logtab[min(2 * d, c.logtab_last)] - st.alpha * x.lk;
                    st.Rl += 1;
                    t.DV(idx) = (v & kWas) | (uint32_t)d | kLive | kFresh;
                }
            }
        }
    }
    wsync<GLOBAL>();
}

// Full decision "f(Kp, Vp) > f(K, V)" in the log domain (K, V > 0 here).
// Four logs of eleven dependent steps and a division each: reached only by
// the few entries that the certified comparisons below leave open.
__device__ __forceinline__ bool decide(int64_t K, int64_t V, int64_t Kp, int64_t Vp, double alpha) {
    // K and V do not change inside a scan: kept opaque here, or the compiler
    // moves their logs before it and every scan pays for both
    asm volatile("" : "+v"(K), "+v"(V));
    const double a = ilog((uint64_t)Kp) - ilog((uint64_t)K);
    const double b = ilog((uint64_t)Vp) - ilog((uint64_t)V);
    const double cc = alpha * b;
    const double t = a - cc;
    return t > kMargin;
}

// Would adding a non-member with (d, k) raise f?  The exact gain is
//   T = ln(1 + x) - alpha ln(1 + y),  x = 2d / K,  y = k / V,
// and for z > 0   2z / (2 + z) < ln(1 + z) < z (6 + z) / (6 + 4z).
// A bound on T that clears zero by 1e-10 settles the decision: the computed
// gain differs from T by less than 1e-11 (alpha <= 1000), the threshold is
// 2^-40, and the bounds, multiplied out by their denominators, carry a
// relative rounding error below 1e-14 (x, y from one reciprocal per state;
// x <= 1024 keeps every term within 1e4 of the denominators near a tie).
// The bounds are x^2 / 12 apart, so for communities of more than a few
// members nearly every entry is settled by about twenty multiplications
// instead of two logs with a division each.  Bound by instruction issue on
// LDS tables and by latency on global ones; with the VALU reductions below
// the 1,000-node sweep's workgroup tier went from 6.0 to 4.4 ms, tier 2 of a
// 1,000,000-node share from 209 to 188 ms.
//
// settle_add: 1 raises f, 0 does not, -1 left open (K > 0).
__device__ __forceinline__ int settle_add(const St &st, int32_t d, int32_t k) {
    const double x = (double)d * st.rK2;
    const double y = (double)k * st.rV;
    const double ay = st.alpha * y;
    const double p = 2.0 + x, q = __builtin_fma(4.0, y, 6.0);
    const double n1 = __builtin_fma(2.0 * x, q, -(ay * (6.0 + y)) * p);
    const double r = 2.0 + y, u = __builtin_fma(4.0, x, 6.0);
    const double n2 = __builtin_fma(x * (6.0 + x), r, -2.0 * ay * u);
    const bool yes = n1 > kCert * (p * q), no = n2 < -kCert * (r * u);
    return x <= 1024.0 ? (yes ? 1 : no ? 0 : -1) : -1;
}

__device__ __forceinline__ bool improves_add(const St &st, int32_t d, int32_t k) {
    if (st.K == 0)
        return true;
    const int t = settle_add(st, d, k);
    return t >= 0 ? t != 0 : decide(st.K, st.V, st.K + 2 * (int64_t)d, st.V + k, st.alpha);
}

// Would removing a member with internal weight d and degree k raise f?  The
// same with T = alpha lny - lnx, lnx = -ln(1 - x), and for 0 < z < 1
//   2z / (2 - z) <= -ln(1 - z) <= z (6 - 5z) / ((1 - z) (6 - 2z)).
// Only x, y <= 1/2 are settled this way (1 - z would lose digits near 1).
__device__ __forceinline__ bool improves_remove(const St &st, int32_t d, int32_t k) {
    const int64_t Kp = st.K - 2 * (int64_t)d;
    if (Kp <= 0)
        return false;
    const double x = (double)d * st.rK2;
    const double y = (double)k * st.rV;
    const double ay = st.alpha * y;
    const double p = 2.0 - y, q = (1.0 - x) * __builtin_fma(-2.0, x, 6.0);
    const double n1 = __builtin_fma(2.0 * ay, q, -(x * __builtin_fma(-5.0, x, 6.0)) * p);
    const double r = 2.0 - x, u = (1.0 - y) * __builtin_fma(-2.0, y, 6.0);
    const double n2 = __builtin_fma(ay * __builtin_fma(-5.0, y, 6.0), r, -2.0 * x * u);
    const bool small = x <= 0.5 && y <= 0.5;
    if (small && n1 > kCert * (p * q))
        return true;
    if (small && n2 < -kCert * (r * u))
        return false;
    return decide(st.K, st.V, Kp, st.V - k, st.alpha);
}

// The reciprocals of the state, after K or V changed.
__device__ __forceinline__ void set_rates(St &st) {
    st.rK2 = st.K > 0 ? 2.0 / (double)st.K : 0.0;
    st.rV = st.V > 0 ? 1.0 / (double)st.V : 0.0;
}

// Lane exchanges inside the VALU: lane i reads lane i - n of its row of 16
// (row_shr) or the last lane of the rows before (row_bcast); a lane with no
// source keeps its own value, so min and max need no neutral element.  Six
// such steps leave the wave's result in lane 63.  A shuffle through LDS costs
// an LDS round trip per step instead, and the argmax of (rank, id, index)
// took four of them in each of six steps.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_from(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xf, 0xf, false);
}

template <int CTRL>
__device__ __forceinline__ double dpp_from(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = dpp_from<CTRL>((uint32_t)b);
    const uint32_t hi = dpp_from<CTRL>((uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

constexpr int kShr1 = 0x111, kShr2 = 0x112, kShr4 = 0x114, kShr8 = 0x118, kBcast15 = 0x142, kBcast31 = 0x143;

__device__ __forceinline__ double read_lane(double v, int l) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ double wave_max(double v) {
    v = fmax(v, dpp_from<kShr1>(v));
    v = fmax(v, dpp_from<kShr2>(v));
    v = fmax(v, dpp_from<kShr4>(v));
    v = fmax(v, dpp_from<kShr8>(v));
    v = fmax(v, dpp_from<kBcast15>(v));
    v = fmax(v, dpp_from<kBcast31>(v));
    return read_lane(v, 63);
}

__device__ __forceinline__ int32_t wave_min(int32_t x) {
    uint32_t v = (uint32_t)x ^ 0x80000000u;   // unsigned order
    v = min(v, dpp_from<kShr1>(v));
    v = min(v, dpp_from<kShr2>(v));
    v = min(v, dpp_from<kShr4>(v));
    v = min(v, dpp_from<kShr8>(v));
    v = min(v, dpp_from<kBcast15>(v));
    v = min(v, dpp_from<kBcast31>(v));
    return (int32_t)((uint32_t)__builtin_amdgcn_readlane((int)v, 63) ^ 0x80000000u);
}

// The lane that holds the entry popping first among (r, u) (i < 0: no entry;
// -1 when no lane has one): the highest rank, and among equal ranks the
// smallest id.  Called by all 64 lanes; the result is wave-uniform.
__device__ __forceinline__ int wave_first(double r, int32_t u, int32_t i) {
    const double m = wave_max(i >= 0 ? r : -__builtin_huge_val());
    uint64_t at = __ballot(i >= 0 && r == m);
    if (at == 0)
        return -1;
    if (at & (at - 1)) {
        const int32_t lo = wave_min(i >= 0 && r == m ? u : INT32_MAX);
        at = __ballot(i >= 0 && r == m && u == lo);
    }
    return (int)__builtin_ctzll(at);
}

// (r, u, i) of the wave's first entry in every lane; i = -1 if there is none.
__device__ __forceinline__ void wave_argmax(double &r, int32_t &u, int32_t &i) {
    const int l = wave_first(r, u, i);
    if (l < 0) {
        r = -__builtin_huge_val();
        u = INT32_MAX;
        i = -1;
        return;
    }
    r = read_lane(r, l);
    u = __builtin_amdgcn_readlane(u, l);
    i = __builtin_amdgcn_readlane(i, l);
}

// The wave's smallest u with its i (u = INT32_MAX, i = -1: none).
__device__ __forceinline__ void wave_argmin(int32_t &u, int32_t &i) {
    const int32_t lo = wave_min(u);
    const uint64_t at = __ballot(u == lo);
    i = __builtin_amdgcn_readlane(i, (int)__builtin_ctzll(at));
    u = lo;
}

__device__ __forceinline__ uint32_t wave_or(uint32_t v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        v |= __shfl_xor(v, off);
    return v;
}

__device__ __forceinline__ uint64_t wave_sum(uint64_t v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        v += __shfl_xor(v, off);
    return v;
}

// Whether any entry of the queue that a call starts with improves.  Most
// calls add nothing (at least one per scale), and for those the ranks need
// not be computed, only counted.
template <bool GLOBAL>
__device__ __forceinline__ bool wave_any_improves(const Tab &t, St &st, int lane) {
    bool any = false;
    const bool zero = st.K == 0;
    st.scanned += (uint64_t)st.count;
    for (int32_t base = 0; base < st.count; base += 128) {
        uint32_t vv[2];
        int32_t kk[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const int32_t i = min(base + 64 * x + lane, st.count - 1);
            vv[x] = t.DV(i);
            kk[x] = t.KV(i);
        }
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const int32_t d = (int32_t)(vv[x] & kDMask);
            const bool in = base + 64 * x + lane < st.count && !(vv[x] & kMember) && d != 0;
            st.Rl += in ? 1 : 0;
            st.Gl += in ? 1 : 0;
            int s = zero ? 1 : settle_add(st, d, kk[x]);
            if (in && !any && s < 0)
                s = decide(st.K, st.V, st.K + 2 * (int64_t)d, st.V + kk[x], st.alpha) ? 1 : 0;
            any = any || (in && s > 0);
        }
    }
    return __ballot(any) != 0;
}

// One call of the growth function (Algorithm 1) at st.alpha.
// Returns the number of moves; stops early on table overflow.
template <bool GLOBAL>
__device__ int64_t grow(const Tab &t, St &st, const Ctx &c, uint32_t k_prune, int lane) {
    int64_t moves = 0;
    bool creation = true;
    if (!wave_any_improves<GLOBAL>(t, st, lane))
        return 0;
    for (;;) {
        double br = -__builtin_huge_val();
        int32_t bu = INT32_MAX;
        int32_t bi = -1;
        st.scanned += (uint64_t)st.count;
        for (int32_t i = lane; i < st.count; i += 64) {
            uint32_t v = t.DV(i);
            double r;
            if (creation) {
                // the queue is built from every non-member with a link into c
                if ((v & kMember) || (v & kDMask) == 0) {
                    if (v & (kLive | kFresh))
                        t.DV(i) = v & ~(kLive | kFresh);
                    continue;
                }
                const int32_t d = (int32_t)(v & kDMask);
                r = rank_of(c, d, t.KV(i), st.alpha);
                t.RK(i) = r;
                v = (v | kLive) & ~kFresh;
                t.DV(i) = v;
            } else {
                if (!(v & kLive))
                    continue;
                r = t.RK(i);
                if (v & kFresh) {
                    v &= ~kFresh;
                    t.DV(i) = v;
                } else if (before(r, t.NODE(i), st.pr, st.pu)) {
                    t.DV(i) = v & ~kLive;      // popped and rejected last step
                    continue;
                }
            }
            const int32_t u = t.NODE(i);
            if (before(r, u, br, bu) && improves_add(st, (int32_t)(v & kDMask), t.KV(i))) {
                br = r;
                bu = u;
                bi = i;
            }
        }
        creation = false;
        wave_argmax(br, bu, bi);
        wsync<GLOBAL>();
        if (bi < 0)
            break;
        // add the best improving node
        const uint32_t v = t.DV(bi);
        const int32_t d = (int32_t)(v & kDMask);
        const int32_t k = t.KV(bi);
        wsync<GLOBAL>();
        if (lane == 0)
            t.DV(bi) = (v | kMember) & ~(kLive | kFresh);
        st.K += 2 * (int64_t)d;
        st.V += k;
        st.nmem += 1;
        st.M += 1;
        moves += 1;
        st.pr = br;
        st.pu = bu;
        set_rates(st);
        wsync<GLOBAL>();
        row_update<GLOBAL, ROW_ADD>(t, st, c, bu, lane);
        if (st.ovf)
            return moves;
        if ((int64_t)st.M > st.move_limit) {
            st.err |= ERR_LIMIT;
            return moves;
        }
        if (over_budget(st))
            return moves;
    }
    if (moves == 0)
        return 0;
    // removal passes over the members in ascending id
    for (uint32_t pass = 0; k_prune == 0 || pass < k_prune; ++pass) {
        st.Gu += (uint64_t)st.nmem;
        int32_t cursor = -1;
        bool removed = false;
        for (;;) {
            int32_t cu = INT32_MAX;
            int32_t ci = -1;
            st.scanned += (uint64_t)st.count;
            for (int32_t i = lane; i < st.count; i += 64) {
                const uint32_t v = t.DV(i);
                if (!(v & kMember))
                    continue;
                const int32_t u = t.NODE(i);
                if (u <= cursor || u >= cu)
                    continue;
                if (improves_remove(st, (int32_t)(v & kDMask), t.KV(i))) {
                    cu = u;
                    ci = i;
                }
            }
            wave_argmin(cu, ci);
            wsync<GLOBAL>();
            if (ci < 0)
                break;
            const uint32_t v = t.DV(ci);
            const int32_t d = (int32_t)(v & kDMask);
            const int32_t k = t.KV(ci);
            wsync<GLOBAL>();
            if (lane == 0)
                t.DV(ci) = v & ~kMember;
            st.K -= 2 * (int64_t)d;
            st.V -= k;
            st.nmem -= 1;
            st.M += 1;
            moves += 1;
            set_rates(st);
            wsync<GLOBAL>();
            row_update<GLOBAL, ROW_REMOVE>(t, st, c, cu, lane);
            removed = true;
            cursor = cu;
            if ((int64_t)st.M > st.move_limit) {
                st.err |= ERR_LIMIT;
                return moves;
            }
            if (over_budget(st))
                return moves;
        }
        if (!removed)
            break;
    }
    return moves;
}

// Ascending sort of a[0..m) by one wave: bitonic network in its all-ascending
// form (each merge starts with a "flip" stage), with virtual +inf padding to
// the next power of two so comparators that touch the padding are no-ops.
template <bool GLOBAL>
__device__ void wave_sort(int32_t *a, int32_t m, int lane) {
    int32_t P = 1;
    while (P < m)
        P <<= 1;
    const int32_t half_n = P >> 1;
    for (int32_t k = 2; k <= P; k <<= 1) {
        const int32_t hk = k >> 1;
        for (int32_t t = lane; t < half_n; t += 64) {
            const int32_t blk = t / hk;
            const int32_t off = t - blk * hk;
            const int32_t i = blk * k + off;
            const int32_t l = blk * k + k - 1 - off;
            if (l < m) {
                const int32_t x = a[i], y = a[l];
                if (x > y) {
                    a[i] = y;
                    a[l] = x;
                }
            }
        }
        wsync<GLOBAL>();
        for (int32_t j = k >> 2; j >= 1; j >>= 1) {
            for (int32_t t = lane; t < half_n; t += 64) {
                const int32_t i = (t / j) * 2 * j + (t % j);
                const int32_t l = i + j;
                if (l < m) {
                    const int32_t x = a[i], y = a[l];
                    if (x > y) {
                        a[i] = y;
                        a[l] = x;
                    }
                }
            }
            wsync<GLOBAL>();
        }
    }
}

// PERSET: each set carries its own scale (query batches, one record per
// set); otherwise every set runs through scales[s_begin, s_end).
// Delta output: the first scale of the set's last full list at or before
// scale s_last (-1 if there is none), and the pool span of record r.
__device__ __forceinline__ int32_t delta_key_scale(const Records &rec, int32_t S, int32_t set, int32_t s_last) {
    int32_t sk = s_last;
    while (sk >= 0 && rec.drem[(int64_t)set * S + sk] >= 0)
        --sk;
    return sk;
}

__device__ __forceinline__ int32_t record_len(const Records &rec, int64_t r) {
    return rec.drem[r] < 0 ? rec.cnt[r] : rec.dadd[r] + rec.drem[r];
}

// Scales that a set did not reach (its start lies outside an overflowed
// pool, or an error ended it) get records that no later launch of the same
// sweep takes for lists: a per-scale loop reads every record of the scale
// before, and what the memory held earlier could name any ids.  Every calling
// thread stores the same values.
__device__ __forceinline__ void void_records(const SweepArgs &A, int32_t set, int32_t s_from) {
    for (int32_t s = s_from; s < A.s_end; ++s) {
        const int64_t r = (int64_t)set * A.S + s;
        A.rec.off[r] = -1;
        A.rec.cnt[r] = 0;
        if (A.rec.drem) {
            A.rec.dadd[r] = 0;
            A.rec.drem[r] = -1;
        }
    }
}

// Delta output, one wave: rebuild in the table the members recorded for
// scale s_last by toggling kMember | kWas for every id of the last full
// list and of each delta after it (an id joins and leaves alternately, so
// the members are the ids seen an odd number of times).  False when a
// record lies outside the pool (it overflowed: the host runs the sweep
// again); no full list before s_last is an error (ERR_MISSING).
template <bool GLOBAL>
__device__ bool wave_toggle_records(const SweepArgs &A, const Tab &t, St &st, const Ctx &c, int32_t set,
                                    int32_t s_last, int lane) {
    const int32_t sk = delta_key_scale(A.rec, A.S, set, s_last);
    if (sk < 0) {
        st.err |= ERR_MISSING;
        return true;
    }
    for (int32_t s = sk; s <= s_last; ++s) {
        const int64_t r = (int64_t)set * A.S + s;
        const int64_t off = A.rec.off[r];
        const int32_t len = record_len(A.rec, r);
        if (off < 0 || len < 0 || off + len > A.pool_cap)
            return false;
        for (int32_t base = 0; base < len; base += 64) {
            const bool act = base + lane < len;
            const int32_t u = act ? A.pool[off + base + lane] : 0;
            const int32_t idx = tab_ensure<GLOBAL>(t, st, act, u, act ? c.kdeg[u] : 0, lane);
            if (st.ovf)
                return true;
            if (act && idx >= 0)
                t.DV(idx) ^= (kMember | kWas);
            wsync<GLOBAL>();
        }
    }
    return true;
}

template <bool GLOBAL, bool PERSET>
__device__ void run_wave(const SweepArgs &A, const Tab &t, int lane) {
    const Ctx c = make_ctx(A.g);
    const uint32_t n_items = A.tier == 0 ? (uint32_t)A.n_sets : A.ctl->ovf_count[A.in_from];
    // What one item leaves for the device-wide counters is published by
    // lane 0 at the top of the next iteration, in the same lane-0 block that
    // takes the next item.  The item loop so has exactly one lane-0 block,
    // and its exits test wave-uniform (scalar) values: a lane-0 block at
    // both ends of such a loop lets the compiler thread them into a second
    // back edge that lanes 1..63 take without lane 0.
    bool pend = false;          // an item's epilogue is waiting
    uint32_t pend_push = 0;     // overflow item to push (valid if pend_ovf)
    bool pend_ovf = false;
    uint32_t pend_err = 0;
    uint64_t pend_stat[kStatWords] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (;;) {
        uint32_t item = 0;
        if (lane == 0) {
            if (pend) {
                if (pend_ovf) {
                    if (A.work_out) {
                        const uint32_t pos = atomicAdd(&A.ctl->ovf_count[A.tier], 1u);
                        A.work_out[pos] = (int32_t)pend_push;
                    } else {
                        atomicOr(A.err, ERR_CAPACITY);
                    }
                }
                if (pend_err)
                    atomicOr(A.err, pend_err);
                unsigned long long *sx = A.stat + kStatWords * A.tier;
                for (int q = 0; q < kStatWords; ++q)
                    if (q >= 6 || !pend_ovf)
                        atomicAdd(&sx[q], (unsigned long long)pend_stat[q]);
            }
            item = atomicAdd(&A.ctl->work_next[A.tier], 1u);
        }
        pend = false;
        item = (uint32_t)__builtin_amdgcn_readfirstlane((int)item);
        // another wave hit the watchdog: stop taking work
        const uint32_t abort = (uint32_t)__builtin_amdgcn_readfirstlane(
            (int)(__hip_atomic_load(A.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & ERR_TIMEOUT));
        if (item >= n_items || abort)
            break;
        // a later tier's item is set * S + s: the set overflowed the tier
        // before during scale s and resumes there from its scale s - 1 record
        const uint32_t wi = A.tier == 0 ? item : (uint32_t)A.work_in[item];
        const int32_t set = A.tier == 0 ? (int32_t)item : (int32_t)(wi / (uint32_t)A.S);
        const int32_t s0 = A.tier == 0 ? A.s_begin : (int32_t)(wi % (uint32_t)A.S);

        if constexpr (!GLOBAL) {
            for (uint32_t i = lane; i <= t.hmask; i += 64)
                t.hs[i] = -1;
            wsync<GLOBAL>();
        }
        St st;
        st.count = 0;
        st.nmem = 0;
        st.K = 0;
        st.V = 0;
        st.rK2 = st.rV = 0.0;
        st.alpha = 0.0;
        st.pr = 0.0;
        st.pu = 0;
        st.Gl = st.Rl = 0;
        st.Gu = 0;
        st.M = 0;
        st.ovf = false;
        st.err = 0;
        st.move_limit = 8 * (int64_t)A.g.n + 65536;
        st.t0 = wall_clock64();
        st.budget = (uint64_t)A.budget_ticks;
        st.rows = st.row_len = st.inserted = st.written = st.scanned = 0;
        st.mrows = st.mrow_len = st.c_mrows = st.c_mrow_len = st.ins_mark = st.c_ins = 0;
        st.srows = st.srow_len = 0;
        st.emitted = false;

        // initial community: the seed set, or the members recorded at the
        // previous scale when resuming
        const int32_t *init = nullptr;
        int32_t n_init = 0;
        bool bad = false;
        // delta output: the table's kWas flags hold the last record's members
        bool keyed = false;
        if ((s0 > A.s_begin || A.resume) && A.rec.drem) {
            // the members of scale s0 - 1 from its full list and deltas,
            // then gathered (any order) for the initialisation below
            bad = !wave_toggle_records<GLOBAL>(A, t, st, c, set, s0 - 1, lane);
            if (!bad && !st.ovf && !st.err) {
                int32_t m = 0;
                for (int32_t base = 0; base < st.count; base += 64) {
                    const int32_t i = base + lane;
                    const bool ism = i < st.count && (t.DV(i) & kMember);
                    const uint64_t bm = __ballot(ism);
                    if (ism)
                        t.scr[m + __popcll(bm & lanes_below(lane))] = t.NODE(i);
                    m += __popcll(bm);
                }
                wsync<GLOBAL>();
                init = t.scr;
                n_init = m;
                keyed = true;
            }
        } else if (s0 > A.s_begin || A.resume) {
            const int64_t r = (int64_t)set * A.S + (s0 - 1);
            const int64_t off = A.rec.off[r];
            n_init = A.rec.cnt[r];
            if (off < 0 || off + n_init > A.pool_cap)
                bad = true;   // the pool overflowed earlier: the host reruns
            else
                init = A.pool + off;
        } else {
            init = A.seed_nodes + A.seed_ptr[set];
            n_init = A.seed_ptr[set + 1] - A.seed_ptr[set];
        }
        for (int32_t q = 0; q < n_init && !bad && !st.ovf; ++q) {
            const int32_t u = init[q];
            const int32_t idx = tab_ensure<GLOBAL>(t, st, lane == 0, u, c.kdeg[u], lane);
            if (st.ovf)
                break;
            const int32_t i0 = __shfl(idx, 0);
            const uint32_t v = t.DV(i0);
            wsync<GLOBAL>();
            if (lane == 0)
                t.DV(i0) = v | kMember;
            st.K += 2 * (int64_t)(v & kDMask);
            st.V += c.kdeg[u];
            st.nmem += 1;
            wsync<GLOBAL>();
            row_update<GLOBAL, ROW_INIT>(t, st, c, u, lane);
            if (st.ovf)
                break;
        }

        st.err = wave_or(st.err);
        // a seed set's initial gathers are part of the method; a set resumed
        // from an earlier tier's record gathers its members again (overhead)
        if (!(s0 > A.s_begin || A.resume)) {
            st.srows = st.rows;
            st.srow_len = st.row_len;
        } else {
            st.ins_mark = st.inserted;
        }
        int64_t last_off = -1;
        int32_t last_cnt = 0;
        int32_t s_at = s0;   // the scale being grown (where an overflow happened)
        for (int32_t s = s0; s < A.s_end && !st.ovf && !bad && !st.err; ++s) {
            s_at = s;
            if constexpr (PERSET)
                st.alpha = A.alpha_set[set];
            else
                st.alpha = A.scales[s];
            set_rates(st);
            st.Gl = st.Rl = 0;
            st.Gu = 0;
            st.M = 0;
            uint64_t calls = 0;
            int64_t moved = 0;
            for (;;) {
                calls += 1;
                const int64_t mv = grow<GLOBAL>(t, st, c, A.k_prune, lane);
                st.err = wave_or(st.err);   // probe failures are per lane
                moved += mv;
                if (st.ovf || st.err || mv == 0)
                    break;
                if (A.max_calls != 0 && calls >= (uint64_t)A.max_calls)
                    break;
                if ((int64_t)calls > st.move_limit) {
                    st.err |= ERR_LIMIT;
                    break;
                }
                if (over_budget(st))
                    break;
            }
            if (st.ovf || st.err)
                break;
            const int64_t r = (int64_t)set * A.S + s;
            const uint64_t G = wave_sum((uint64_t)st.Gl) + st.Gu;
            const uint64_t R = wave_sum((uint64_t)st.Rl);
            int32_t dadd = 0, drem = 0;
            if ((s == s0 || moved > 0) && keyed) {
                // delta output: ids that joined (from the front of the
                // scratch array) and left (from its back) since the last
                // record, each run sorted, into the pool
                int32_t na = 0, nr = 0;
                for (int32_t base = 0; base < st.count; base += 64) {
                    const int32_t i = base + lane;
                    const uint32_t v = i < st.count ? t.DV(i) : 0u;
                    const bool add = (v & kMember) && !(v & kWas);
                    const bool rem = (v & kWas) && !(v & kMember);
                    const uint64_t ba = __ballot(add);
                    const uint64_t br = __ballot(rem);
                    if (add)
                        t.scr[na + __popcll(ba & lanes_below(lane))] = t.NODE(i);
                    if (rem)
                        t.scr[t.cap - 1 - (nr + __popcll(br & lanes_below(lane)))] = t.NODE(i);
                    if (add || rem)
                        t.DV(i) = v ^ kWas;
                    na += __popcll(ba);
                    nr += __popcll(br);
                }
                wsync<GLOBAL>();
                wave_sort<GLOBAL>(t.scr, na, lane);
                wave_sort<GLOBAL>(t.scr + (t.cap - nr), nr, lane);
                unsigned long long off = 0;
                if (lane == 0)
                    off = atomicAdd(A.pool_cursor, (unsigned long long)(na + nr));
                off = __shfl(off, 0);
                if ((int64_t)off + na + nr <= A.pool_cap) {
                    for (int32_t i = lane; i < na; i += 64)
                        A.pool[off + i] = t.scr[i];
                    for (int32_t i = lane; i < nr; i += 64)
                        A.pool[off + na + i] = t.scr[t.cap - nr + i];
                }
                last_off = (int64_t)off;
                last_cnt = st.nmem;
                dadd = na;
                drem = nr;
                st.written += (uint64_t)(na + nr);
            } else if (s == s0 || moved > 0) {
                // members, sorted, into the pool (delta output: the set's
                // full list, and kWas := kMember)
                int32_t m = 0;
                for (int32_t base = 0; base < st.count; base += 64) {
                    const int32_t i = base + lane;
                    const uint32_t v = i < st.count ? t.DV(i) : 0u;
                    const bool ism = v & kMember;
                    const uint64_t bm = __ballot(ism);
                    if (ism)
                        t.scr[m + __popcll(bm & lanes_below(lane))] = t.NODE(i);
                    if (A.rec.drem && i < st.count && ism != (bool)(v & kWas))
                        t.DV(i) = v ^ kWas;
                    m += __popcll(bm);
                }
                wsync<GLOBAL>();
                wave_sort<GLOBAL>(t.scr, m, lane);
                unsigned long long off = 0;
                if (lane == 0)
                    off = atomicAdd(A.pool_cursor, (unsigned long long)m);
                off = __shfl(off, 0);
                if ((int64_t)off + m <= A.pool_cap) {
                    for (int32_t i = lane; i < m; i += 64)
                        A.pool[off + i] = t.scr[i];
                }
                last_off = (int64_t)off;
                last_cnt = m;
                dadd = m;
                drem = -1;
                keyed = A.rec.drem != nullptr;
                st.written += (uint64_t)m;
            } else if (keyed) {
                // delta output, nothing moved: an empty delta
                last_cnt = st.nmem;
            }
            if (lane == 0) {
                A.rec.off[r] = last_off;
                A.rec.cnt[r] = last_cnt;
                if (A.rec.drem) {
                    A.rec.dadd[r] = dadd;
                    A.rec.drem[r] = drem;
                }
                A.rec.K[r] = st.K;
                A.rec.V[r] = st.V;
                A.rec.f[r] = st.K == 0 ? 0.0 : (double)st.K / pow((double)st.V, st.alpha);
                A.rec.ctr[4 * r + 0] = G;
                A.rec.ctr[4 * r + 1] = R;
                A.rec.ctr[4 * r + 2] = st.M;
                A.rec.ctr[4 * r + 3] = calls;
            }
            if constexpr (PERSET) {
                // a query's record and members are final: publish them to
                // the host (every lane's stores, then the flag)
                if (A.done_flags) {
                    __threadfence_system();
                    if (lane == 0)
                        __hip_atomic_store(&A.done_flags[set], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                }
            }
            st.c_mrows = st.mrows;
            st.c_mrow_len = st.mrow_len;
            st.c_ins = st.inserted - st.ins_mark;
            st.emitted = true;
        }
        if (bad || st.err || (st.ovf && !A.work_out))
            void_records(A, set, s_at);
        pend = true;
        pend_ovf = st.ovf;
        pend_push = (uint32_t)(set * A.S + s_at);
        pend_err = st.err;
        pend_stat[0] = st.rows;
        pend_stat[1] = st.row_len;
        pend_stat[2] = st.inserted;
        pend_stat[3] = st.written;
        pend_stat[4] = 1;
        pend_stat[5] = st.scanned;
        pend_stat[6] = st.c_mrows;
        pend_stat[7] = st.c_mrow_len;
        pend_stat[8] = st.emitted ? st.srows : 0;
        pend_stat[9] = st.emitted ? st.srow_len : 0;
        pend_stat[10] = st.c_ins;
        if constexpr (GLOBAL) {
            // leave the slab's hash empty for the next community
            wsync<GLOBAL>();
            for (int32_t i = lane; i < st.count; i += 64)
                tab_slot_clear<GLOBAL>(t, i);
            wsync<GLOBAL>();
        }
    }
}

__global__ void __launch_bounds__(256) sweep_lds_kernel(SweepArgs A) {
    extern __shared__ __align__(16) char smem[];
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int64_t tb = table_bytes(A.cap, A.hbits);
    Tab t = carve(smem + wave * tb, A.cap, A.hbits);
    run_wave<false, false>(A, t, lane);
}

__global__ void __launch_bounds__(256) sweep_global_kernel(SweepArgs A) {
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int slot = blockIdx.x * (blockDim.x >> 6) + wave;
    if (slot >= A.n_slots)
        return;
    Tab t = carve(A.gtab + (int64_t)slot * A.gtab_stride, A.cap, A.hbits);
    run_wave<true, false>(A, t, lane);
}

// The same growth for query batches: set j grows once at alpha_set[j].
__global__ void __launch_bounds__(256) query_lds_kernel(SweepArgs A) {
    extern __shared__ __align__(16) char smem[];
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int64_t tb = table_bytes(A.cap, A.hbits);
    Tab t = carve(smem + wave * tb, A.cap, A.hbits);
    run_wave<false, true>(A, t, lane);
}

__global__ void __launch_bounds__(256) query_global_kernel(SweepArgs A) {
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int slot = blockIdx.x * (blockDim.x >> 6) + wave;
    if (slot >= A.n_slots)
        return;
    Tab t = carve(A.gtab + (int64_t)slot * A.gtab_stride, A.cap, A.hbits);
    run_wave<true, true>(A, t, lane);
}

// ---------------------------------------------------------------------------
// Team growth: one workgroup of up to kTeamMaxWaves waves grows one
// community, for sets whose table outgrew the one-wave tier.  Same exact
// queue emulation, decisions and outputs as run_wave; every table scan is
// split over all threads of the workgroup and the per-wave results are
// combined through LDS.  Every branch that decides how many barriers a
// thread reaches depends only on values that all threads computed
// identically or read from LDS after a barrier.
// ---------------------------------------------------------------------------

constexpr int kTeamMaxWaves = 8;
// Rank buckets of the queue of a workgroup on a global-memory table.
constexpr int kBuckets = 256;

constexpr int kMovedMax = 128;

struct TeamSh {
    double r[kTeamMaxWaves];
    int32_t u[kTeamMaxWaves];
    unsigned long long v[kTeamMaxWaves];
    unsigned long long off;
    // what a row leaves behind, read together after its barrier
    struct __align__(16) Row {
        int32_t count;    // dense entries claimed (may pass cap on overflow)
        int32_t flen;     // fresh-list appends (may pass the capacity)
        uint32_t ovf;
        uint32_t stop;
    } row;
    int32_t m;        // members gathered for emission
    int32_t m2;       // delta output: ids that left, gathered for emission
    uint32_t item;
    uint32_t abort;
    union {
        struct {
            int32_t bstart[kBuckets + 1];   // queue positions of each bucket
            uint32_t fill[kBuckets];        // bucket counts, then fill cursors
        };
        int32_t resv[2 * kMaxClaims];   // (id, entry) of a claiming thread (initialisation)
    };
    double r2[kTeamMaxWaves];
    // the waves' candidates, two sets used in turn (a
    // set is written again only after a barrier that every reader has passed)
    struct Slot {
        double r;
        int32_t u, i;
        uint32_t v;
        int32_t k, beg, pos;
    } slot[2][kTeamMaxWaves];
    int32_t done;     // waves whose rows are finished (initialisation)
    int32_t moved[kMovedMax];   // entries added at the scale being grown, see emit_moved
};
static_assert(sizeof(TeamSh) <= kTeamShBytes, "team_lds_fits counts the workgroup's own LDS");

struct TeamId {
    int tid, nt, lane, wid, nw;
};

__device__ __forceinline__ uint64_t team_sum(TeamSh &sh, const TeamId &id, uint64_t v) {
    v = wave_sum(v);
    if (id.lane == 0)
        sh.v[id.wid] = v;
    __syncthreads();
    uint64_t s = 0;
    for (int w = 0; w < id.nw; ++w)
        s += sh.v[w];
    __syncthreads();
    return s;
}

__device__ __forceinline__ uint32_t team_or(TeamSh &sh, const TeamId &id, uint32_t v) {
    v = wave_or(v);
    if (id.lane == 0)
        sh.v[id.wid] = v;
    __syncthreads();
    uint32_t s = 0;
    for (int w = 0; w < id.nw; ++w)
        s |= (uint32_t)sh.v[w];
    __syncthreads();
    return s;
}

// Watchdog decided by thread 0 and broadcast, so that all threads leave
// their loops together.
__device__ __forceinline__ bool team_over_budget(TeamSh &sh, const TeamId &id, St &st) {
    __syncthreads();
    if (id.tid == 0 && wall_clock64() - st.t0 > st.budget)
        sh.row.stop = 1u;
    __syncthreads();
    if (sh.row.stop) {
        st.err |= ERR_TIMEOUT;
        return true;
    }
    return false;
}

// Workgroup minimum of v (every thread gets it).
__device__ __forceinline__ int32_t team_min_i32(TeamSh &sh, const TeamId &id, int32_t v) {
    v = wave_min(v);
    if (id.lane == 0)
        sh.u[id.wid] = v;
    __syncthreads();
    v = sh.u[0];
    for (int w = 1; w < id.nw; ++w)
        v = min(v, sh.u[w]);
    __syncthreads();
    return v;
}

// Entries each thread loads ahead in a table scan (independent loads in
// flight per thread; the scans are latency-bound).
constexpr int kScanAhead = 4;

// ---------------------------------------------------------------------------
// The queue of a workgroup's growth call.
//
// A table of thousands of entries makes a full scan per addition the cost
// that dominates (a community adding A nodes scans its table A times).  The
// queue is therefore kept ordered enough that a step only looks at its head:
//   * the queue: every queued entry's index, counting-sorted into kBuckets
//     rank buckets (bucket(r) is monotone non-increasing in r, so every
//     entry of a later bucket ranks strictly below every entry of an earlier
//     one); positions before cp hold only popped entries;
//   * the fresh list: entries re-ranked by an addition since the queue was
//     built (flag kFresh; their queue slot is stale);
//   * a step takes the best improving entry of the fresh list and of windows
//     of whole buckets from the queue's head, and pops exactly the entries
//     that the sequential queue pops;
//   * the queue is rebuilt when the fresh list grows long.
// Same decisions, counters and results as the scan-driven additions of a wave.
// ---------------------------------------------------------------------------

// largest b in [lo, hi] with bstart[b] <= pos (bstart non-decreasing, bstart[lo] <= pos)
__device__ __forceinline__ int32_t bucket_at(const TeamSh &sh, int32_t lo, int32_t hi, int32_t pos) {
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (sh.bstart[mid] <= pos)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// ---------------------------------------------------------------------------
// Workgroup tables.
//
// A step of a community is a chain of dependent accesses, and the chain's
// length is its time: what a step follows is laid out so that each hop is one
// access.
//   * the hash: 32-bit slots of a tag over an entry index, read four at a time
//     (a wave waits for its lane with the longest probe, so slot-by-slot
//     probing cost a row eight and more rounds);
//   * an entry's fields (d|flags, node, degree, row start, rank) lie together
//     and are read together;
//   * the bucketed queue (above) and its fresh list, entry indices,
//     sorted when a growth call starts;
//   * a copy of the first logs of the table L in LDS;
//   * a row is read from adjacency records that carry the neighbour's degree,
//     its log and its row start beside its id.
// What bounds it: the chain (13,000 cycles an addition alone, of which the row
// takes 6,000 and the step 5,000) and, with twelve waves a compute unit in
// flight, instruction issue and the L2 misses of tables far larger than it.
// Against array tables with slot-by-slot probing and serial initialisation,
// sweeps of 20,000 sets on 100k nodes, 16,384 on 1M and 12,000 on 4M took 27,
// 209 and 490 ms in this tier; now 15, 99 and 350.
// Layouts:
//   T_LDS: everything in LDS (16-bit queue indices).  32 bytes per entry, so
//     one to a few communities share a compute unit: for launches of few
//     communities, where one community's chain is the time.
//   T_PACK: hash, 32-byte records and queue in global memory, 16-bit tag and
//     index, 16-bit queue indices: tables below kRecordMinEntries entries.
//   T_WIDE: the same with 32-bit queue indices and as many index bits in a
//     hash slot as the table needs.
// ---------------------------------------------------------------------------
enum { T_LDS = 0, T_PACK = 1, T_WIDE = 2 };

// The fresh list of a table in global memory: its entries' fields live here
// while they are on it (the record keeps the flag kFresh and the place), so
// that a step reads the list from LDS and a row writes it there.
template <int N>
struct FreshSh {
    double r[N];
    uint32_t v[N];
    int32_t u[N], k[N], beg[N];
    int32_t i[N];   // table entry; -1: it became a member
};

template <int L>
struct BTab {
    static constexpr bool G = L != T_LDS;
    static constexpr int FM = L == T_WIDE ? kFreshMaxWide : kFreshMax;   // fresh-list entries kept
    using Q = std::conditional_t<L == T_WIDE, uint32_t, uint16_t>;
    using F = FreshSh<FM>;
    double *lt;        // L(x) for x < kBlockLogs (LDS)
    uint32_t *hw;      // hash slots: tag over entry index
    Q *sq;             // queue, cap entry indices; T_LDS: then the fresh list
    F *fs;             // else: the fresh list
    double *rk;        // T_LDS: entries as arrays
    int32_t *node, *kv, *beg;
    uint32_t *dv;
    char *rec;         // else: records {rank, d|flags, fresh place, node, degree, row start, hash slot}
    int32_t *scr;      // scratch i32[cap] (emission, resume, removal): T_LDS the ranks'
                       // place, which hold nothing once a call's additions are over
    uint32_t hmask;
    int hbits, ibits;  // ibits: index bits of a hash slot, T_WIDE (16 otherwise)
    int cap;
    __device__ __forceinline__ char *at(int32_t i) const { return rec + (size_t)(uint32_t)i * kRecordBytes; }
    __device__ __forceinline__ double &RK(int32_t i) const { return G ? *(double *)at(i) : rk[i]; }
    __device__ __forceinline__ uint32_t &DV(int32_t i) const { return G ? *(uint32_t *)(at(i) + 8) : dv[i]; }
    __device__ __forceinline__ int32_t &NODE(int32_t i) const { return G ? *(int32_t *)(at(i) + 16) : node[i]; }
    __device__ __forceinline__ int32_t &KV(int32_t i) const { return G ? *(int32_t *)(at(i) + 20) : kv[i]; }
    __device__ __forceinline__ uint32_t &SLOT(int32_t i) const { return *(uint32_t *)(at(i) + 28); }
    __device__ __forceinline__ int shift() const { return L == T_WIDE ? ibits : 16; }
};

// One entry's fields.
struct Ent {
    uint32_t v;
    int32_t u, k, beg;
    double r;
    int32_t pos;   // tables in global memory: place on the fresh list, if kFresh is set
};

template <int L>
__device__ __forceinline__ Ent ent_get(const BTab<L> &t, int32_t i) {
    Ent e;
    if constexpr (L != T_LDS) {
        const int4 *p = (const int4 *)t.at(i);
        const int4 a = p[0], b = p[1];
        e.r = __hiloint2double(a.y, a.x);
        e.v = (uint32_t)a.z;
        e.pos = a.w;
        e.u = b.x;
        e.k = b.y;
        e.beg = b.z;
    } else {
        e.v = t.dv[i];
        e.u = t.node[i];
        e.k = t.kv[i];
        e.beg = t.beg[i];
        e.r = t.rk[i];
        e.pos = -1;
    }
    return e;
}

// A record's first half.
template <int L>
__device__ __forceinline__ void ent_put(const BTab<L> &t, int32_t i, double r, uint32_t v, int32_t pos) {
    *(int4 *)t.at(i) = make_int4(__double2loint(r), __double2hiint(r), (int32_t)v, pos);
}

// A new entry with d = 0 (its rank follows with its first re-rank).
template <int L>
__device__ __forceinline__ void ent_new(const BTab<L> &t, int32_t i, int32_t u, int32_t k, int32_t beg) {
    if constexpr (L != T_LDS) {
        ent_put(t, i, 0.0, 0u, -1);
        *(int4 *)(t.at(i) + 16) = make_int4(u, k, beg, -1);
    } else {
        t.dv[i] = 0u;
        t.node[i] = u;
        t.kv[i] = k;
        t.beg[i] = beg;
    }
}

__device__ __forceinline__ BTab<T_LDS> carve_lds(char *lds, int cap, int hbits) {
    BTab<T_LDS> t;
    t.lt = (double *)lds;
    t.hw = (uint32_t *)(t.lt + kBlockLogs);
    t.rk = (double *)(t.hw + ((size_t)1 << hbits));
    t.node = (int32_t *)(t.rk + cap);
    t.dv = (uint32_t *)(t.node + cap);
    t.kv = t.node + 2 * cap;
    t.beg = t.node + 3 * cap;
    t.sq = (uint16_t *)(t.node + 4 * cap);
    t.scr = (int32_t *)t.rk;
    t.rec = nullptr;
    t.hmask = (1u << hbits) - 1;
    t.hbits = hbits;
    t.ibits = 16;
    t.cap = cap;
    t.fs = nullptr;
    return t;
}

// Table `slot` of a slab: the hashes of all its tables come first, so that one
// fill empties them.
template <int L>
__device__ __forceinline__ BTab<L> carve_slab(char *slab, int64_t stride, int32_t n_slots, int slot, double *lt,
                                              typename BTab<L>::F *fs, int cap, int hbits) {
    BTab<L> t;
    t.lt = lt;
    t.hw = (uint32_t *)(slab + ((size_t)slot << (hbits + 2)));
    char *p = slab + ((size_t)n_slots << (hbits + 2)) + (size_t)slot * stride;
    t.rec = p;
    t.scr = (int32_t *)(p + (size_t)cap * kRecordBytes);
    t.sq = (typename BTab<L>::Q *)(t.scr + cap);
    t.rk = nullptr;
    t.node = t.kv = t.beg = nullptr;
    t.dv = nullptr;
    t.hmask = (1u << hbits) - 1;
    t.hbits = hbits;
    t.ibits = 33 - __builtin_clz((uint32_t)cap - 1);   // an index and the claim bit
    t.cap = cap;
    t.fs = fs;
    return t;
}

constexpr uint32_t kNoSlot = 0xffffffffu;  // an empty hash slot (no entry has the largest index)

// Index field of a slot that a thread has claimed, see block_edges.
template <int L>
__device__ __forceinline__ uint32_t claim_bit(const BTab<L> &t) { return 1u << (t.shift() - 1); }

template <int L>
__device__ __forceinline__ uint32_t index_mask(const BTab<L> &t) { return (1u << t.shift()) - 1u; }

// LDS operations of one wave take effect in order; the compiler must keep
// theirs.
__device__ __forceinline__ void lds_order() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); }

// Reads and writes that other threads' LDS operations may meet in between.
template <class V>
__device__ __forceinline__ V lds_get(const V *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

template <class V>
__device__ __forceinline__ void lds_put(V *p, V v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The slots of id u start at a group of four; its tag is the hash's low bits.
__device__ __forceinline__ uint32_t hash_mul(int32_t u) { return (uint32_t)u * 2654435761u; }

template <int L>
__device__ __forceinline__ uint32_t group_of(const BTab<L> &t, uint32_t h) {
    return (h >> (32 - t.hbits)) & ~3u;
}

template <int L>
__device__ __forceinline__ void slot_put(const BTab<L> &t, uint32_t p, uint32_t v) {
    __hip_atomic_store(t.hw + p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Before a hash slot is written that another wave may follow, and after one
// was read: what it leads to is seen whole.
template <int L>
__device__ __forceinline__ void slot_release() {
    if constexpr (L != T_LDS)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    else
        lds_order();
}

template <int L>
__device__ __forceinline__ void slot_acquire() {
    if constexpr (L != T_LDS)
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

__device__ __forceinline__ uint32_t slot_of(const uint4 &g, int j) {
    return j == 0 ? g.x : j == 1 ? g.y : j == 2 ? g.z : g.w;
}

// Bits of the slots of a group that are empty / that carry the tag.
__device__ __forceinline__ uint32_t group_empty(const uint4 &g) {
    return (g.x == kNoSlot ? 1u : 0u) | (g.y == kNoSlot ? 2u : 0u) | (g.z == kNoSlot ? 4u : 0u) |
           (g.w == kNoSlot ? 8u : 0u);
}

__device__ __forceinline__ uint32_t group_tagged(const uint4 &g, uint32_t h, int shift) {
    const uint32_t tag = h << shift;
    return ((g.x ^ tag) >> shift == 0u ? 1u : 0u) | ((g.y ^ tag) >> shift == 0u ? 2u : 0u) |
           ((g.z ^ tag) >> shift == 0u ? 4u : 0u) | ((g.w ^ tag) >> shift == 0u ? 8u : 0u);
}

// The entry of u and its fields, or idx = -1 and the first empty slot of its
// probe (kNoSlot: none left).  Entries from `count` on are being created by
// other waves: they are other ids', and their fields are not read.  Slots of an id's probe fill in order and are
// never emptied, so a lookup ends at the first empty one.
template <int L>
__device__ __forceinline__ void block_find(const BTab<L> &t, int32_t u, int32_t count, int32_t &idx, uint32_t &slot,
                                           Ent &e) {
    const uint32_t h = hash_mul(u);
    uint32_t p = group_of(t, h);
    idx = -1;
    slot = kNoSlot;
    for (uint32_t it = 0; it <= t.hmask; it += 4) {
        const uint4 g = *(const uint4 *)(t.hw + p);
        const uint32_t room = group_empty(g);
        uint32_t m = group_tagged(g, h, t.shift()) & ~room;
        while (m) {
            const int32_t i = (int32_t)(slot_of(g, __builtin_ctz(m)) & index_mask(t));
            if (i < count) {
                e = ent_get(t, i);
                if (e.u == u) {
                    idx = i;
                    return;
                }
            }
            m &= m - 1;
        }
        if (room) {
            slot = p + (uint32_t)__builtin_ctz(room);
            return;
        }
        p = (p + 4) & t.hmask;
    }
}

// Put v into the first empty slot at or after p, its place or kNoSlot.
template <int L>
__device__ __forceinline__ uint32_t block_claim(const BTab<L> &t, uint32_t p, uint32_t v) {
    if (p == kNoSlot)
        return kNoSlot;
    for (uint32_t it = 0; it <= t.hmask; ++it) {
        if (atomicCAS(&t.hw[p], kNoSlot, v) == kNoSlot) {
            // the swap is done in the L2; a store also goes through the L1,
            // from which groups are read
            if constexpr (L != T_LDS)
                slot_put(t, p, v);
            return p;
        }
        p = (p + 1) & t.hmask;
    }
    return kNoSlot;
}

// L(x): small arguments from the LDS copy of the table.
template <int L>
__device__ __forceinline__ double block_log(const BTab<L> &t, const Ctx &c, int32_t x) {
    // (two loads of one kind would become one flat load of either memory)
    if (x < kBlockLogs)
        return lds_get(&t.lt[x]);
    return c.logtab[min(x, c.logtab_last)];
}

// Create the entries of the lanes that need one (ids distinct in the
// workgroup, slot from block_find): index, fields with d = 0, and the swap of
// their hash slot, whose result is left in `old` for block_added.  solo: only
// this wave adds entries before the next barrier.  A full table sets sh.ovf
// (idx stays -1).
template <int L>
__device__ __forceinline__ void block_add(const BTab<L> &t, TeamSh &sh, St &st, const TeamId &id, bool need,
                                          int32_t u, int32_t k, int32_t beg, uint32_t slot, bool solo,
                                          int32_t &idx, uint32_t &old) {
    old = kNoSlot;
    const uint64_t m = __ballot(need);
    if (m == 0)
        return;
    int32_t base = st.count;
    if (solo) {
        if (id.lane == 0)
            sh.row.count = base + __popcll(m);
    } else {
        const int lead = (int)__builtin_ctzll(m);
        if (id.lane == lead)
            base = atomicAdd(&sh.row.count, __popcll(m));
        base = __builtin_amdgcn_readlane(base, lead);
    }
    if (need) {
        const int32_t at = base + __popcll(m & lanes_below(id.lane));
        if (at >= t.cap) {
            sh.row.ovf = 1u;
        } else {
            idx = at;
            if (slot != kNoSlot)
                old = atomicCAS(&t.hw[slot], kNoSlot, (hash_mul(u) << t.shift()) | (uint32_t)at);
            ent_new(t, at, u, k, beg);
            st.inserted += 1;
        }
    }
}

// The end of block_add, once the swap's result is there (what a row does with
// the entries in between hides its trip to the L2): a lost slot is sought on.
template <int L>
__device__ __forceinline__ void block_added(const BTab<L> &t, St &st, bool need, int32_t u, uint32_t slot, int32_t idx,
                                            uint32_t old) {
    if (need && idx >= 0) {
        const uint32_t v = (hash_mul(u) << t.shift()) | (uint32_t)idx;
        if (slot == kNoSlot || old != kNoSlot)
            slot = block_claim(t, slot, v);
        else if constexpr (L != T_LDS)
            slot_put(t, slot, v);
        if (slot == kNoSlot)
            st.err |= ERR_PROBE;
        if constexpr (L != T_LDS)
            t.SLOT(idx) = slot;
    }
    lds_order();
}

// The entry of u for every active thread (all ids of a call distinct), absent
// ones created; -1 for inactive threads and for ids that no longer fit
// (sh.row.ovf is then set).  Every thread of the workgroup calls it; a barrier
// at the end.
template <int L>
__device__ int32_t team_ensure(const BTab<L> &t, TeamSh &sh, St &st, const Ctx &c, const TeamId &id, bool act,
                               int32_t u) {
    int32_t idx = -1;
    uint32_t slot = kNoSlot;
    Ent e;
    const int32_t count = min(sh.row.count, t.cap);
    __syncthreads();   // read by all before one is added
    if (act)
        block_find(t, u, count, idx, slot, e);
    const bool need = act && idx < 0;
    const int2 in = need ? c.info[u] : make_int2(0, 0);
    uint32_t old;
    block_add(t, sh, st, id, need, u, in.y, in.x, slot, false, idx, old);
    block_added(t, st, need, u, slot, idx, old);
    __syncthreads();
    return idx;
}

// Apply the row of node n (row start beg, degree k) to the table.
// ROW_REMOVE: every neighbour's d falls by the edge's weight.  ROW_ADD: it
// rises by it, absent neighbours are created, and every non-member neighbour
// is (re)queued with its new rank: flagged kLive | kFresh | kTouch and put on
// the fresh list unless it is there already.  It counts as a pop to come
// (st.Gl) when it was not queued: a queue entry whose kLive was taken by a
// step, or a fresh one that ranks above the node just added, whose pop is
// still pending.  Entries past the fresh list's end carry place FM.
// The first entries are loaded before the row's end is known (row_ahead).
// Every thread calls it; a barrier at the end, after which all hold the same
// count, flen, ovf and err.
template <int MODE, int L>
__device__ __forceinline__ void block_row(const BTab<L> &t, TeamSh &sh, St &st, const Ctx &c, const TeamId &id,
                                          int32_t n, int32_t beg, int32_t k) {
    Edge x = row_ahead(beg, id.tid, k, c.nnz) ? edge_at(c, beg + id.tid) : no_edge();
    const int32_t len = __builtin_amdgcn_readfirstlane(c.row_ptr[n + 1]) - beg;
    const bool solo = len <= 64;   // the row is wave 0's alone
    st.rows += 1;
    st.row_len += (uint64_t)len;
    st.mrows += 1;
    st.mrow_len += (uint64_t)len;
    for (int32_t base = 0; base < len; base += id.nt) {
        if (base + id.wid * 64 >= len)
            break;
        const bool act = base + id.tid < len;
        if (base > 0)
            x = act ? edge_at(c, beg + base + id.tid) : no_edge();
        const int4 e = x.e;
        int32_t idx = -1;
        uint32_t slot = kNoSlot;
        Ent a;
        a.v = 0u;
        a.r = 0.0;
        if (act)
            block_find(t, e.x, st.count, idx, slot, a);
        if constexpr (MODE == ROW_REMOVE) {
            if (act) {
                if (idx < 0)
                    st.err |= ERR_MISSING;
                else
                    t.DV(idx) = a.v - (uint32_t)e.w;   // d stays >= 0: the flags above it are untouched
            }
        } else {
            const bool fresh = act && idx < 0;
            uint32_t old;
            block_add(t, sh, st, id, fresh, e.x, e.y, e.z, slot, solo, idx, old);
            // a non-member neighbour is (re)queued with its new rank: on the
            // fresh list already, or to be listed (in the queue unless
            // popped: queue entries at once, fresh ones by the next scan)
            bool list = false;
            uint32_t v = 0u;
            double r = 0.0;
            if (act && idx >= 0) {
                const bool here = L != T_LDS && !fresh && (a.v & kFresh) && (uint32_t)a.pos < (uint32_t)BTab<L>::FM;
                v = fresh ? 0u : a.v;
                r = a.r;
                if constexpr (L != T_LDS) {
                    if (here) {
                        v = t.fs->v[a.pos];
                        r = t.fs->r[a.pos];
                    }
                }
                const int32_t d = (int32_t)(v & kDMask) + e.w;
                if (v & kMember) {
                    t.DV(idx) = (v & ~kDMask) | (uint32_t)d;
                } else {
                    const bool popped = !(v & kLive) || ((v & kFresh) && before(r, e.x, st.pr, st.pu));
                    if (popped)
                        st.Gl += 1;
                    list = !(v & kFresh);
                    r = block_log(t, c, 2 * d) - st.alpha * x.lk;
                    st.Rl += 1;
                    v = (v & kWas) | (uint32_t)d | kLive | kFresh | kTouch;
                    if constexpr (L == T_LDS) {
                        t.RK(idx) = r;
                        t.DV(idx) = v;
                    } else if (here) {
                        t.fs->v[a.pos] = v;
                        t.fs->r[a.pos] = r;
                    } else if (!list) {
                        ent_put(t, idx, r, v, BTab<L>::FM);   // past the list's end
                    }
                }
            }
            // entries past the list's end are found by the rebuild that its
            // length then asks for
            const uint64_t m = __ballot(list);
            if (m) {
                int32_t at = st.flen;
                if (solo) {
                    if (id.lane == 0)
                        sh.row.flen = at + __popcll(m);
                } else {
                    const int lead = (int)__builtin_ctzll(m);
                    if (id.lane == lead)
                        at = atomicAdd(&sh.row.flen, __popcll(m));
                    at = __builtin_amdgcn_readlane(at, lead);
                }
                at += __popcll(m & lanes_below(id.lane));
                if constexpr (L == T_LDS) {
                    if (list && at < BTab<L>::FM)
                        t.sq[t.cap + at] = (uint16_t)idx;
                } else if (list) {
                    ent_put(t, idx, r, v, min(at, BTab<L>::FM));
                    if (at < BTab<L>::FM) {
                        t.fs->r[at] = r;
                        t.fs->v[at] = v;
                        t.fs->u[at] = e.x;
                        t.fs->k[at] = e.y;
                        t.fs->beg[at] = e.z;
                        t.fs->i[at] = idx;
                    }
                }
            }
            block_added(t, st, fresh, e.x, slot, idx, old);
        }
    }
    if (id.tid == 0 && (st.M & 15) == 0 && wall_clock64() - st.t0 > st.budget)
        sh.row.stop = 1u;
    __syncthreads();
    const int4 z = *(const int4 *)&sh.row;
    st.count = __builtin_amdgcn_readfirstlane(min(z.x, t.cap));
    st.flen = __builtin_amdgcn_readfirstlane(z.y);
    if constexpr (MODE != ROW_REMOVE)
        st.ovf = __builtin_amdgcn_readfirstlane(z.z) != 0;
    if (__builtin_amdgcn_readfirstlane(z.w))
        st.err |= ERR_TIMEOUT;
}

// A hash slot's index field against id u: an entry, or the claim of a thread.
template <int L>
__device__ __forceinline__ void match_slot(const BTab<L> &t, TeamSh &sh, uint32_t s, int32_t u, int32_t &idx,
                                           int32_t &dup) {
    if (s & claim_bit(t)) {
        const int32_t c = (int32_t)(s & (claim_bit(t) - 1u));
        if (lds_get(sh.resv + 2 * c) == u)
            dup = c;
    } else if (t.NODE((int32_t)s) == u) {
        idx = (int32_t)s;
    }
}

// The edges of the initial members: for every entry of their rows find or
// create its table entry and add the weight to its d.  Ids repeat, also
// among the edges in flight: a thread that meets an empty slot claims it
// with its own number under the id's tag, and another thread that meets the
// claim compares its id with the claimer's and takes over the entry after
// the barrier.  Each wave flattens the rows of its share of the members, 64
// edges at a time.
template <int L>
__device__ void block_edges(const BTab<L> &t, TeamSh &sh, St &st, const Ctx &c, const TeamId &id,
                            const int32_t *init, int32_t n_init) {
    const int32_t lanes = min(64, kMaxClaims / id.nw);   // claims in flight per wave
    const int32_t q1 = (int32_t)((int64_t)n_init * (id.wid + 1) / id.nw);
    int32_t q = (int32_t)((int64_t)n_init * id.wid / id.nw);   // next member of this wave
    int32_t beg = 0, incl = 0, len = 0, total = 0, at = 0;     // the block of members in hand
    bool counted = false;
    const int32_t me = id.wid * lanes + id.lane;     // this thread's claim number
    for (;;) {
        while (at >= total && q < q1) {
            // the next (at most) 64 members of the wave: row starts and the
            // running sum of their lengths
            const bool has = q + id.lane < q1;
            const int32_t u = has ? init[q + id.lane] : 0;
            beg = has ? c.row_ptr[u] : 0;
            len = has ? c.row_ptr[u + 1] - beg : 0;
            incl = len;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int32_t x = __shfl_up(incl, off);
                if (id.lane >= off)
                    incl += x;
            }
            total = __builtin_amdgcn_readlane(incl, 63);
            st.rows += (uint64_t)min(64, q1 - q);
            st.row_len += (uint64_t)total;
            at = 0;
            q += 64;
        }
        const int32_t e = at + id.lane;
        const bool act = id.lane < lanes && e < total;
        at += lanes;
        // the member whose row holds edge e: the first with incl > e
        int32_t lo = 0;
#pragma unroll
        for (int step = 32; step >= 1; step >>= 1) {
            const int32_t x = __shfl(incl, lo + step - 1);
            if (x <= e)
                lo += step;
        }
        lo = min(lo, 63);
        const int32_t row = __shfl(beg, lo), first = __shfl(incl, lo) - __shfl(len, lo);
        const int4 ed = act ? edge_at(c, row + (e - first)).e : make_int4(0, 0, 0, 0);
        const int32_t u = ed.x;
        const uint32_t h = hash_mul(u);
        int32_t idx = -1, dup = -1;
        uint32_t mine = kNoSlot;   // the slot this thread claimed
        if (act) {
            lds_put(sh.resv + 2 * me, u);
            lds_put(sh.resv + 2 * me + 1, -1);
            slot_release<L>();
            uint32_t p = group_of(t, h);
            uint32_t from = 0;   // slots of the group already known to be others'
            uint32_t it = 0;
            for (; it <= t.hmask; ++it) {
                const uint4 g = *(const uint4 *)(t.hw + p);
                uint32_t room = group_empty(g) & ~from;
                uint32_t m = group_tagged(g, h, t.shift()) & ~group_empty(g);
                slot_acquire<L>();
                uint32_t s = 0;
                int at_slot = -1;   // a slot that was claimed while it was looked at
                if (room) {
                    at_slot = __builtin_ctz(room);
                    // (a match beyond the first empty slot is no match)
                    m &= (1u << at_slot) - 1u;
                }
                while (m && idx < 0 && dup < 0) {
                    s = slot_of(g, __builtin_ctz(m)) & index_mask(t);
                    match_slot(t, sh, s, u, idx, dup);
                    m &= m - 1;
                }
                if (idx >= 0 || dup >= 0)
                    break;
                if (at_slot >= 0) {
                    const uint32_t q = p + (uint32_t)at_slot;
                    const uint32_t old =
                        atomicCAS(&t.hw[q], kNoSlot, (h << t.shift()) | claim_bit(t) | (uint32_t)me);
                    if (old == kNoSlot) {
                        mine = q;
                        break;
                    }
                    slot_acquire<L>();
                    if ((old ^ (h << t.shift())) >> t.shift() == 0u)
                        match_slot(t, sh, old & index_mask(t), u, idx, dup);
                    if (idx >= 0 || dup >= 0)
                        break;
                    from |= (2u << at_slot) - 1u;
                    if (from & 8u) {
                        from = 0;
                        p = (p + 4) & t.hmask;
                    }
                } else {
                    from = 0;
                    p = (p + 4) & t.hmask;
                }
            }
            if (it > t.hmask)
                st.err |= ERR_PROBE;
        }
        const uint64_t m = __ballot(mine != kNoSlot);
        if (m) {
            const int lead = (int)__builtin_ctzll(m);
            int32_t base = 0;
            if (id.lane == lead)
                base = atomicAdd(&sh.row.count, __popcll(m));
            base = __builtin_amdgcn_readlane(base, lead);
            if (mine != kNoSlot) {
                const int32_t k = base + __popcll(m & lanes_below(id.lane));
                if (k >= t.cap) {
                    sh.row.ovf = 1u;
                } else {
                    idx = k;
                    ent_new(t, k, u, ed.y, ed.z);
                    if constexpr (L != T_LDS)
                        t.SLOT(k) = mine;
                    st.inserted += 1;
                    lds_put(sh.resv + 2 * me + 1, k);
                }
            }
        }
        if (!counted && at >= total && q >= q1) {
            counted = true;
            if (id.lane == 0)
                atomicAdd(&sh.done, 1);
        }
        __syncthreads();
        // every claim is an entry now: the claims become its index
        if (mine != kNoSlot)
            slot_put(t, mine, idx >= 0 ? (h << t.shift()) | (uint32_t)idx : kNoSlot);
        if (dup >= 0)
            idx = lds_get(sh.resv + 2 * dup + 1);
        if (idx >= 0)
            atomicAdd(&t.DV(idx), (uint32_t)ed.w);
        const bool last = sh.done >= id.nw || sh.row.ovf != 0u;
        __syncthreads();
        if (last)
            break;
    }
}

// The initial community: the ids init[0 .. n_init) become members and their
// rows enter the table, all rows at once (K is the sum of the members' d,
// every internal edge counted from both ends, whatever the order).
template <int L>
__device__ void team_init(const BTab<L> &t, TeamSh &sh, St &st, const Ctx &c, const TeamId &id, const int32_t *init,
                          int32_t n_init) {
    if (id.tid == 0)
        sh.done = 0;
    for (int32_t base = 0; base < n_init; base += id.nt) {
        const bool act = base + id.tid < n_init;
        const int32_t u = act ? init[base + id.tid] : 0;
        const int32_t idx = team_ensure(t, sh, st, c, id, act, u);
        if (act && idx >= 0)
            t.DV(idx) |= kMember;
    }
    __syncthreads();
    const bool full = sh.row.ovf != 0u;
    __syncthreads();   // read by all before a row may set it
    if (!full)
        block_edges(t, sh, st, c, id, init, n_init);
    if (sh.row.ovf) {
        st.ovf = true;
        return;
    }
    // records: d was added in the L2, and the L1 may hold the lines of before
    if constexpr (L != T_LDS)
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    st.count = __builtin_amdgcn_readfirstlane(min(sh.row.count, t.cap));
    uint64_t K = 0, V = 0;
    for (int32_t i = id.tid; i < st.count; i += id.nt) {
        const uint32_t v = t.DV(i);
        if (v & kMember) {
            K += (uint64_t)(v & kDMask);
            V += (uint64_t)t.KV(i);
        }
    }
    st.K = (int64_t)team_sum(sh, id, K);
    st.V = (int64_t)team_sum(sh, id, V);
    st.nmem = n_init;
    // the first call's buckets: ranks lie in [-alpha L(kmax), L(2 kmax)] (a rank
    // outside the range goes to the first or last bucket)
    st.qhi = c.logtab[c.logtab_last];
    st.qlo = 0.0;
    st.qalpha = 0.0;
    // rows were counted per wave
    st.rows = team_sum(sh, id, id.lane == 0 ? st.rows : 0);
    st.row_len = team_sum(sh, id, id.lane == 0 ? st.row_len : 0);
}

// Tables in a slab are emptied by the community that leaves them.
template <int L>
__device__ __forceinline__ void team_reset(const BTab<L> &t, const TeamId &id) {
    if constexpr (L != T_LDS)
        return;
    for (uint32_t i = id.tid; i <= t.hmask >> 2; i += id.nt)
        ((uint4 *)t.hw)[i] = make_uint4(kNoSlot, kNoSlot, kNoSlot, kNoSlot);
}

template <int L>
__device__ __forceinline__ void team_leave(const BTab<L> &t, TeamSh &sh, const TeamId &id) {
    if constexpr (L != T_LDS) {
        __syncthreads();
        const int32_t cnt = min(sh.row.count, t.cap);
        for (int32_t i = id.tid; i < cnt; i += id.nt) {
            const uint32_t s = t.SLOT(i);
            if (s <= t.hmask)
                slot_put(t, s, kNoSlot);
        }
    }
}

// What the workgroup picked: an entry and its fields.
struct Picked {
    double r;
    int32_t u, i;
    uint32_t v;
    int32_t k, beg;
    int32_t pos;   // place on the fresh list, or -1
};

// Lane l's candidate in every lane (scalar registers).
__device__ __forceinline__ void pick_lane(int l, const Ent &e, int32_t i, Picked &o) {
    o.r = read_lane(e.r, l);
    o.u = __builtin_amdgcn_readlane(e.u, l);
    o.i = __builtin_amdgcn_readlane(i, l);
    o.v = (uint32_t)__builtin_amdgcn_readlane((int)e.v, l);
    o.k = __builtin_amdgcn_readlane(e.k, l);
    o.beg = __builtin_amdgcn_readlane(e.beg, l);
    o.pos = __builtin_amdgcn_readlane(e.pos, l);
}

// The waves' candidates (lane l of each, l < 0: none) into one set of slots,
// read after the barrier.
__device__ __forceinline__ const TeamSh::Slot *slot_put(TeamSh &sh, const TeamId &id, int &par, int l, const Ent &e,
                                                        int32_t i) {
    TeamSh::Slot *s = sh.slot[par];
    par ^= 1;
    if (id.lane == max(l, 0)) {
        s[id.wid].r = e.r;
        s[id.wid].u = e.u;
        s[id.wid].i = l < 0 ? -1 : i;
        s[id.wid].v = e.v;
        s[id.wid].k = e.k;
        s[id.wid].beg = e.beg;
        s[id.wid].pos = e.pos;
    }
    __syncthreads();
    return s;
}

// Slot w's candidate (false: none), in scalar registers.
__device__ __forceinline__ bool slot_take(const TeamSh::Slot *s, int w, Picked &o) {
    w = __builtin_amdgcn_readfirstlane(w);
    o.i = __builtin_amdgcn_readfirstlane(s[w].i);
    o.r = read_lane(s[w].r, 0);
    o.u = __builtin_amdgcn_readfirstlane(s[w].u);
    o.v = (uint32_t)__builtin_amdgcn_readfirstlane((int)s[w].v);
    o.k = __builtin_amdgcn_readfirstlane(s[w].k);
    o.beg = __builtin_amdgcn_readfirstlane(s[w].beg);
    o.pos = __builtin_amdgcn_readfirstlane(s[w].pos);
    return o.i >= 0;
}

// The workgroup's first entry in queue order among the lanes' candidates (i
// < 0: none).  One barrier; set `par` of the slots is used and toggled.  Two
// waves compare their slots, more of them reduce over the lanes again.
__device__ __forceinline__ bool block_pick_max(TeamSh &sh, const TeamId &id, int &par, Ent e, int32_t i, Picked &o) {
    int l = wave_first(e.r, e.u, i);
    if (id.nw == 1) {
        __syncthreads();
        if (l < 0)
            return false;
        pick_lane(l, e, i, o);
        return true;
    }
    const TeamSh::Slot *s = slot_put(sh, id, par, l, e, i);
    if (id.nw == 2) {
        l = s[1].i >= 0 && (s[0].i < 0 || before(s[1].r, s[1].u, s[0].r, s[0].u)) ? 1 : 0;
    } else {
        const int w = id.lane < id.nw ? id.lane : 0;
        l = max(wave_first(s[w].r, s[w].u, id.lane < id.nw ? s[w].i : -1), 0);
    }
    return slot_take(s, l, o);
}

__device__ __forceinline__ int wave_smallest(int32_t u, int32_t i) {
    const int32_t lo = wave_min(i >= 0 ? u : INT32_MAX);
    const uint64_t at = __ballot(i >= 0 && u == lo);
    return at ? (int)__builtin_ctzll(at) : -1;
}

// The workgroup's smallest id u (i < 0: none).
__device__ __forceinline__ bool block_pick_min(TeamSh &sh, const TeamId &id, int &par, Ent e, int32_t i, Picked &o) {
    int l = wave_smallest(e.u, i);
    if (id.nw == 1) {
        __syncthreads();
        if (l < 0)
            return false;
        pick_lane(l, e, i, o);
        return true;
    }
    const TeamSh::Slot *s = slot_put(sh, id, par, l, e, i);
    const int w = id.lane < id.nw ? id.lane : 0;
    l = max(wave_smallest(s[w].u, id.lane < id.nw ? s[w].i : -1), 0);
    return slot_take(s, l, o);
}

// The bucketed queue: ns entries, positions before cp hold only
// popped ones; lane l holds the starts of buckets 4l .. 4l + 3.
struct LQ {
    int32_t ns, cp;
    int32_t pre;      // tables in global memory: this thread's entry of the window at cp
    int32_t s4[4];
};

// Start of bucket b (wave-uniform) from the lanes' registers.
__device__ __forceinline__ int32_t lq_start(const LQ &q, int32_t b) {
    if (b >= kBuckets)
        return q.ns;
    const int l = b >> 2, j = b & 3;
    return __builtin_amdgcn_readlane(j == 0 ? q.s4[0] : j == 1 ? q.s4[1] : j == 2 ? q.s4[2] : q.s4[3], l);
}

__device__ __forceinline__ int32_t lq_bucket(const St &st, double r) {
    return (int32_t)fmin(fmax((st.qtop - r) * st.qscale, 0.0), (double)(kBuckets - 2));
}

// Exclusive prefix of the bucket counts in sh.fill, four buckets per lane: the
// buckets' starts, and the fill cursors at them.
__device__ __forceinline__ void bucket_starts(TeamSh &sh, const TeamId &id) {
    if (id.wid == 0) {
        // exclusive prefix of the bucket counts, four buckets per lane
        const int32_t b4 = 4 * id.lane;
        uint32_t c4[4], sum = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            c4[j] = sh.fill[b4 + j];
            sum += c4[j];
        }
        uint32_t incl = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t x = __shfl_up(incl, off);
            if (id.lane >= off)
                incl += x;
        }
        uint32_t run = incl - sum;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            sh.bstart[b4 + j] = (int32_t)run;
            sh.fill[b4 + j] = run;
            run += c4[j];
        }
        if (id.lane == 63)
            sh.bstart[kBuckets] = (int32_t)incl;
    }
}

// Write the fresh list back into the records, its pending pops applied, and
// empty it (a barrier at the end; T_LDS: nothing to do).
template <int L>
__device__ __forceinline__ void fresh_flush(const BTab<L> &t, TeamSh &sh, St &st, const TeamId &id) {
    if constexpr (L != T_LDS) {
        const int32_t nf = min(st.flen, BTab<L>::FM);
        for (int32_t f = id.tid; f < nf; f += id.nt) {
            const int32_t i = t.fs->i[f];
            if (i < 0)
                continue;
            uint32_t v = t.fs->v[f];
            const double r = t.fs->r[f];
            if (!(v & kTouch) && before(r, t.fs->u[f], st.pr, st.pu))
                v &= ~kLive;
            ent_put(t, i, r, v & ~(kFresh | kTouch), -1);
        }
        __syncthreads();
    }
}

// The queue does not change between builds: a thread's entry of the next
// window is read as soon as cp is known, so that its trip lies behind the row.
template <int L>
__device__ __forceinline__ void lq_ahead(const BTab<L> &t, const TeamId &id, LQ &q) {
    if constexpr (L != T_LDS)
        q.pre = q.cp + id.tid < q.ns ? (int32_t)t.sq[q.cp + id.tid] : 0;
}

// Sort the queue into its buckets: at a call's start (CREATE: every
// non-member with a link into c enters it, with its rank) or when the fresh
// list has grown long (the pops still pending on it are applied first, as by
// the next scan).  Two passes over the table: count, scatter.
template <bool CREATE, int L>
__device__ __forceinline__ void lq_build(const BTab<L> &t, TeamSh &sh, St &st, const Ctx &c, const TeamId &id,
                                         LQ &q) {
    double hi = -__builtin_huge_val(), lo = __builtin_huge_val();
    st.scanned += 2 * (uint64_t)st.count;
    for (int32_t b = id.tid; b < kBuckets; b += id.nt)
        sh.fill[b] = 0u;
    if constexpr (CREATE) {
        // the ranks' range of the last build, moved by the change of scale
        st.qtop = st.qhi + fmax(st.qalpha - st.alpha, 0.0) * c.logtab[c.logtab_last] + 0.25;
        st.qscale = (double)(kBuckets - 1) /
                    (st.qtop - (st.qlo + fmin(st.qalpha - st.alpha, 0.0) * c.logtab[c.logtab_last]) + 0.25);
    } else {
        fresh_flush(t, sh, st, id);
    }
    __syncthreads();
    if (id.tid == 0)
        sh.row.flen = 0;
    st.flen = 0;
    // tables in global memory: the buckets of a thread's entries, a byte each
    // (kBuckets - 1: not queued), go to the scratch, so that the second pass
    // reads one word for kScanAhead records
    uint32_t *packed = (uint32_t *)t.scr + id.tid;
    for (int32_t base = id.tid; base < st.count; base += kScanAhead * id.nt, packed += id.nt) {
        uint32_t vv[kScanAhead];
        int32_t kk[kScanAhead];
        double rr[kScanAhead];
        uint32_t pk = 0u;
#pragma unroll
        for (int x = 0; x < kScanAhead; ++x) {
            const int32_t i = min(base + x * id.nt, st.count - 1);
            vv[x] = t.DV(i);
            kk[x] = CREATE ? t.KV(i) : L == T_LDS ? t.NODE(i) : 0;
            rr[x] = CREATE ? 0.0 : t.RK(i);
        }
        if constexpr (CREATE) {
#pragma unroll
            for (int x = 0; x < kScanAhead; ++x)
                rr[x] = (vv[x] & kMember) || (vv[x] & kDMask) == 0
                            ? 0.0
                            : block_log(t, c, 2 * (int32_t)(vv[x] & kDMask)) - st.alpha * block_log(t, c, kk[x]);
        }
#pragma unroll
        for (int x = 0; x < kScanAhead; ++x) {
            const int32_t i = base + x * id.nt;
            const uint32_t v = vv[x];
            const double r = rr[x];
            uint32_t nv;
            bool in = false;
            if constexpr (CREATE) {
                in = i < st.count && !(v & kMember) && (v & kDMask) != 0;
                nv = (v & ~(kLive | kFresh | kTouch)) | (in ? kLive : 0u);
                if (in) {
                    if constexpr (L == T_LDS)
                        t.RK(i) = r;
                    else
                        ent_put(t, i, r, nv, -1);
                    hi = fmax(hi, r);
                    lo = fmin(lo, r);
                }
            } else {
                in = i < st.count && (v & kLive) && !(v & kMember);
                if (in && (v & kFresh) && !(v & kTouch))
                    in = !before(r, L == T_LDS ? kk[x] : t.NODE(i), st.pr, st.pu);
                nv = v & ~(kFresh | kTouch | (in ? 0u : kLive));
            }
            const int32_t b = lq_bucket(st, r);
            if (in)
                atomicAdd(&sh.fill[b], 1u);
            if (i < st.count && nv != v && !(CREATE && L != T_LDS && in))
                t.DV(i) = nv;
            pk |= (uint32_t)(in ? b : kBuckets - 1) << (8 * x);
        }
        if constexpr (L != T_LDS)
            *packed = pk;
    }
    if constexpr (CREATE) {
        const double h = wave_max(hi), l = -wave_max(-lo);
        if (id.lane == 0) {
            sh.r[id.wid] = h;
            sh.r2[id.wid] = l;
        }
    }
    __syncthreads();
    bucket_starts(sh, id);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j)
        q.s4[j] = sh.bstart[4 * id.lane + j];
    q.ns = __builtin_amdgcn_readfirstlane(sh.bstart[kBuckets]);
    q.cp = 0;
    if constexpr (L == T_LDS) {
        for (int32_t base = id.tid; base < st.count; base += kScanAhead * id.nt) {
            uint32_t vv[kScanAhead];
            double rr[kScanAhead];
#pragma unroll
            for (int x = 0; x < kScanAhead; ++x) {
                const int32_t i = min(base + x * id.nt, st.count - 1);
                vv[x] = t.DV(i);
                rr[x] = t.RK(i);
            }
#pragma unroll
            for (int x = 0; x < kScanAhead; ++x) {
                const int32_t i = base + x * id.nt;
                if (i < st.count && (vv[x] & (kLive | kMember)) == kLive)
                    t.sq[atomicAdd(&sh.fill[lq_bucket(st, rr[x])], 1u)] = (uint16_t)i;
            }
        }
    } else {
        packed = (uint32_t *)t.scr + id.tid;
        for (int32_t base = id.tid; base < st.count; base += kScanAhead * id.nt, packed += id.nt) {
            const uint32_t pk = *packed;
#pragma unroll
            for (int x = 0; x < kScanAhead; ++x) {
                const uint32_t b = (pk >> (8 * x)) & 255u;
                if (b != kBuckets - 1)
                    t.sq[atomicAdd(&sh.fill[b], 1u)] = (typename BTab<L>::Q)(base + x * id.nt);
            }
        }
    }
    if constexpr (CREATE) {
        double h = sh.r[0], l = sh.r2[0];
        for (int w = 1; w < id.nw; ++w) {
            h = fmax(h, sh.r[w]);
            l = fmin(l, sh.r2[w]);
        }
        st.qhi = h;
        st.qlo = l;
        st.qalpha = st.alpha;
    }
    __syncthreads();
    lq_ahead(t, id, q);
}

// Whether any entry of the queue that a call starts with improves.  Most
// calls add nothing (at least one per scale): for those the queue need not
// be built, only counted.
template <int L>
__device__ __forceinline__ bool any_improves(const BTab<L> &t, TeamSh &sh, St &st, const TeamId &id) {
    bool any = false;
    const bool zero = st.K == 0;
    st.scanned += (uint64_t)st.count;
    for (int32_t base = id.tid; base < st.count; base += kScanAhead * id.nt) {
        uint32_t vv[kScanAhead];
        int32_t kk[kScanAhead];
#pragma unroll
        for (int x = 0; x < kScanAhead; ++x) {
            const int32_t i = min(base + x * id.nt, st.count - 1);
            vv[x] = t.DV(i);
            kk[x] = t.KV(i);
        }
#pragma unroll
        for (int x = 0; x < kScanAhead; ++x) {
            const int32_t d = (int32_t)(vv[x] & kDMask);
            const bool in = base + x * id.nt < st.count && !(vv[x] & kMember) && d != 0;
            st.Rl += in ? 1 : 0;
            st.Gl += in ? 1 : 0;
            int s = zero ? 1 : settle_add(st, d, kk[x]);
            if (in && !any && s < 0)
                s = decide(st.K, st.V, st.K + 2 * (int64_t)d, st.V + kk[x], st.alpha) ? 1 : 0;
            any = any || (in && s > 0);
        }
    }
    if (id.nw == 1)
        return __ballot(any) != 0;
    return team_or(sh, id, any ? 1u : 0u) != 0;
}

// The fresh list's length from which the queue is rebuilt.  A step reads the
// whole list and a rebuild the whole table, so the cost per addition is about
// a count / f + b f, least at f in proportion to the root of count.
template <int L>
__device__ __forceinline__ int32_t fresh_limit(int32_t count) {
    return min(max(kFreshRebuild, (int32_t)(4.0f * sqrtf((float)count))), BTab<L>::FM - 64);
}

// The next addition (false: no queued entry improves): the best improving
// entry of the fresh list and of windows of whole buckets from the queue's
// head.  It is the queue's first improving entry once its bucket lies before
// the window's end (every entry outside ranks strictly below it); until then
// the window holds no improving entry and is popped whole.  What ranks above
// the addition is popped (kLive cleared): queue entries at once, fresh ones by
// the next scan of the list, which drops an entry above the last addition
// (st.pr, st.pu) unless that addition's row re-ranked it (kTouch).
// Both lists are read as one, two entries per thread at a time and without
// branches up to the choice, so that the reads and the chains of dependent
// operations of the two overlap.
constexpr int kStepAhead = 2;

// One candidate of a step: entry e (on: it is queued; ff: on the fresh list).
// True when it has to be written back as v; cand: +1 improves, -1 undecided.
__device__ __forceinline__ bool step_look(const St &st, const Ent &e, bool on, bool ff, bool zero, uint32_t &v,
                                          int &cand) {
    const bool pop = ff && !(e.v & kTouch) && before(e.r, e.u, st.pr, st.pu);
    v = pop ? e.v & ~kLive : e.v & ~kTouch;   // (a popped fresh entry keeps its place)
    const int s = settle_add(st, (int32_t)(e.v & kDMask), e.k);
    cand = on && !pop ? (zero ? 1 : s) : 0;
    return on && v != e.v;
}

__device__ __forceinline__ void step_take(const St &st, const Ent &e, int32_t i, int cand, Ent &b, int32_t &bi) {
    bool take = cand != 0 && before(e.r, e.u, b.r, b.u);
    if (take && cand < 0)
        take = decide(st.K, st.V, st.K + 2 * (int64_t)(e.v & kDMask), st.V + e.k, st.alpha);
    b.r = take ? e.r : b.r;
    b.u = take ? e.u : b.u;
    b.v = take ? e.v : b.v;
    b.k = take ? e.k : b.k;
    b.beg = take ? e.beg : b.beg;
    b.pos = take ? e.pos : b.pos;
    bi = take ? i : bi;
}

template <int L>
__device__ __forceinline__ bool lq_step(const BTab<L> &t, TeamSh &sh, St &st, const TeamId &id, LQ &q, int &par,
                                        Picked &o) {
    // entries in flight per thread: LDS tables two, to overlap the round trips;
    // else one (a window is one entry per thread, and registers are short)
    constexpr int A = L == T_LDS ? kStepAhead : 1;
    Ent b;
    b.r = -__builtin_huge_val();
    b.u = INT32_MAX;
    b.v = 0u;
    b.k = b.beg = 0;
    b.pos = -1;
    int32_t bi = -1;
    const bool zero = st.K == 0;
    int32_t nf = min(st.flen, BTab<L>::FM);   // fresh entries in this window's scan
    int32_t win = id.nt;
    int32_t at = q.cp;    // the window's start; the ones before it hold no improving entry
    for (;;) {
        // buckets b0 (where the window starts) and b1 (its end): the largest
        // that start at or before those positions
        int32_t b0 = -1, b1 = -1;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            b0 += __popcll(__ballot(q.s4[j] <= at));
            b1 += __popcll(__ballot(q.s4[j] <= at + win));
        }
        b0 += q.ns <= at;
        b1 += q.ns <= at + win;
        if (b1 <= b0)
            b1 = min(b0 + 1, kBuckets);
        const int32_t end = lq_start(q, b1);
        const int32_t total = nf + (end - at);
        st.scanned += (uint64_t)total;
        // one: its entries stay in registers for their pops
        bool one;
        Ent ee[A];
        int32_t ii[A];
        bool wi[A];   // queued entries of the window
        uint32_t nv;
        int ok[A];
        if constexpr (L == T_LDS) {
            one = at == q.cp && total <= A * id.nt;
            for (int32_t x0 = 0; x0 < total; x0 += A * id.nt) {
                bool in[A], ff[A];
#pragma unroll
                for (int y = 0; y < A; ++y) {
                    const int32_t x = x0 + y * id.nt + id.tid;
                    in[y] = x < total;
                    ff[y] = x < nf;
                    // the fresh list lies right behind the queue
                    ii[y] = (int32_t)t.sq[in[y] ? (ff[y] ? t.cap + x : at + x - nf) : 0];
                }
#pragma unroll
                for (int y = 0; y < A; ++y) {
                    ii[y] = in[y] ? ii[y] : 0;
                    ee[y] = ent_get(t, ii[y]);
                }
#pragma unroll
                for (int y = 0; y < A; ++y) {
                    const bool on =
                        in[y] && (ee[y].v & (kLive | kFresh | kMember)) == (ff[y] ? kLive | kFresh : kLive);
                    wi[y] = on && !ff[y];
                    if (step_look(st, ee[y], on, ff[y], zero, nv, ok[y]))
                        t.DV(ii[y]) = nv;
                }
#pragma unroll
                for (int y = 0; y < A; ++y)
                    step_take(st, ee[y], ii[y], ok[y], b, bi);
            }
        } else {
            // the window's first entry of each thread is in flight while the
            // fresh list is looked at
            one = at == q.cp && end - at <= A * id.nt;
            bool in[A];
            const auto load = [&](int32_t x0, bool ahead) {
#pragma unroll
                for (int y = 0; y < A; ++y) {
                    const int32_t x = x0 + y * id.nt;
                    in[y] = x < end;
                    ii[y] = ahead && y == 0 ? q.pre : (int32_t)t.sq[in[y] ? x : 0];
                }
#pragma unroll
                for (int y = 0; y < A; ++y) {
                    ii[y] = in[y] ? ii[y] : 0;
                    ee[y] = ent_get(t, ii[y]);
                }
            };
            int32_t x0 = at + id.tid;
            load(x0, at == q.cp);
            for (int32_t f0 = id.tid; f0 < nf; f0 += A * id.nt) {
                Ent g[A];
                int32_t gi[A];
#pragma unroll
                for (int y = 0; y < A; ++y) {
                    const int32_t f = f0 + y * id.nt, p = min(f, BTab<L>::FM - 1);
                    g[y].r = t.fs->r[p];
                    g[y].v = t.fs->v[p];
                    g[y].u = t.fs->u[p];
                    g[y].k = t.fs->k[p];
                    g[y].beg = t.fs->beg[p];
                    g[y].pos = p;
                    gi[y] = f < nf ? t.fs->i[p] : -1;
                }
#pragma unroll
                for (int y = 0; y < A; ++y)
                    if (step_look(st, g[y], gi[y] >= 0 && (g[y].v & kLive), true, zero, nv, ok[y]))
                        t.fs->v[g[y].pos] = nv;
#pragma unroll
                for (int y = 0; y < A; ++y)
                    step_take(st, g[y], gi[y], ok[y], b, bi);
            }
            for (;;) {
#pragma unroll
                for (int y = 0; y < A; ++y) {
                    wi[y] = in[y] && (ee[y].v & (kLive | kFresh | kMember)) == kLive;
                    step_look(st, ee[y], wi[y], false, zero, nv, ok[y]);
                    ee[y].pos = -1;
                }
#pragma unroll
                for (int y = 0; y < A; ++y)
                    step_take(st, ee[y], ii[y], ok[y], b, bi);
                x0 += A * id.nt;
                if (x0 - id.tid >= end)
                    break;
                load(x0, false);
            }
        }
        const bool found = block_pick_max(sh, id, par, b, bi, o);
        const int32_t bo = found ? __builtin_amdgcn_readfirstlane(lq_bucket(st, o.r)) : kBuckets;
        const bool last = end >= q.ns;
        const bool decided = found && (bo < b1 || last);
        if (!decided) {
            // (nothing reads a call's flags once no entry improves)
            if (last)
                return false;
            at = end;
            win = min(win, 1 << 26) * 8;   // (at + win stays below 2^31)
            nf = 0;
            continue;
        }
        // pop what ranks above the addition
        if (one) {
            if (total > 0) {
#pragma unroll
                for (int y = 0; y < A; ++y)
                    if (wi[y] && ii[y] != o.i && before(ee[y].r, ee[y].u, o.r, o.u))
                        t.DV(ii[y]) = ee[y].v & ~kLive;
            }
        } else {
            for (int32_t p = q.cp + id.tid; p < end; p += id.nt) {
                const int32_t i = t.sq[p];
                const uint32_t v = t.DV(i);
                if ((v & (kLive | kFresh | kMember)) == kLive && i != o.i &&
                    before(t.RK(i), t.NODE(i), o.r, o.u))
                    t.DV(i) = v & ~kLive;
            }
        }
        // the buckets before the addition's hold only popped entries
        q.cp = max(q.cp, lq_start(q, bo));
        lq_ahead(t, id, q);
        __syncthreads();   // the pops are in place before the row's updates
        return true;
    }
}

// The smallest removable id above the cursor among the entries i[] (< 0: none).
template <int L, int N>
__device__ __forceinline__ void removal_look(const BTab<L> &t, const St &st, const int32_t *i, int32_t cursor, Ent &b,
                                             int32_t &bi) {
    Ent e[N];
#pragma unroll
    for (int x = 0; x < N; ++x)
        e[x] = ent_get(t, max(i[x], 0));
#pragma unroll
    for (int x = 0; x < N; ++x) {
        if (i[x] < 0 || !(e[x].v & kMember) || e[x].u <= cursor || e[x].u >= b.u)
            continue;
        if (improves_remove(st, (int32_t)(e[x].v & kDMask), e[x].k)) {
            b = e[x];
            bi = i[x];
        }
    }
}

// The members gathered once (t.scr), for the removal passes of a call on
// tables in global memory.  Wide tables of more than by_id_min entries sort
// the list into kBuckets ranges of node id (the queue's bucket arrays are
// free once the additions are over), so that a search for the smallest
// removable id above the cursor walks whole buckets from the cursor's one and
// stops at the first that holds one; smaller tables scan their whole list per
// search, which costs less than the sort and the extra barriers there.
template <int L>
__device__ int32_t removal_list(const BTab<L> &t, TeamSh &sh, St &st, const TeamId &id, bool by_id, int shift) {
    if (!by_id) {
        if (id.tid == 0)
            sh.m = 0;
        __syncthreads();
        for (int32_t i = id.tid; i < st.count; i += id.nt) {
            if (t.DV(i) & kMember)
                t.scr[atomicAdd(&sh.m, 1)] = i;
        }
        __syncthreads();
        st.scanned += (uint64_t)st.count;
        return sh.m;
    }
    for (int32_t b = id.tid; b < kBuckets; b += id.nt)
        sh.fill[b] = 0u;
    __syncthreads();
    for (int32_t i = id.tid; i < st.count; i += id.nt) {
        if (t.DV(i) & kMember)
            atomicAdd(&sh.fill[t.NODE(i) >> shift], 1u);
    }
    __syncthreads();
    bucket_starts(sh, id);
    __syncthreads();
    for (int32_t i = id.tid; i < st.count; i += id.nt) {
        if (t.DV(i) & kMember)
            t.scr[atomicAdd(&sh.fill[t.NODE(i) >> shift], 1u)] = i;
    }
    __syncthreads();
    st.scanned += 2 * (uint64_t)st.count;
    return sh.bstart[kBuckets];
}

// One call of the growth function (Algorithm 1).
template <int L>
__device__ int64_t team_grow(const BTab<L> &t, TeamSh &sh, St &st, const Ctx &c, const TeamId &id, uint32_t k_prune,
                             int32_t by_id_min) {
    int64_t moves = 0;
    int par = 0;
    if (!any_improves(t, sh, st, id))
        return 0;
    LQ q;
    lq_build<true>(t, sh, st, c, id, q);
    for (;;) {
        if (st.flen > fresh_limit<L>(st.count))
            lq_build<false>(t, sh, st, c, id, q);
        Picked o;
        if (!lq_step(t, sh, st, id, q, par, o))
            break;
        if (id.tid == 0) {
            t.DV(o.i) = (o.v | kMember) & ~(kLive | kFresh | kTouch);
            if (L != T_LDS && o.pos >= 0)
                t.fs->i[o.pos] = -1;
            if (st.nadd < kMovedMax)
                sh.moved[st.nadd] = o.i;
        }
        st.nadd += 1;
        st.K += 2 * (int64_t)(o.v & kDMask);
        st.V += o.k;
        st.nmem += 1;
        st.M += 1;
        moves += 1;
        st.pr = o.r;
        st.pu = o.u;
        set_rates(st);
        block_row<ROW_ADD>(t, sh, st, c, id, o.u, o.beg, o.k);
        if (st.ovf)
            return moves;
        if ((int64_t)st.M > st.move_limit) {
            st.err |= ERR_LIMIT;
            return moves;
        }
        if (st.err & ERR_TIMEOUT)
            return moves;
    }
    fresh_flush(t, sh, st, id);
    if (moves == 0)
        return 0;
    // removal passes over the members in ascending id
    const bool by_id = L == T_WIDE && st.count > by_id_min;
    const int shift = max(0, (32 - __builtin_clz((uint32_t)max(c.n - 1, 1))) - 8);
    int32_t ml = 0;
    if constexpr (L != T_LDS)
        ml = removal_list(t, sh, st, id, by_id, shift);
    for (uint32_t pass = 0; k_prune == 0 || pass < k_prune; ++pass) {
        st.Gu += (uint64_t)st.nmem;
        int32_t cursor = -1;
        int32_t bkt = 0;   // by_id: the bucket of the cursor
        bool removed = false;
        for (;;) {
            Ent b;
            b.u = INT32_MAX;
            b.r = 0.0;
            b.v = 0u;
            b.k = b.beg = 0;
            int32_t bi = -1;
            int32_t ii[kScanAhead];
            if constexpr (L == T_LDS) {
                st.scanned += (uint64_t)st.count;
                for (int32_t base = id.tid; base < st.count; base += kScanAhead * id.nt) {
#pragma unroll
                    for (int x = 0; x < kScanAhead; ++x)
                        ii[x] = base + x * id.nt < st.count ? base + x * id.nt : -1;
                    removal_look<L, kScanAhead>(t, st, ii, cursor, b, bi);
                }
            } else {
                int32_t pos = by_id ? sh.bstart[bkt] : 0;
                while (pos < ml) {
                    int32_t end = ml;
                    if (by_id) {
                        const int32_t b0 = bucket_at(sh, 0, kBuckets - 1, pos);
                        const int32_t b1 = bucket_at(sh, b0, kBuckets, pos + kScanAhead * id.nt);
                        end = sh.bstart[max(b1, b0 + 1)];
                    }
                    st.scanned += (uint64_t)(end - pos);
                    for (int32_t base = pos + id.tid; base < end; base += kScanAhead * id.nt) {
#pragma unroll
                        for (int x = 0; x < kScanAhead; ++x)
                            ii[x] = base + x * id.nt < end ? t.scr[base + x * id.nt] : -1;
                        removal_look<L, kScanAhead>(t, st, ii, cursor, b, bi);
                    }
                    if (end >= ml)
                        break;   // the last window: the pick below decides
                    if (team_min_i32(sh, id, bi < 0 ? INT32_MAX : b.u) != INT32_MAX)
                        break;
                    pos = end;
                }
            }
            Picked o;
            if (!block_pick_min(sh, id, par, b, bi, o))
                break;
            if (id.tid == 0)
                t.DV(o.i) = o.v & ~kMember;
            st.nrem += 1;
            st.K -= 2 * (int64_t)(o.v & kDMask);
            st.V -= o.k;
            st.nmem -= 1;
            st.M += 1;
            moves += 1;
            set_rates(st);
            block_row<ROW_REMOVE>(t, sh, st, c, id, o.u, o.beg, o.k);
            removed = true;
            cursor = o.u;
            if (by_id)
                bkt = cursor >> shift;
            if ((int64_t)st.M > st.move_limit) {
                st.err |= ERR_LIMIT;
                return moves;
            }
            if (st.err & ERR_TIMEOUT)
                return moves;
        }
        if (!removed)
            break;
    }
    return moves;
}

// One compare-exchange round of the bitonic network over a[0..m): pair q
// of the round compares positions (i, l); kScanAhead pairs per thread with
// all loads issued first (the pairs of a round are disjoint).
template <typename PairOf>
__device__ __forceinline__ void team_sort_round(int32_t *a, int32_t m, int32_t half_n, const TeamId &id,
                                                PairOf pair_of) {
    for (int32_t q0 = id.tid; q0 < half_n; q0 += kScanAhead * id.nt) {
        int32_t ii[kScanAhead], ll[kScanAhead], xx[kScanAhead], yy[kScanAhead];
#pragma unroll
        for (int x = 0; x < kScanAhead; ++x) {
            const int32_t q = q0 + x * id.nt;
            ii[x] = -1;
            ll[x] = -1;
            if (q < half_n) {
                pair_of(q, ii[x], ll[x]);
                if (ll[x] >= m)
                    ii[x] = -1;
            }
            xx[x] = 0;
            yy[x] = 0;
            if (ii[x] >= 0) {
                xx[x] = a[ii[x]];
                yy[x] = a[ll[x]];
            }
        }
#pragma unroll
        for (int x = 0; x < kScanAhead; ++x) {
            if (ii[x] >= 0 && xx[x] > yy[x]) {
                a[ii[x]] = yy[x];
                a[ll[x]] = xx[x];
            }
        }
    }
    __syncthreads();
}

// Ascending sort of a[0..m) by the workgroup (same network as wave_sort).
__device__ void team_sort(int32_t *a, int32_t m, const TeamId &id) {
    int32_t P = 1;
    while (P < m)
        P <<= 1;
    const int32_t half_n = P >> 1;
    for (int32_t k = 2; k <= P; k <<= 1) {
        const int32_t hk = k >> 1;
        team_sort_round(a, m, half_n, id, [=](int32_t q, int32_t &i, int32_t &l) {
            const int32_t blk = q / hk;
            const int32_t off = q - blk * hk;
            i = blk * k + off;
            l = blk * k + k - 1 - off;
        });
        for (int32_t j = k >> 2; j >= 1; j >>= 1) {
            team_sort_round(a, m, half_n, id, [=](int32_t q, int32_t &i, int32_t &l) {
                i = (q / j) * 2 * j + (q % j);
                l = i + j;
            });
        }
    }
}

// Delta output, one workgroup: wave_toggle_records for the workgroup.
template <class T>
__device__ bool team_toggle_records(const SweepArgs &A, const T &t, TeamSh &sh, St &st, const Ctx &c,
                                    const TeamId &id, int32_t set, int32_t s_last) {
    const int32_t sk = delta_key_scale(A.rec, A.S, set, s_last);
    if (sk < 0) {
        st.err |= ERR_MISSING;
        return true;
    }
    for (int32_t s = sk; s <= s_last; ++s) {
        const int64_t r = (int64_t)set * A.S + s;
        const int64_t off = A.rec.off[r];
        const int32_t len = record_len(A.rec, r);
        if (off < 0 || len < 0 || off + len > A.pool_cap)
            return false;
        for (int32_t base = 0; base < len; base += id.nt) {
            const bool act = base + id.tid < len;
            const int32_t u = act ? A.pool[off + base + id.tid] : 0;
            const int32_t idx = team_ensure(t, sh, st, c, id, act, u);
            if (sh.row.ovf) {
                st.ovf = true;
                return true;
            }
            if (act && idx >= 0)
                t.DV(idx) ^= (kMember | kWas);
            st.count = min(sh.row.count, t.cap);
            __syncthreads();
        }
    }
    return true;
}

// Sort a[0..m) (global memory) through the LDS buffer lbuf when it fits:
// the bitonic network's rounds then wait on LDS, not on memory.
constexpr int kLdsSort = (int)(sizeof(FreshSh<kFreshMax>) / 4);

__device__ void team_sort_via(int32_t *a, int32_t m, const TeamId &id, int32_t *lbuf) {
    if (m <= 1)
        return;
    if (!lbuf || m > kLdsSort) {
        team_sort(a, m, id);
        return;
    }
    for (int32_t i = id.tid; i < m; i += id.nt)
        lbuf[i] = a[i];
    __syncthreads();
    team_sort(lbuf, m, id);
    for (int32_t i = id.tid; i < m; i += id.nt)
        a[i] = lbuf[i];
    __syncthreads();
}

// The ids added at a scale that removed none, ascending, in sh.resv[0 .. na)
// (na = st.nadd <= kMovedMax): by counting the smaller ones.  Delta output:
// their entries are marked as emitted.
template <class T>
__device__ void moved_ids(const T &t, TeamSh &sh, const TeamId &id, int32_t na, bool mark) {
    const int32_t i = id.tid < na ? sh.moved[id.tid] : 0;
    const int32_t j = id.tid + id.nt < na ? sh.moved[id.tid + id.nt] : 0;   // (na <= 2 * 64)
    const int32_t u = t.NODE(i), w = t.NODE(j);
    __syncthreads();
    if (id.tid < na) {
        sh.moved[id.tid] = u;
        if (mark)
            t.DV(i) |= kWas;
    }
    if (id.tid + id.nt < na) {
        sh.moved[id.tid + id.nt] = w;
        if (mark)
            t.DV(j) |= kWas;
    }
    __syncthreads();
    int32_t ru = 0, rw = 0;
    for (int32_t q = 0; q < na; ++q) {
        const int32_t x = sh.moved[q];
        ru += x < u;
        rw += x < w;
    }
    if (id.tid < na)
        sh.resv[ru] = u;
    if (id.tid + id.nt < na)
        sh.resv[rw] = w;
    __syncthreads();
}

// How many of the ascending a[0 .. n) are below x (n <= 2^8 - 1).
__device__ __forceinline__ int32_t lower_count(const int32_t *a, int32_t n, int32_t x) {
    int32_t lo = 0;
#pragma unroll
    for (int step = 128; step >= 1; step >>= 1)
        if (lo + step <= n && a[lo + step - 1] < x)
            lo += step;
    return lo;
}

// Merge the ascending list from[0 .. n) with the ascending ids sh.resv[0 .. na),
// none in common, into to[0 .. n + na).
__device__ void merge_moved(TeamSh &sh, const TeamId &id, const int32_t *from, int32_t n, int32_t na, int32_t *to) {
    for (int32_t i = id.tid; i < n; i += id.nt) {
        const int32_t x = from[i], y = i > 0 ? from[i - 1] : -1;
        const int32_t a = i > 0 ? lower_count(sh.resv, na, y) : 0, b = lower_count(sh.resv, na, x);
        to[i + b] = x;
        for (int32_t q = a; q < b; ++q)   // the ids between y and x
            to[i + q] = sh.resv[q];
        if (i == n - 1)
            for (int32_t q = b; q < na; ++q)
                to[n + q] = sh.resv[q];
    }
}

// lbuf: LDS sort buffer of kLdsSort entries, or nullptr (tables in LDS sort in place).
template <bool PERSET, class T>
__device__ void run_team(const SweepArgs &A, const T &t, TeamSh &sh, int32_t *lbuf) {
    TeamId id;
    id.tid = (int)threadIdx.x;
    id.nt = (int)blockDim.x;
    id.lane = id.tid & 63;
    id.wid = id.tid >> 6;
    id.nw = id.nt >> 6;
    const Ctx c = make_ctx(A.g);
    const uint32_t n_items = A.tier == 0 ? (uint32_t)A.n_sets : A.ctl->ovf_count[A.in_from];
    for (;;) {
        __syncthreads();
        if (id.tid == 0) {
            sh.item = atomicAdd(&A.ctl->work_next[A.tier], 1u);
            sh.abort = __hip_atomic_load(A.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & ERR_TIMEOUT;
            sh.row.count = 0;
            sh.row.ovf = 0u;
            sh.row.stop = 0u;
        }
        team_reset(t, id);
        __syncthreads();
        const uint32_t item = sh.item;
        if (item >= n_items || sh.abort)
            break;
        // a later tier's item is set * S + s (see run_wave)
        const uint32_t wi = A.tier == 0 ? item : (uint32_t)A.work_in[item];
        const int32_t set = A.tier == 0 ? (int32_t)item : (int32_t)(wi / (uint32_t)A.S);
        const int32_t s0 = A.tier == 0 ? A.s_begin : (int32_t)(wi % (uint32_t)A.S);

        St st;
        st.count = 0;
        st.nmem = 0;
        st.K = 0;
        st.V = 0;
        st.rK2 = st.rV = 0.0;
        st.alpha = 0.0;
        st.pr = 0.0;
        st.pu = 0;
        st.Gl = st.Rl = 0;
        st.Gu = 0;
        st.M = 0;
        st.ovf = false;
        st.err = 0;
        st.move_limit = 8 * (int64_t)A.g.n + 65536;
        st.t0 = wall_clock64();
        st.budget = (uint64_t)A.budget_ticks;
        st.rows = st.row_len = st.inserted = st.written = st.scanned = 0;
        st.mrows = st.mrow_len = st.c_mrows = st.c_mrow_len = st.ins_mark = st.c_ins = 0;
        st.srows = st.srow_len = 0;
        st.emitted = false;

        const int32_t *init = nullptr;
        int32_t n_init = 0;
        bool bad = false;
        bool keyed = false;   // delta output (see run_wave)
        if ((s0 > A.s_begin || A.resume) && A.rec.drem) {
            bad = !team_toggle_records(A, t, sh, st, c, id, set, s0 - 1);
            st.err = team_or(sh, id, st.err);
            if (!bad && !st.ovf && !st.err) {
                if (id.tid == 0)
                    sh.m = 0;
                __syncthreads();
                for (int32_t i = id.tid; i < st.count; i += id.nt) {
                    if (t.DV(i) & kMember)
                        t.scr[atomicAdd(&sh.m, 1)] = t.NODE(i);
                }
                __syncthreads();
                init = t.scr;
                n_init = sh.m;
                keyed = true;
            }
        } else if (s0 > A.s_begin || A.resume) {
            const int64_t r = (int64_t)set * A.S + (s0 - 1);
            const int64_t off = A.rec.off[r];
            n_init = A.rec.cnt[r];
            if (off < 0 || off + n_init > A.pool_cap)
                bad = true;
            else
                init = A.pool + off;
        } else {
            init = A.seed_nodes + A.seed_ptr[set];
            n_init = A.seed_ptr[set + 1] - A.seed_ptr[set];
        }
        if (!bad && !st.ovf)
            team_init(t, sh, st, c, id, init, n_init);
        st.err = team_or(sh, id, st.err);
        // seed-set gathers are the method's; a resumed set's are overhead
        if (!(s0 > A.s_begin || A.resume)) {
            st.srows = st.rows;
            st.srow_len = st.row_len;
        } else {
            st.ins_mark = st.inserted;
        }

        int64_t last_off = -1;
        int32_t last_cnt = 0;
        bool listed = false;   // pool[last_off ..) holds the members at the last emission, ascending
        int32_t s_at = s0;   // the scale being grown (where an overflow happened)
        for (int32_t s = s0; s < A.s_end && !st.ovf && !bad && !st.err; ++s) {
            s_at = s;
            if constexpr (PERSET)
                st.alpha = A.alpha_set[set];
            else
                st.alpha = A.scales[s];
            set_rates(st);
            st.Gl = st.Rl = 0;
            st.Gu = 0;
            st.M = 0;
            uint64_t calls = 0;
            int64_t moved = 0;
            st.nadd = st.nrem = 0;
            for (;;) {
                calls += 1;
                const int64_t mv = team_grow(t, sh, st, c, id, A.k_prune, A.by_id_min);
                st.err = team_or(sh, id, st.err);
                moved += mv;
                if (st.ovf || st.err || mv == 0)
                    break;
                if (A.max_calls != 0 && calls >= (uint64_t)A.max_calls)
                    break;
                if ((int64_t)calls > st.move_limit) {
                    st.err |= ERR_LIMIT;
                    break;
                }
                if (team_over_budget(sh, id, st))
                    break;
            }
            if (st.ovf || st.err)
                break;
            const int64_t r = (int64_t)set * A.S + s;
            const uint64_t G = team_sum(sh, id, (uint64_t)st.Gl) + st.Gu;
            const uint64_t R = team_sum(sh, id, (uint64_t)st.Rl);
            int32_t dadd = 0, drem = 0;
            if ((s == s0 || moved > 0) && keyed) {
                // delta output (see run_wave)
                const bool few = s > s0 && st.nrem == 0 && st.nadd <= kMovedMax;
                if (id.tid == 0) {
                    sh.m = few ? st.nadd : 0;
                    sh.m2 = 0;
                }
                __syncthreads();
                if (few)
                    moved_ids(t, sh, id, st.nadd, true);
                else for (int32_t i = id.tid; i < st.count; i += id.nt) {
                    const uint32_t v = t.DV(i);
                    const bool add = (v & kMember) && !(v & kWas);
                    const bool rem = (v & kWas) && !(v & kMember);
                    if (add)
                        t.scr[atomicAdd(&sh.m, 1)] = t.NODE(i);
                    if (rem)
                        t.scr[t.cap - 1 - atomicAdd(&sh.m2, 1)] = t.NODE(i);
                    if (add || rem)
                        t.DV(i) = v ^ kWas;
                }
                __syncthreads();
                const int32_t na = sh.m, nr = sh.m2;
                if (!few)
                    team_sort_via(t.scr, na, id, lbuf);
                team_sort_via(t.scr + (t.cap - nr), nr, id, lbuf);
                if (id.tid == 0)
                    sh.off = atomicAdd(A.pool_cursor, (unsigned long long)(na + nr));
                __syncthreads();
                const unsigned long long off = sh.off;
                if ((int64_t)off + na + nr <= A.pool_cap) {
                    for (int32_t i = id.tid; i < na; i += id.nt)
                        A.pool[off + i] = few ? sh.resv[i] : t.scr[i];
                    for (int32_t i = id.tid; i < nr; i += id.nt)
                        A.pool[off + na + i] = t.scr[t.cap - nr + i];
                }
                last_off = (int64_t)off;
                last_cnt = st.nmem;
                dadd = na;
                drem = nr;
                st.written += (uint64_t)(na + nr);
                __syncthreads();
            } else if (moved > 0 && listed && last_cnt > 0 && st.nrem == 0 && st.nadd <= kMovedMax && !A.rec.drem) {
                // the last list and the ids added since
                const int32_t na = st.nadd, m = last_cnt + na;
                moved_ids(t, sh, id, na, false);
                if (id.tid == 0)
                    sh.off = atomicAdd(A.pool_cursor, (unsigned long long)m);
                __syncthreads();
                const unsigned long long off = sh.off;
                listed = (int64_t)off + m <= A.pool_cap;
                if (listed)
                    merge_moved(sh, id, A.pool + last_off, last_cnt, na, A.pool + off);
                last_off = (int64_t)off;
                last_cnt = m;
                st.written += (uint64_t)m;
                __syncthreads();
            } else if (s == s0 || moved > 0) {
                if (id.tid == 0)
                    sh.m = 0;
                __syncthreads();
                for (int32_t i = id.tid; i < st.count; i += id.nt) {
                    const uint32_t v = t.DV(i);
                    const bool ism = v & kMember;
                    if (ism) {
                        const int32_t p = atomicAdd(&sh.m, 1);
                        t.scr[p] = t.NODE(i);
                    }
                    if (A.rec.drem && ism != (bool)(v & kWas))
                        t.DV(i) = v ^ kWas;
                }
                __syncthreads();
                const int32_t m = sh.m;
                team_sort_via(t.scr, m, id, lbuf);
                if (id.tid == 0)
                    sh.off = atomicAdd(A.pool_cursor, (unsigned long long)m);
                __syncthreads();
                const unsigned long long off = sh.off;
                if ((int64_t)off + m <= A.pool_cap) {
                    for (int32_t i = id.tid; i < m; i += id.nt)
                        A.pool[off + i] = t.scr[i];
                }
                listed = (int64_t)off + m <= A.pool_cap;
                last_off = (int64_t)off;
                last_cnt = m;
                dadd = m;
                drem = -1;
                keyed = A.rec.drem != nullptr;
                st.written += (uint64_t)m;
                __syncthreads();
            } else if (keyed) {
                last_cnt = st.nmem;
            }
            if (id.tid == 0) {
                A.rec.off[r] = last_off;
                A.rec.cnt[r] = last_cnt;
                if (A.rec.drem) {
                    A.rec.dadd[r] = dadd;
                    A.rec.drem[r] = drem;
                }
                A.rec.K[r] = st.K;
                A.rec.V[r] = st.V;
                A.rec.f[r] = st.K == 0 ? 0.0 : (double)st.K / pow((double)st.V, st.alpha);
                A.rec.ctr[4 * r + 0] = G;
                A.rec.ctr[4 * r + 1] = R;
                A.rec.ctr[4 * r + 2] = st.M;
                A.rec.ctr[4 * r + 3] = calls;
            }
            if constexpr (PERSET) {
                // see run_wave: every thread's stores, then the flag
                if (A.done_flags) {
                    __threadfence_system();
                    __syncthreads();
                    if (id.tid == 0)
                        __hip_atomic_store(&A.done_flags[set], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                }
            }
            st.c_mrows = st.mrows;
            st.c_mrow_len = st.mrow_len;
            st.c_ins = st.inserted - st.ins_mark;
            st.emitted = true;
        }
        const uint64_t inserted = team_sum(sh, id, st.inserted);
        const uint64_t cins = team_sum(sh, id, st.c_ins);
        if (id.tid == 0) {
            if (bad || st.err || (st.ovf && !A.work_out))
                void_records(A, set, s_at);
            if (st.ovf) {
                if (A.work_out) {
                    const uint32_t pos = atomicAdd(&A.ctl->ovf_count[A.tier], 1u);
                    A.work_out[pos] = set * A.S + s_at;
                } else {
                    atomicOr(A.err, ERR_CAPACITY);
                }
            }
            if (st.err)
                atomicOr(A.err, st.err);
            if (!st.ovf) {
                unsigned long long *sx = A.stat + kStatWords * A.tier;
                atomicAdd(&sx[0], (unsigned long long)st.rows);
                atomicAdd(&sx[1], (unsigned long long)st.row_len);
                atomicAdd(&sx[2], (unsigned long long)inserted);
                atomicAdd(&sx[3], (unsigned long long)st.written);
                atomicAdd(&sx[4], 1ull);
                atomicAdd(&sx[5], (unsigned long long)st.scanned);
            }
            unsigned long long *sa = A.stat + kStatWords * A.tier;
            atomicAdd(&sa[6], (unsigned long long)st.c_mrows);
            atomicAdd(&sa[7], (unsigned long long)st.c_mrow_len);
            if (st.emitted) {
                atomicAdd(&sa[8], (unsigned long long)st.srows);
                atomicAdd(&sa[9], (unsigned long long)st.srow_len);
            }
            atomicAdd(&sa[10], (unsigned long long)cins);
        }
        team_leave(t, sh, id);
    }
}

// Fill a workgroup's copy of the first logs (run_team starts with a barrier).
__device__ __forceinline__ void load_logs(const SweepArgs &A, double *lt) {
    for (int32_t i = (int32_t)threadIdx.x; i < min(kBlockLogs, A.g.logtab_n); i += (int32_t)blockDim.x)
        lt[i] = A.g.logtab[i];
}

template <bool PERSET, int L>
__device__ __forceinline__ void team_entry(const SweepArgs &A) {
    __shared__ TeamSh sh;
    double *lt;
    if constexpr (L == T_LDS) {
        extern __shared__ __align__(16) char smem[];
        lt = (double *)smem;
        const BTab<L> t = carve_lds(smem, A.cap, A.hbits);
        load_logs(A, lt);
        run_team<PERSET>(A, t, sh, nullptr);
    } else {
        __shared__ double logs[kBlockLogs];
        __shared__ typename BTab<L>::F fresh;   // between growth calls: sort buffer
        if ((int)blockIdx.x >= A.n_slots)
            return;
        const BTab<L> t = carve_slab<L>(A.gtab, A.gtab_stride, A.n_slots, blockIdx.x, logs, &fresh, A.cap,
                                        A.hbits);
        load_logs(A, logs);
        run_team<PERSET>(A, t, sh, (int32_t *)&fresh);
    }
}

// Register bounds.  LDS tables leave room for a few workgroups per compute
// unit, so their kernel takes the 256 VGPRs of two waves per SIMD and spills
// nothing.  On global tables three waves per SIMD (168 VGPRs, 100 spilled)
// are best: sweeps of the 100k-, 1M- and 4M-node graphs 19.6, 107 and 373 ms
// at the same waves per community; two (no spills) 22.9, 124 and 428, four
// 21.3, 113 and 407.
#define LCD_TEAM_KERNEL(w) __global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(w)))
LCD_TEAM_KERNEL(2) sweep_team_lds_kernel(SweepArgs A) { team_entry<false, T_LDS>(A); }
LCD_TEAM_KERNEL(3) sweep_team_global_kernel(SweepArgs A) { team_entry<false, T_PACK>(A); }
LCD_TEAM_KERNEL(3) sweep_team_global_rec_kernel(SweepArgs A) { team_entry<false, T_WIDE>(A); }
LCD_TEAM_KERNEL(2) query_team_lds_kernel(SweepArgs A) { team_entry<true, T_LDS>(A); }
LCD_TEAM_KERNEL(3) query_team_global_kernel(SweepArgs A) { team_entry<true, T_PACK>(A); }
LCD_TEAM_KERNEL(3) query_team_global_rec_kernel(SweepArgs A) { team_entry<true, T_WIDE>(A); }
#undef LCD_TEAM_KERNEL

// ---------------------------------------------------------------------------
// Graph preparation
// ---------------------------------------------------------------------------
// Weighted degrees, their largest and their sum (64 bits; a degree past 2^31
// is refused by its largest).
__global__ void __launch_bounds__(256) degrees_kernel(const int32_t *row_ptr, const uint8_t *w, int32_t *kdeg, int32_t n,
                                                      GraphCheck *chk) {
    uint64_t most = 0, sum = 0;
    for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < n; u += (int64_t)gridDim.x * blockDim.x) {
        const int32_t b = row_ptr[u], e = row_ptr[u + 1];
        uint64_t k = (uint64_t)(e - b);
        if (w) {
            k = 0;
            for (int32_t j = b; j < e; ++j)
                k += w[j];
        }
        kdeg[u] = (int32_t)k;
        most = k > most ? k : most;
        sum += k;
    }
    for (int off = 32; off >= 1; off >>= 1) {
        const uint64_t x = __shfl_xor(most, off);
        most = x > most ? x : most;
        sum += __shfl_xor(sum, off);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicMax((unsigned long long *)&chk->maxk, (unsigned long long)most);
        atomicAdd((unsigned long long *)&chk->volume, (unsigned long long)sum);
    }
}

// The first directed entry that breaks a rule of the input (chk->bad: entry
// << 3 | rule): id in range, no self-loop, rows strictly ascending, weights
// at least 1, a reverse entry of the same weight.  Bound by the dependent
// reads of two binary searches an entry, independent between entries: 40 us
// for 60,000 nodes, 0.75 ms for 1,000,000 of mean degree 18 (the upload of a
// 10,000,000-node graph, checked by host threads, took 4.7 s; now 0.7).
__global__ void __launch_bounds__(256) check_graph_kernel(const int32_t *row_ptr, const int32_t *col, const uint8_t *w,
                                                          int32_t n, int64_t nnz, GraphCheck *chk) {
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < nnz; j += (int64_t)gridDim.x * blockDim.x) {
        // the row: the last u with row_ptr[u] <= j
        int32_t lo = 0, len = n;
        while (len > 0) {
            const int32_t half = len >> 1;
            if ((int64_t)row_ptr[lo + half + 1] <= j) {
                lo += half + 1;
                len -= half + 1;
            } else {
                len = half;
            }
        }
        const int32_t u = lo, v = col[j];
        uint64_t rule = 0;
        if (v < 0 || v >= n)
            rule = 1;
        else if (v == u)
            rule = 2;
        else if (j > row_ptr[u] && col[j - 1] >= v)
            rule = 3;
        else if (w && w[j] < 1)
            rule = 4;
        else {
            int64_t at = row_ptr[v];
            const int64_t end = row_ptr[v + 1];
            int64_t m = end - at;
            while (m > 0) {
                const int64_t half = m >> 1;
                if (col[at + half] < u) {
                    at += half + 1;
                    m -= half + 1;
                } else {
                    m = half;
                }
            }
            if (at == end || col[at] != u)
                rule = 5;
            else if (w && w[at] != w[j])
                rule = 6;
        }
        if (rule)
            atomicMin((unsigned long long *)&chk->bad, (unsigned long long)((uint64_t)j << 3 | rule));
    }
}

__global__ void node_info_kernel(const int32_t *row_ptr, const int32_t *kdeg, int2 *info, int32_t n) {
    for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < n; u += (int64_t)gridDim.x * blockDim.x)
        info[u] = make_int2(row_ptr[u], kdeg[u]);
}

__global__ void adj_kernel(const int32_t *row_ptr, const int32_t *col, const uint8_t *w, const int32_t *kdeg,
                           const double *logtab, int64_t nnz, int4 *adj, double *adjl) {
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < nnz;
         j += (int64_t)gridDim.x * blockDim.x) {
        const int32_t u = col[j];
        const int32_t k = kdeg[u];
        adj[j] = make_int4(u, k, row_ptr[u], w ? (int32_t)w[j] : 1);
        adjl[j] = logtab[k];
    }
}

__global__ void logtab_kernel(double *tab, int32_t m) {
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= m)
        return;
    tab[x] = x == 0 ? 0.0 : ilog((uint64_t)x);
}

__global__ void log_kernel(const uint64_t *x, double *out, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const uint64_t v = x[i];
    out[i] = v == 0 ? 0.0 : ilog(v);
}

__global__ void fill_i32_kernel(int32_t *p, int32_t v, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// ---------------------------------------------------------------------------
// Readout
// ---------------------------------------------------------------------------

// Exclusive scan of the member counts of one scale; the exact int64 total goes
// to *total, so the host can refuse a scale whose int32 offsets would wrap
// before it sizes or gathers anything.  The counts lie S apart, a cache line
// or more each: workgroup b sums all before its chunk by itself, with every
// read independent, instead of waiting for the others (20,000 sets, 32
// scales: one workgroup took 46 us a scale, 20 take 19, the misses of the
// counts' lines; scanning by wave shuffles instead of LDS steps changed nothing).
__global__ void __launch_bounds__(1024) scale_scan_kernel(const int32_t *cnt, int32_t S, int32_t s,
                                                          int32_t n_sets, int32_t chunk, int32_t *comm_ptr,
                                                          long long *total) {
    __shared__ int64_t part[1024];
    __shared__ int64_t before;
    const int tid = threadIdx.x;
    const int64_t lo = min((int64_t)blockIdx.x * chunk, (int64_t)n_sets), hi = min(lo + chunk, (int64_t)n_sets);
    int64_t sum = 0;
    for (int64_t j = tid; j < lo; j += 4096) {
        int32_t x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            x[q] = j + 1024 * q < lo ? cnt[(j + 1024 * q) * S + s] : 0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            sum += x[q];
    }
    part[tid] = sum;
    __syncthreads();
    for (int off = 512; off >= 1; off >>= 1) {
        if (tid < off)
            part[tid] += part[tid + off];
        __syncthreads();
    }
    if (tid == 0)
        before = part[0];
    __syncthreads();
    int64_t base = before;
    for (int64_t j0 = lo; j0 < hi; j0 += 1024) {
        const int64_t j = j0 + tid;
        const int64_t x = j < hi ? cnt[j * S + s] : 0;
        part[tid] = x;
        __syncthreads();
        for (int off = 1; off < 1024; off <<= 1) {
            const int64_t v = tid >= off ? part[tid - off] : 0;
            __syncthreads();
            part[tid] += v;
            __syncthreads();
        }
        if (j < hi)
            comm_ptr[j] = (int32_t)(base + part[tid] - x);
        base += part[1023];
        __syncthreads();
    }
    if (hi == n_sets && lo < n_sets + (n_sets == 0) && tid == 0) {
        comm_ptr[n_sets] = (int32_t)base;
        *total = (long long)base;
    }
}

__global__ void __launch_bounds__(256) scale_gather_kernel(Records rec, const int32_t *pool,
                                                           const double *scales, int32_t S,
                                                           int32_t s, int32_t n_sets,
                                                           const int32_t *comm_ptr, int32_t *members,
                                                           int64_t *k_in, int64_t *vol, double *f) {
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int64_t j = (int64_t)blockIdx.x * (blockDim.x >> 6) + wave;
    if (j >= n_sets)
        return;
    const int64_t r = j * S + s;
    const int64_t off = rec.off[r];
    const int32_t m = rec.cnt[r];
    const int32_t dst = comm_ptr[j];
    if (members)
        for (int32_t i = lane; i < m; i += 64)
            members[dst + i] = pool[off + i];
    if (lane == 0) {
        if (k_in)
            k_in[j] = rec.K[r];
        if (vol)
            vol[j] = rec.V[r];
        if (f)
            f[j] = rec.f[r];
    }
}

// Delta output readout.  The members of scale s of a set are the ids that
// occur an odd number of times among the ids of its records from its last
// full list at or before s through s (every id alternately joins and
// leaves).  sets: listed set ids (nullptr: set q for q < n).

// Per listed set: ids in those records (ev[q]); a set with no full list
// before s sets bit 1 of *err.
__global__ void delta_events_kernel(Records rec, int32_t S, int32_t s, const int32_t *sets, int32_t n,
                                    int64_t *ev, uint32_t *err) {
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n;
         q += (int64_t)gridDim.x * blockDim.x) {
        const int32_t set = sets ? sets[q] : (int32_t)q;
        const int32_t sk = delta_key_scale(rec, S, set, s);
        int64_t e = 0;
        if (sk < 0)
            atomicOr(err, 1u);
        else
            for (int32_t x = sk; x <= s; ++x)
                e += record_len(rec, (int64_t)set * S + x);
        ev[q] = e;
    }
}

// Exclusive prefix sums of x[0..n) into out[0..n] (one block).
__global__ void __launch_bounds__(1024) scan_i64_kernel(const int64_t *x, int64_t n, int64_t *out) {
    __shared__ int64_t part[1024];
    const int tid = threadIdx.x;
    const int64_t per = (n + 1023) / 1024;
    const int64_t lo = tid * per;
    const int64_t hi = lo + per < n ? lo + per : n;
    int64_t sum = 0;
    for (int64_t j = lo; j < hi; ++j)
        sum += x[j];
    part[tid] = sum;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int64_t v = tid >= off ? part[tid - off] : 0;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    int64_t run = part[tid] - sum;
    for (int64_t j = lo; j < hi; ++j) {
        const int64_t v = x[j];
        out[j] = run;
        run += v;
    }
    if (tid == 1023)
        out[n] = part[1023];
}

// One workgroup per listed set: its records' ids into scratch[ev_off[q]..),
// sorted, then the ids of odd multiplicity, in order, to
// members[out_ptr[q]..).  A count other than the record's sets bit 2 of
// *err.
__global__ void __launch_bounds__(256) delta_rebuild_kernel(Records rec, const int32_t *pool, int32_t S,
                                                            int32_t s, const int32_t *sets, int32_t n,
                                                            const int64_t *ev_off, int32_t *scratch,
                                                            const int32_t *out_ptr, int32_t *members,
                                                            uint32_t *err) {
    TeamId id;
    id.tid = (int)threadIdx.x;
    id.nt = (int)blockDim.x;
    id.lane = id.tid & 63;
    id.wid = id.tid >> 6;
    id.nw = id.nt >> 6;
    __shared__ int32_t wcount[kTeamMaxWaves];
    for (int64_t q = blockIdx.x; q < n; q += gridDim.x) {
        const int32_t set = sets ? sets[q] : (int32_t)q;
        const int32_t sk = delta_key_scale(rec, S, set, s);
        if (sk < 0)
            continue;   // reported by delta_events_kernel
        int32_t *a = scratch + ev_off[q];
        int64_t pos = 0;
        for (int32_t x = sk; x <= s; ++x) {
            const int64_t r = (int64_t)set * S + x;
            const int64_t off = rec.off[r];
            const int32_t len = record_len(rec, r);
            for (int32_t i = id.tid; i < len; i += id.nt)
                a[pos + i] = pool[off + i];
            pos += len;
        }
        const int32_t E = (int32_t)pos;
        __syncthreads();
        team_sort(a, E, id);
        int32_t outn = 0;
        const int32_t dst = out_ptr[q];
        for (int32_t base = 0; base < E; base += id.nt) {
            const int32_t p = base + id.tid;
            bool keep = false;
            if (p < E && (p == 0 || a[p - 1] != a[p])) {
                int32_t L = 1;
                while (p + L < E && a[p + L] == a[p])
                    ++L;
                keep = (L & 1) != 0;
            }
            const uint64_t bm = __ballot(keep);
            if (id.lane == 0)
                wcount[id.wid] = __popcll(bm);
            __syncthreads();
            int32_t before_w = 0, total = 0;
            for (int w = 0; w < id.nw; ++w) {
                if (w < id.wid)
                    before_w += wcount[w];
                total += wcount[w];
            }
            if (keep)
                members[dst + outn + before_w + __popcll(bm & lanes_below(id.lane))] = a[p];
            outn += total;
            __syncthreads();
        }
        if (id.tid == 0 && outn != rec.cnt[(int64_t)set * S + s])
            atomicOr(err, 2u);
        __syncthreads();
    }
}

// Per set: the ids added and removed at scale s (a full list counts as
// added), their counts first.
__global__ void delta_counts_kernel(Records rec, int32_t S, int32_t s, int32_t n, int64_t *na, int64_t *nr) {
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = j * S + s;
        const bool full = rec.drem[r] < 0;
        na[j] = full ? rec.cnt[r] : rec.dadd[r];
        nr[j] = full ? 0 : rec.drem[r];
    }
}

__global__ void __launch_bounds__(256) delta_gather_kernel(Records rec, const int32_t *pool, int32_t S,
                                                           int32_t s, int32_t n, const int64_t *add_off,
                                                           int32_t *added, const int64_t *rem_off,
                                                           int32_t *removed) {
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int64_t j = (int64_t)blockIdx.x * (blockDim.x >> 6) + wave;
    if (j >= n)
        return;
    const int64_t r = j * S + s;
    const int64_t off = rec.off[r];
    const int32_t a = (int32_t)(add_off[j + 1] - add_off[j]);
    const int32_t m = (int32_t)(rem_off[j + 1] - rem_off[j]);
    if (added)
        for (int32_t i = lane; i < a; i += 64)
            added[add_off[j] + i] = pool[off + i];
    if (removed)
        for (int32_t i = lane; i < m; i += 64)
            removed[rem_off[j] + i] = pool[off + a + i];
}

__global__ void overlap_count_kernel(const int32_t *members, int64_t total, int32_t *cnt) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x)
        atomicAdd(&cnt[members[i]], 1);
}

// ---------------------------------------------------------------------------
// Seed selection (Sec. 3, initialisation of Algorithm 2) in parallel rounds.
// Candidate nodes (at least two neighbours) are visited in the order perm;
// the sequential rule keeps a node that is still a candidate and drops its
// neighbours (rule 1) or everything within two hops (rule 2).  That set is
// the first independent set in visiting order of the conflict graph (two
// candidates conflict within 1 or 2 hops), which rounds of "an undecided
// candidate joins when it comes first among the undecided candidates it
// conflicts with" produce exactly (Blelloch, Fineman and Shun, SPAA 2012).
// st: 0 undecided candidate, 1 seed, 2 not a seed.
// ---------------------------------------------------------------------------

// Positions of the nodes in perm (pos: INT32_MAX before), the first entry out
// of range or that a later pass finds repeated in *bad.
__global__ void seed_perm_kernel(const int32_t *perm, int32_t n, int32_t *pos, unsigned *bad) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = perm[i];
        if (v < 0 || v >= n)
            atomicMin(bad, (unsigned)i);
        else
            atomicMin(&pos[v], (int32_t)i);
    }
}

// key[v]: the position of an undecided candidate, INT32_MAX of any other node.
__global__ void seed_init_kernel(const int32_t *row_ptr, const int32_t *perm, int32_t n, const int32_t *pos,
                                 uint8_t *st, uint8_t *act, int32_t *key, unsigned *bad) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = perm[i];
        if (v >= 0 && v < n && pos[v] != (int32_t)i)
            atomicMin(bad, (unsigned)i);   // repeated: an earlier entry holds it
        const bool cand = row_ptr[i + 1] - row_ptr[i] >= 2;
        st[i] = cand ? 0 : 2;
        key[i] = cand ? pos[i] : INT32_MAX;
        act[i] = 1;
    }
}

// A round whose previous round counted no undecided candidate (*prev == 0)
// does nothing, so that the host can queue many rounds and read the count
// once.  A candidate comes first among the undecided candidates within R
// hops iff the smallest visiting position of an undecided candidate in its
// closed R-hop neighbourhood is its own.  That minimum is built one hop at a
// time: m1[u] = min over the closed neighbourhood of u (undecided
// candidates only), then, for rule 2, the min of m1 over the closed
// neighbourhood of v: two passes over the edges instead of a walk over
// every two-hop path.  Candidates never become undecided again, so a node
// whose closed neighbourhood holds none keeps m1 = INT32_MAX for good and
// is skipped from then on (act[v] = 0).
__global__ void seed_min1_kernel(const int32_t *row_ptr, const int32_t *col, const int32_t *key, uint8_t *act,
                                 int32_t n, int32_t *m1, const unsigned *prev, unsigned *undecided) {
    if (prev && *prev == 0u)
        return;
    unsigned cnt = 0;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * blockDim.x) {
        if (!act[v])
            continue;
        int32_t m = key[v];
        if (m != INT32_MAX)
            cnt += 1;
        // four neighbours at a time: their reads are in flight together
        const int32_t beg = row_ptr[v], len = row_ptr[v + 1] - beg;
        for (int32_t j = 0; j < len; j += 4) {
            int32_t u[4], x[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                u[q] = col[beg + min(j + q, len - 1)];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                x[q] = key[u[q]];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                m = min(m, x[q]);
        }
        m1[v] = m;
        if (m == INT32_MAX)
            act[v] = 0;
    }
    if (cnt)
        atomicAdd(undecided, cnt);
}

// Rule 2: sel[v] for undecided v whose closed two-hop minimum is its own.
__global__ void seed_min2_kernel(const int32_t *row_ptr, const int32_t *col, const int32_t *pos,
                                 const uint8_t *st, const int32_t *m1, uint8_t *sel, int32_t n,
                                 const unsigned *undecided) {
    if (*undecided == 0u)
        return;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * blockDim.x) {
        uint8_t ok = 0;
        if (st[v] == 0) {
            const int32_t pv = pos[v];
            ok = m1[v] == pv;
            for (int32_t j = row_ptr[v]; j < row_ptr[v + 1] && ok; ++j)
                ok = m1[col[j]] >= pv;
        }
        sel[v] = ok;
    }
}

// Rule 1: the selected candidates (m1 == own position) become seeds and
// their undecided neighbours are dropped.  Selected nodes are pairwise
// further apart than one hop, so a selected node's flag is written by its
// own thread only, and every other write is the same value from whichever
// thread makes it.
__global__ void seed_apply1_kernel(const int32_t *row_ptr, const int32_t *col, const int32_t *pos,
                                   const int32_t *m1, uint8_t *st, int32_t *key, int32_t n,
                                   const unsigned *undecided) {
    if (*undecided == 0u)
        return;   // the round found nothing to decide
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * blockDim.x) {
        if (st[v] != 0 || m1[v] != pos[v])
            continue;
        st[v] = 1;
        key[v] = INT32_MAX;
        for (int32_t j = row_ptr[v]; j < row_ptr[v + 1]; ++j) {
            const int32_t u = col[j];
            if (st[u] == 0) {
                st[u] = 2;
                key[u] = INT32_MAX;
            }
        }
    }
}

// Rule 2 in two one-hop passes instead of a walk over the two-hop paths of
// each selected node (one thread per selected node walked up to max-degree
// squared entries in turn): near[v] = some selected node in the closed
// neighbourhood of v; an undecided candidate then becomes a seed if
// selected, and is dropped if some node of its closed neighbourhood is
// near a selected one, i.e. if a selected node lies within two hops.
// Nodes with no undecided candidate within one hop (act[v] = 0) are never
// read by the second pass and are skipped.
__global__ void seed_near_kernel(const int32_t *row_ptr, const int32_t *col, const uint8_t *sel,
                                 const uint8_t *act, int32_t n, uint8_t *near, const unsigned *undecided) {
    if (*undecided == 0u)
        return;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * blockDim.x) {
        if (!act[v])
            continue;
        uint8_t x = sel[v];
        for (int32_t j = row_ptr[v]; j < row_ptr[v + 1] && !x; ++j)
            x = sel[col[j]];
        near[v] = x;
    }
}

__global__ void seed_apply2_kernel(const int32_t *row_ptr, const int32_t *col, const uint8_t *sel,
                                   const uint8_t *near, uint8_t *st, int32_t *key, int32_t n,
                                   const unsigned *undecided) {
    if (*undecided == 0u)
        return;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * blockDim.x) {
        if (st[v] != 0)
            continue;
        if (sel[v]) {
            st[v] = 1;
            key[v] = INT32_MAX;
            continue;
        }
        uint8_t x = near[v];
        for (int32_t j = row_ptr[v]; j < row_ptr[v + 1] && !x; ++j)
            x = near[col[j]];
        if (x) {
            st[v] = 2;
            key[v] = INT32_MAX;
        }
    }
}

__global__ void seed_flag_kernel(const int32_t *perm, const uint8_t *st, int32_t n, int32_t *flag) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        flag[i] = st[perm[i]] == 1 ? 1 : 0;
}

__global__ void seed_scatter_kernel(const int32_t *perm, const int32_t *flag, const int32_t *at, int32_t n,
                                    int32_t *out) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        if (flag[i])
            out[at[i]] = perm[i];
}

// ---------------------------------------------------------------------------
// Overlap partner of a community (check phase of Algorithm 2, and the
// overlap pre-test of Algorithm 3).  One wave per listed community c: walk
// c's members in ascending order and, for each member v, the communities
// holding v in ascending order, counting per community; the first community
// i != c whose count x reaches x * den >= num * min(|c|, |i|) is the partner
// (-1: none).  The order of the walk decides which partner is "first", so
// lanes take consecutive entries of one member's list and the lowest lane
// that reaches the threshold wins.  Counts only grow, so whether a community
// reaches its threshold within a batch of members does not depend on the
// order inside it: batches of 64 members, a lane each, are counted at once,
// and only the batch that reaches one is undone and walked again, in batches
// of 8 and then member by member.  (Walked member by member throughout, each
// a chain of five dependent reads: 0.78 ms a launch of the 20,000-node merge.)  cnt_all: one int32[n_comms] per wave
// slot, zero on entry and left zero.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) partner_kernel(const int32_t *comm_ptr, const int32_t *members,
                                                      const int32_t *node_ptr, const int32_t *node_sets,
                                                      const int32_t *list, int32_t n_list, int32_t n_comms,
                                                      int32_t eta_num, int32_t eta_den, int32_t *cnt_all,
                                                      int32_t n_slots, unsigned *next, int32_t *partner) {
    const int lane = threadIdx.x & 63;
    const int slot = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (slot >= n_slots)
        return;
    int32_t *cnt = cnt_all + (int64_t)slot * n_comms;
    // item and found are held wave-uniform (scalar registers), and the loop
    // has no lane-0-only block at its end: a lane-0 block at both ends of the
    // loop lets the compiler thread them into a second back edge that lanes
    // 1..63 take alone, with no exit for them while lane 0 waits outside.
    for (;;) {
        unsigned item = 0;
        if (lane == 0)
            item = atomicAdd(next, 1u);
        item = (unsigned)__builtin_amdgcn_readfirstlane((int)item);
        if (item >= (unsigned)n_list)
            break;
        const int32_t c = list[item];
        const int32_t nm = comm_ptr[c + 1] - comm_ptr[c];
        const int32_t *mem = members + comm_ptr[c];
        const int64_t sc = nm;
        int32_t found = -1;
        // counts of the incidences of the members [q, q + 64 / per), per lanes
        // to a member's list; by: +1 (true when some community reaches its
        // threshold) or -1 (undone)
        const auto visit = [&](int32_t q, int32_t end, int per, int by) -> bool {
            const int32_t at = q + lane / per;
            const int32_t v = at < end ? mem[at] : -1;
            const int32_t t0 = v >= 0 ? node_ptr[v] : 0;
            const int32_t len = v >= 0 ? node_ptr[v + 1] - t0 : 0;
            bool hit = false;
            for (int32_t t = lane % per; t < len; t += per) {
                const int32_t i = node_sets[t0 + t];
                if (i == c)
                    continue;
                const int64_t x = (int64_t)atomicAdd(&cnt[i], by) + by;
                const int64_t si = comm_ptr[i + 1] - comm_ptr[i];
                const int64_t small = sc < si ? sc : si;
                hit = hit || x * eta_den >= (int64_t)eta_num * small;
            }
            // the next lanes to count a community see these counts
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
            __builtin_amdgcn_wave_barrier();
            return __ballot(hit) != 0;
        };
        int32_t done = 0;   // members before done have been counted
        for (int32_t q = 0; q < nm && found < 0; q += 64) {
            done = min(q + 64, nm);
            if (!visit(q, done, 1, 1))
                continue;
            visit(q, done, 1, -1);
            for (int32_t s = q; s < done && found < 0; s += 8) {
                const int32_t s1 = min(s + 8, done);
                if (!visit(s, s1, 8, 1))
                    continue;
                visit(s, s1, 8, -1);
                for (int32_t r = s; r < s1 && found < 0; ++r) {
                    const int32_t v = mem[r];
                    const int32_t t0 = node_ptr[v], len = node_ptr[v + 1] - t0;
                    for (int32_t t = 0; t < len && found < 0; t += 64) {
                        const int32_t i = t + lane < len ? node_sets[t0 + t + lane] : -1;
                        bool hit = false;
                        if (i >= 0 && i != c) {
                            const int64_t x = (int64_t)atomicAdd(&cnt[i], 1) + 1;
                            const int64_t si = comm_ptr[i + 1] - comm_ptr[i];
                            const int64_t small = sc < si ? sc : si;
                            hit = x * eta_den >= (int64_t)eta_num * small;
                        }
                        const uint64_t m = __ballot(hit);
                        if (m)
                            found = __builtin_amdgcn_readlane(i, (int)__builtin_ctzll(m));
                    }
                }
            }
        }
        // leave the counts at zero for the next community
        for (int32_t q = lane; q < done; q += 64) {
            const int32_t v = mem[q];
            for (int32_t t = node_ptr[v]; t < node_ptr[v + 1]; ++t) {
                const int32_t i = node_sets[t];
                if (i != c)
                    atomicExch(&cnt[i], 0);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        __builtin_amdgcn_wave_barrier();
        // every lane stores the same value (no lane-0 branch, see above)
        partner[item] = found;
    }
}

// Order one tier's overflow list for the next tier: items set * S + s by
// ascending s, so that the sets with the most scales left start first (a
// tier lasts as long as its slowest workgroup).  One workgroup; the order
// never changes a result.
__global__ void __launch_bounds__(1024) order_spills_kernel(const int32_t *in, const uint32_t *count,
                                                            uint32_t n_max, int32_t S, int32_t *out) {
    __shared__ uint32_t hist[1024];
    const uint32_t n = min(*count, n_max);
    const uint32_t tid = threadIdx.x;
    for (int32_t s = (int32_t)tid; s < S; s += 1024)
        hist[s] = 0u;
    __syncthreads();
    for (uint32_t i = tid; i < n; i += 1024)
        atomicAdd(&hist[(uint32_t)in[i] % (uint32_t)S], 1u);
    __syncthreads();
    if (tid == 0) {
        uint32_t run = 0;
        for (int32_t s = 0; s < S; ++s) {
            const uint32_t c = hist[s];
            hist[s] = run;
            run += c;
        }
    }
    __syncthreads();
    for (uint32_t i = tid; i < n; i += 1024) {
        const int32_t w = in[i];
        const uint32_t pos = atomicAdd(&hist[(uint32_t)w % (uint32_t)S], 1u);
        out[pos] = w;
    }
}

// three-phase exclusive scan of n counts into ptr[0..n]
__global__ void __launch_bounds__(1024) scan_blocks_kernel(const int32_t *cnt, int64_t n,
                                                           int32_t *ptr, int32_t *block_sums) {
    __shared__ int32_t part[1024];
    const int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    const int32_t v = i < n ? cnt[i] : 0;
    part[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        int32_t x = threadIdx.x >= off ? part[threadIdx.x - off] : 0;
        __syncthreads();
        part[threadIdx.x] += x;
        __syncthreads();
    }
    if (i < n)
        ptr[i] = part[threadIdx.x] - v;
    if (threadIdx.x == 1023)
        block_sums[blockIdx.x] = part[1023];
}

__global__ void __launch_bounds__(1024) scan_sums_kernel(int32_t *block_sums, int32_t nb,
                                                         int32_t *total_out) {
    __shared__ int32_t part[1024];
    const int tid = threadIdx.x;
    const int per = (nb + 1023) / 1024;
    const int lo = tid * per;
    const int hi = lo + per < nb ? lo + per : nb;
    int32_t sum = 0;
    for (int j = lo; j < hi; ++j)
        sum += block_sums[j];
    part[tid] = sum;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        int32_t x = tid >= off ? part[tid - off] : 0;
        __syncthreads();
        part[tid] += x;
        __syncthreads();
    }
    int32_t run = part[tid] - sum;
    for (int j = lo; j < hi; ++j) {
        const int32_t b = block_sums[j];
        block_sums[j] = run;
        run += b;
    }
    if (tid == 1023)
        *total_out = part[1023];
}

__global__ void scan_add_kernel(int32_t *ptr, int64_t n, const int32_t *block_sums) {
    const int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    if (i < n)
        ptr[i] += block_sums[blockIdx.x];
}

__global__ void __launch_bounds__(256) overlap_scatter_kernel(const int32_t *comm_ptr,
                                                              const int32_t *members, int32_t n_sets,
                                                              const int32_t *node_ptr, int32_t *fill,
                                                              int32_t *node_sets) {
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int64_t j = (int64_t)blockIdx.x * (blockDim.x >> 6) + wave;
    if (j >= n_sets)
        return;
    const int32_t beg = comm_ptr[j], len = comm_ptr[j + 1] - beg;
    for (int32_t i = lane; i < len; i += 64) {
        const int32_t u = members[beg + i];
        const int32_t pos = atomicAdd(&fill[u], 1);
        node_sets[node_ptr[u] + pos] = (int32_t)j;
    }
}

// Sort every node's list: lanes sort short lists alone; each long list is
// then sorted by the whole wave.
__global__ void __launch_bounds__(256) overlap_sort_kernel(const int32_t *node_ptr, int32_t n,
                                                           int32_t *node_sets) {
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int64_t u = ((int64_t)blockIdx.x * (blockDim.x >> 6) + wave) * 64 + lane;
    int32_t lo = 0, len = 0;
    if (u < n) {
        lo = node_ptr[u];
        len = node_ptr[u + 1] - lo;
    }
    const bool longl = len > 32;
    if (!longl && len > 1) {
        int32_t *a = node_sets + lo;
        for (int32_t i = 1; i < len; ++i) {
            const int32_t x = a[i];
            int32_t j = i - 1;
            while (j >= 0 && a[j] > x) {
                a[j + 1] = a[j];
                --j;
            }
            a[j + 1] = x;
        }
    }
    uint64_t todo = __ballot(longl);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    while (todo) {
        const int src = __builtin_ctzll(todo);
        todo &= todo - 1;
        const int32_t l0 = __shfl(lo, src);
        const int32_t n0 = __shfl(len, src);
        wave_sort<true>(node_sets + l0, n0, lane);
    }
}

// (one atomic per workgroup and counter: per wave, 40,000 of them on four
// addresses took 0.49 ms for 640,000 records)
__global__ void __launch_bounds__(256) counter_sum_kernel(const uint64_t *ctr, int64_t n_rec,
                                                          unsigned long long *tot) {
    __shared__ unsigned long long part[4][4];
    unsigned long long s[4] = {0, 0, 0, 0};
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n_rec;
         r += (int64_t)gridDim.x * blockDim.x) {
        for (int q = 0; q < 4; ++q)
            s[q] += ctr[4 * r + q];
    }
    for (int q = 0; q < 4; ++q) {
        unsigned long long v = s[q];
        for (int off = 32; off >= 1; off >>= 1)
            v += __shfl_xor(v, off);
        if ((threadIdx.x & 63) == 0)
            part[threadIdx.x >> 6][q] = v;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int q = threadIdx.x;
        const unsigned long long v = part[0][q] + part[1][q] + part[2][q] + part[3][q];
        if (v)
            atomicAdd(&tot[q], v);
    }
}

// ---------------------------------------------------------------------------
// Normalised mutual information of two covers (Sec. 4 compares community
// sets of successive scales with the overlapping-community NMI of
// Lancichinetti, Fortunato and Kertesz, 2009).  Entropies are in nats,
// h(c) = (c / n) (L(n) - L(c)) for a count c of n nodes, taken from a table
// built with the specified integer log, so that the admission test
// h(a) + h(e) > h(b) + h(c) decides exactly as in any other implementation
// of the same specification.  Empty communities are skipped.
// ---------------------------------------------------------------------------
__global__ void nmi_htab_kernel(double *h, int32_t n) {
    const double ln_n = n > 0 ? ilog((uint64_t)n) : 0.0;
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c <= n;
         c += (int64_t)gridDim.x * blockDim.x) {
        if (c == 0) {
            h[c] = 0.0;
            continue;
        }
        const double t = ln_n - ilog((uint64_t)c);
        const double p = (double)c / (double)n;
        h[c] = p * t;
    }
}

// H(X_k | Y) / H(X_k) for every community k of X, one wave per community
// from a work counter: the wave counts X_k's intersections with every Y_l
// through Y's node -> communities lists (cnt: one zeroed int32[ky] row per
// wave slot, left zeroed), then takes the least admitted conditional
// entropy over all non-empty Y_l.  term[k] = -1 marks an empty X_k.
__global__ void __launch_bounds__(256) nmi_half_kernel(const int32_t *px, const int32_t *mx, int32_t kx,
                                                       const int32_t *py, int32_t ky, const int32_t *node_ptr,
                                                       const int32_t *node_sets, const double *h, int32_t n,
                                                       int32_t *cnt_all, int32_t n_slots, unsigned *next,
                                                       double *term) {
    const int lane = threadIdx.x & 63;
    const int slot = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (slot >= n_slots)
        return;
    int32_t *cnt = cnt_all + (int64_t)slot * ky;
    // the item is wave-uniform and the loop has no lane-0 block at its end
    for (;;) {
        unsigned item = 0;
        if (lane == 0)
            item = atomicAdd(next, 1u);
        item = (unsigned)__builtin_amdgcn_readfirstlane((int)item);
        if (item >= (unsigned)kx)
            break;
        const int32_t k = (int32_t)item;
        const int32_t x0 = px[k], x1 = px[k + 1];
        const int32_t sx = x1 - x0;
        double out = -1.0;
        if (sx > 0) {
            for (int32_t q = lane; q < sx; q += 64) {
                const int32_t v = mx[x0 + q];
                for (int32_t t = node_ptr[v]; t < node_ptr[v + 1]; ++t)
                    atomicAdd(&cnt[node_sets[t]], 1);
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
            __builtin_amdgcn_wave_barrier();
            const double hx = h[sx] + h[n - sx];
            double best = 0.0;
            int found = 0;
            for (int32_t l = lane; l < ky; l += 64) {
                const int32_t sy = py[l + 1] - py[l];
                if (sy == 0)
                    continue;
                const int32_t a = atomicExch(&cnt[l], 0);   // read at L2 and leave it zero
                const int32_t b = sx - a, c = sy - a, e = n - a - b - c;
                const double ha = h[a], hb = h[b], hc = h[c], he = h[e];
                if (!(ha + he > hb + hc))
                    continue;
                const double hxy = ((ha + hb) + hc) + he;
                const double hy = h[sy] + h[n - sy];
                const double cond = hxy - hy;
                if (!found || cond < best) {
                    best = cond;
                    found = 1;
                }
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                const double b2 = __shfl_xor(best, off);
                const int f2 = __shfl_xor(found, off);
                if (f2 && (!found || b2 < best)) {
                    best = b2;
                    found = 1;
                }
            }
            if (!found)
                best = hx;
            out = hx > 0.0 ? best / hx : 0.0;
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
            __builtin_amdgcn_wave_barrier();
        }
        // every lane stores the same value
        term[k] = out;
    }
}

// Mean of the terms that are not -1 (one workgroup, fixed order), written
// with its count: res[0] = mean, res[1] = count.
__global__ void __launch_bounds__(1024) nmi_mean_kernel(const double *term, int32_t k, double *res) {
    __shared__ double s[1024];
    __shared__ int c[1024];
    double acc = 0.0;
    int cc = 0;
    for (int32_t i = threadIdx.x; i < k; i += 1024) {
        const double x = term[i];
        if (x >= 0.0) {
            acc += x;
            cc += 1;
        }
    }
    s[threadIdx.x] = acc;
    c[threadIdx.x] = cc;
    __syncthreads();
    for (int off = 512; off >= 1; off >>= 1) {
        if ((int)threadIdx.x < off) {
            s[threadIdx.x] += s[threadIdx.x + off];
            c[threadIdx.x] += c[threadIdx.x + off];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        res[0] = c[0] > 0 ? s[0] / (double)c[0] : 0.0;
        res[1] = (double)c[0];
    }
}

// Checks a cover given as CSR: offsets from 0 to total, non-decreasing;
// every community strictly ascending with ids in [0, n).  Any breach sets
// *bad.
// One wave per community: a thread per community read its list entry by
// entry, 150 us for 50,000 nodes.
__global__ void __launch_bounds__(256) cover_check_kernel(const int32_t *ptr, const int32_t *mem, int32_t k,
                                                          int64_t total, int32_t n, uint32_t *bad) {
    const int lane = threadIdx.x & 63;
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x >> 6);
    bool breach = false;
    for (int64_t j = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); j < k; j += waves) {
        const int32_t a = ptr[j], b = ptr[j + 1];
        if (b < a || a < 0 || (int64_t)b > total || (j == 0 && a != 0) || (j == k - 1 && (int64_t)b != total)) {
            breach = true;
            continue;
        }
        for (int32_t q = lane; q < b - a; q += 64) {
            const int32_t v = mem[a + q];
            breach = breach || v < 0 || v >= n || (q > 0 && v <= mem[a + q - 1]);
        }
    }
    if (breach)
        atomicOr(bad, 1u);
}

// Means of the p - 1 consecutive pair values of each window of p scales.
__global__ void nmi_windows_kernel(const double *pair, int32_t S, int32_t p, double *out) {
    const int32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s > S - p)
        return;
    double acc = 0.0;
    for (int32_t t = s; t < s + p - 1; ++t)
        acc += pair[t];
    out[s] = acc / (double)(p - 1);
}

// NMI from the two halves (N4: a cover without a non-empty community).
__global__ void nmi_final_kernel(const double *hx, const double *hy, double *out) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        const bool ex = hx[1] > 0.0, ey = hy[1] > 0.0;
        if (!ex || !ey)
            *out = (!ex && !ey) ? 1.0 : 0.0;
        else
            *out = 1.0 - (hx[0] + hy[0]) / 2.0;
    }
}

inline int grid_for(int64_t n, int block) {
    int64_t g = (n + block - 1) / block;
    if (g < 1)
        g = 1;
    if (g > 65535 * 64)
        g = 65535 * 64;
    return (int)g;
}

}  // namespace

hipError_t launch_check_graph(const int32_t *row_ptr, const int32_t *col, const uint8_t *w, int32_t *kdeg, int32_t n,
                              int64_t nnz, GraphCheck *chk, hipStream_t st) {
    if (n <= 0)
        return hipSuccess;
    const int rows = (int)std::min<int64_t>(((int64_t)n + 255) / 256, 4096);
    hipLaunchKernelGGL(degrees_kernel, dim3(rows), dim3(256), 0, st, row_ptr, w, kdeg, n, chk);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || nnz <= 0)
        return e;
    const int blocks = (int)std::min<int64_t>((nnz + 255) / 256, 16384);
    hipLaunchKernelGGL(check_graph_kernel, dim3(blocks), dim3(256), 0, st, row_ptr, col, w, n, nnz, chk);
    return hipGetLastError();
}

hipError_t launch_node_info(const int32_t *row_ptr, const int32_t *kdeg, int2 *info, int32_t n, hipStream_t st) {
    if (n == 0)
        return hipSuccess;
    hipLaunchKernelGGL(node_info_kernel, dim3(grid_for(n, 256)), dim3(256), 0, st, row_ptr, kdeg, info, n);
    return hipGetLastError();
}

hipError_t launch_adj(const int32_t *row_ptr, const int32_t *col, const uint8_t *w, const int32_t *kdeg,
                      const double *logtab, int64_t nnz, int4 *adj, double *adjl, hipStream_t st) {
    if (nnz == 0)
        return hipSuccess;
    const int g = grid_for(nnz, 256) < 16384 ? grid_for(nnz, 256) : 16384;
    hipLaunchKernelGGL(adj_kernel, dim3(g), dim3(256), 0, st, row_ptr, col, w, kdeg, logtab, nnz, adj, adjl);
    return hipGetLastError();
}

hipError_t launch_logtab(double *tab, int32_t m, hipStream_t st) {
    hipLaunchKernelGGL(logtab_kernel, dim3(grid_for(m, 256)), dim3(256), 0, st, tab, m);
    return hipGetLastError();
}

hipError_t launch_log(const uint64_t *x, double *out, int64_t n, hipStream_t st) {
    if (n == 0)
        return hipSuccess;
    hipLaunchKernelGGL(log_kernel, dim3(grid_for(n, 256)), dim3(256), 0, st, x, out, n);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t st) {
    if (n == 0)
        return hipSuccess;
    int64_t g = (n + 255) / 256;
    if (g > 16384)
        g = 16384;
    hipLaunchKernelGGL(fill_i32_kernel, dim3((int)g), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}

hipError_t launch_zero_bytes(void *p, int64_t bytes, hipStream_t st) {
    // callers pass 4-byte multiples
    return launch_fill_i32((int32_t *)p, 0, bytes / 4, st);
}

hipError_t launch_sweep(const SweepArgs &a, int32_t blocks, int32_t waves_per_block, hipStream_t st) {
    if (blocks <= 0)
        return hipSuccess;
    const bool q = a.alpha_set != nullptr;
    if (q && (a.S != 1 || a.s_begin != 0 || a.s_end != 1 || a.resume))
        return hipErrorInvalidValue;
    const dim3 grid(blocks), block(64 * waves_per_block);
    switch (a.kind) {
    case TIER_WAVE_LDS: {
        if (waves_per_block < 1 || waves_per_block > 4)
            return hipErrorInvalidValue;
        const size_t smem = (size_t)waves_per_block * (size_t)table_bytes(a.cap, a.hbits);
        hipLaunchKernelGGL(q ? query_lds_kernel : sweep_lds_kernel, grid, block, smem, st, a);
        break;
    }
    case TIER_WAVE_GLOBAL:
        if (waves_per_block < 1 || waves_per_block > 4 || a.gtab == nullptr)
            return hipErrorInvalidValue;
        hipLaunchKernelGGL(q ? query_global_kernel : sweep_global_kernel, grid, block, 0, st, a);
        break;
    case TIER_TEAM_LDS: {
        if (waves_per_block < 1 || 64 * waves_per_block > kTeamMaxThreads || a.cap > kPackMaxEntries)
            return hipErrorInvalidValue;
        const size_t smem = (size_t)block_table_bytes(a.cap, a.hbits);
        hipLaunchKernelGGL(q ? query_team_lds_kernel : sweep_team_lds_kernel, grid, block, smem, st, a);
        break;
    }
    case TIER_TEAM_GLOBAL:
        if (waves_per_block < 1 || 64 * waves_per_block > kTeamMaxThreads || a.gtab == nullptr ||
            !team_table_holds(a.cap))
            return hipErrorInvalidValue;
        if (a.cap >= kRecordMinEntries)
            hipLaunchKernelGGL(q ? query_team_global_rec_kernel : sweep_team_global_rec_kernel, grid, block, 0, st,
                               a);
        else
            hipLaunchKernelGGL(q ? query_team_global_kernel : sweep_team_global_kernel, grid, block, 0, st, a);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t tier_blocks_per_cu(int32_t kind, int32_t cap, int32_t waves, size_t lds_bytes, int32_t *out) {
    const void *f = nullptr;
    switch (kind) {
    case TIER_WAVE_LDS: f = reinterpret_cast<const void *>(&sweep_lds_kernel); break;
    case TIER_WAVE_GLOBAL: f = reinterpret_cast<const void *>(&sweep_global_kernel); break;
    case TIER_TEAM_LDS: f = reinterpret_cast<const void *>(&sweep_team_lds_kernel); break;
    case TIER_TEAM_GLOBAL:
        f = cap >= kRecordMinEntries ? reinterpret_cast<const void *>(&sweep_team_global_rec_kernel)
                                     : reinterpret_cast<const void *>(&sweep_team_global_kernel);
        break;
    default: return hipErrorInvalidValue;
    }
    int nb = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, 64 * waves, lds_bytes);
    *out = nb;
    return e;
}

hipError_t launch_scale_scan(const Records &rec, int32_t S, int32_t s, int32_t n_sets,
                             int32_t *comm_ptr, long long *total, hipStream_t st) {
    // a chunk per workgroup, at most 64 of them
    const int32_t chunk = std::max(1, (int32_t)(((int64_t)n_sets + 65535) / 65536)) * 1024;
    const int32_t blocks = std::max(1, (int32_t)(((int64_t)n_sets + chunk - 1) / chunk));
    hipLaunchKernelGGL(scale_scan_kernel, dim3(blocks), dim3(1024), 0, st, rec.cnt, S, s, n_sets, chunk, comm_ptr,
                       total);
    return hipGetLastError();
}

hipError_t launch_scale_gather(const Records &rec, const int32_t *pool, const double *scales,
                               int32_t S, int32_t s, int32_t n_sets, const int32_t *comm_ptr,
                               int32_t *members, int64_t *k_in, int64_t *vol, double *f,
                               hipStream_t st) {
    if (n_sets == 0)
        return hipSuccess;
    hipLaunchKernelGGL(scale_gather_kernel, dim3((n_sets + 3) / 4), dim3(256), 0, st, rec, pool, scales,
                       S, s, n_sets, comm_ptr, members, k_in, vol, f);
    return hipGetLastError();
}

hipError_t launch_delta_events(const Records &rec, int32_t S, int32_t s, const int32_t *sets, int32_t n,
                               int64_t *ev, int64_t *ev_off, uint32_t *err, hipStream_t st) {
    if (n > 0) {
        hipLaunchKernelGGL(delta_events_kernel, dim3((unsigned)std::min<int64_t>(4096, (n + 255) / 256)), dim3(256),
                           0, st, rec, S, s, sets, n, ev, err);
    }
    hipLaunchKernelGGL(scan_i64_kernel, dim3(1), dim3(1024), 0, st, ev, (int64_t)n, ev_off);
    return hipGetLastError();
}

hipError_t launch_delta_rebuild(const Records &rec, const int32_t *pool, int32_t S, int32_t s,
                                const int32_t *sets, int32_t n, const int64_t *ev_off, int32_t *scratch,
                                const int32_t *out_ptr, int32_t *members, uint32_t *err, hipStream_t st) {
    if (n == 0)
        return hipSuccess;
    hipLaunchKernelGGL(delta_rebuild_kernel, dim3((unsigned)std::min<int64_t>(65536, n)), dim3(256), 0, st, rec,
                       pool, S, s, sets, n, ev_off, scratch, out_ptr, members, err);
    return hipGetLastError();
}

hipError_t launch_delta_lists(const Records &rec, const int32_t *pool, int32_t S, int32_t s, int32_t n,
                              int64_t *na, int64_t *nr, int64_t *add_off, int64_t *rem_off, int32_t *added,
                              int32_t *removed, hipStream_t st) {
    if (n > 0)
        hipLaunchKernelGGL(delta_counts_kernel, dim3((unsigned)std::min<int64_t>(4096, (n + 255) / 256)),
                           dim3(256), 0, st, rec, S, s, n, na, nr);
    hipLaunchKernelGGL(scan_i64_kernel, dim3(1), dim3(1024), 0, st, na, (int64_t)n, add_off);
    hipLaunchKernelGGL(scan_i64_kernel, dim3(1), dim3(1024), 0, st, nr, (int64_t)n, rem_off);
    if ((added || removed) && n > 0)
        hipLaunchKernelGGL(delta_gather_kernel, dim3((n + 3) / 4), dim3(256), 0, st, rec, pool, S, s, n, add_off,
                           added, rem_off, removed);
    return hipGetLastError();
}

hipError_t launch_overlap(const int32_t *comm_ptr, const int32_t *members, int64_t total,
                               int32_t n_sets, int32_t n, int32_t *node_ptr, int32_t *node_sets,
                               int32_t *cnt, int32_t *block_sums, hipStream_t st) {
    hipError_t e;
    if ((e = launch_fill_i32(cnt, 0, (int64_t)n + 1, st)) != hipSuccess)
        return e;
    if (total > 0) {
        hipLaunchKernelGGL(overlap_count_kernel, dim3(grid_for(total, 256) < 8192 ? grid_for(total, 256) : 8192),
                           dim3(256), 0, st, members, total, cnt);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
    }
    const int64_t nn = (int64_t)n + 1;
    const int nb = (int)((nn + 1023) / 1024);
    hipLaunchKernelGGL(scan_blocks_kernel, dim3(nb), dim3(1024), 0, st, cnt, nn, node_ptr, block_sums);
    hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(1024), 0, st, block_sums, nb, block_sums + nb);
    hipLaunchKernelGGL(scan_add_kernel, dim3(nb), dim3(1024), 0, st, node_ptr, nn, block_sums);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    if ((e = launch_fill_i32(cnt, 0, (int64_t)n + 1, st)) != hipSuccess)
        return e;
    if (n_sets > 0) {
        hipLaunchKernelGGL(overlap_scatter_kernel, dim3((n_sets + 3) / 4), dim3(256), 0, st, comm_ptr,
                           members, n_sets, node_ptr, cnt, node_sets);
    }
    if (n > 0) {
        const int64_t waves = ((int64_t)n + 63) / 64;
        hipLaunchKernelGGL(overlap_sort_kernel, dim3((int)((waves + 3) / 4)), dim3(256), 0, st, node_ptr,
                           n, node_sets);
    }
    return hipGetLastError();
}

hipError_t launch_order_spills(const int32_t *in, const uint32_t *count, uint32_t n_max, int32_t S,
                               int32_t *out, hipStream_t st) {
    if (S < 2 || S > 1024 || n_max == 0)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(order_spills_kernel, dim3(1), dim3(1024), 0, st, in, count, n_max, S, out);
    return hipGetLastError();
}

hipError_t launch_exclusive_scan(const int32_t *in, int64_t n, int32_t *out, int32_t *block_sums,
                                 hipStream_t st) {
    const int nb = (int)((n + 1023) / 1024);
    if (nb == 0)
        return hipSuccess;
    if (nb > 1024 * 1024)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(scan_blocks_kernel, dim3(nb), dim3(1024), 0, st, in, n, out, block_sums);
    hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(1024), 0, st, block_sums, nb, block_sums + nb);
    hipLaunchKernelGGL(scan_add_kernel, dim3(nb), dim3(1024), 0, st, out, n, block_sums);
    return hipGetLastError();
}

hipError_t launch_seed_init(const int32_t *row_ptr, const int32_t *perm, int32_t n, int32_t *pos, uint8_t *st,
                            uint8_t *act, int32_t *key, unsigned *bad, hipStream_t s) {
    if (n == 0)
        return hipSuccess;
    hipError_t e = launch_fill_i32(pos, INT32_MAX, n, s);
    if (e == hipSuccess)
        e = launch_fill_i32((int32_t *)bad, -1, 1, s);
    if (e != hipSuccess)
        return e;
    const dim3 g(grid_for(n, 256)), b(256);
    hipLaunchKernelGGL(seed_perm_kernel, g, b, 0, s, perm, n, pos, bad);
    hipLaunchKernelGGL(seed_init_kernel, g, b, 0, s, row_ptr, perm, n, pos, st, act, key, bad);
    return hipGetLastError();
}

hipError_t launch_seed_round(int32_t rule, const int32_t *row_ptr, const int32_t *col, const int32_t *pos,
                             uint8_t *st, uint8_t *sel, uint8_t *act, uint8_t *near, int32_t *m1, int32_t *key, int32_t n,
                             const unsigned *prev, unsigned *undecided, hipStream_t s) {
    if (n == 0)
        return hipSuccess;
    if (rule != 1 && rule != 2)
        return hipErrorInvalidValue;
    const dim3 g(grid_for(n, 256)), b(256);
    hipLaunchKernelGGL(seed_min1_kernel, g, b, 0, s, row_ptr, col, key, act, n, m1, prev, undecided);
    if (rule == 1) {
        hipLaunchKernelGGL(seed_apply1_kernel, g, b, 0, s, row_ptr, col, pos, m1, st, key, n, undecided);
    } else {
        hipLaunchKernelGGL(seed_min2_kernel, g, b, 0, s, row_ptr, col, pos, st, m1, sel, n, undecided);
        hipLaunchKernelGGL(seed_near_kernel, g, b, 0, s, row_ptr, col, sel, act, n, near, undecided);
        hipLaunchKernelGGL(seed_apply2_kernel, g, b, 0, s, row_ptr, col, sel, near, st, key, n, undecided);
    }
    return hipGetLastError();
}

hipError_t launch_seed_collect(const int32_t *perm, const uint8_t *st, int32_t n, int32_t *flag, int32_t *at,
                               int32_t *block_sums, int32_t *out, hipStream_t s) {
    if (n == 0)
        return hipSuccess;
    hipLaunchKernelGGL(seed_flag_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, perm, st, n, flag);
    hipError_t e = launch_exclusive_scan(flag, n, at, block_sums, s);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(seed_scatter_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, perm, flag, at, n, out);
    return hipGetLastError();
}

hipError_t launch_partner(const int32_t *comm_ptr, const int32_t *members, const int32_t *node_ptr,
                          const int32_t *node_sets, const int32_t *list, int32_t n_list, int32_t n_comms,
                          int32_t eta_num, int32_t eta_den, int32_t *cnt_all, int32_t n_slots, unsigned *next,
                          int32_t *partner, hipStream_t st) {
    if (n_list == 0)
        return hipSuccess;
    hipError_t e = launch_zero_bytes(next, 4, st);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(partner_kernel, dim3((n_slots + 3) / 4), dim3(256), 0, st, comm_ptr, members, node_ptr,
                       node_sets, list, n_list, n_comms, eta_num, eta_den, cnt_all, n_slots, next, partner);
    return hipGetLastError();
}

hipError_t launch_nmi_htab(double *h, int32_t n, hipStream_t st) {
    hipLaunchKernelGGL(nmi_htab_kernel, dim3(grid_for((int64_t)n + 1, 256)), dim3(256), 0, st, h, n);
    return hipGetLastError();
}

hipError_t launch_nmi_half(const int32_t *px, const int32_t *mx, int32_t kx, const int32_t *py, int32_t ky,
                           const int32_t *node_ptr, const int32_t *node_sets, const double *h, int32_t n,
                           int32_t *cnt_all, int32_t n_slots, unsigned *next, double *term, double *res,
                           hipStream_t st) {
    hipError_t e = launch_zero_bytes(next, 4, st);
    if (e != hipSuccess)
        return e;
    if (kx > 0)
        hipLaunchKernelGGL(nmi_half_kernel, dim3((n_slots + 3) / 4), dim3(256), 0, st, px, mx, kx, py, ky, node_ptr,
                           node_sets, h, n, cnt_all, n_slots, next, term);
    hipLaunchKernelGGL(nmi_mean_kernel, dim3(1), dim3(1024), 0, st, term, kx, res);
    return hipGetLastError();
}

hipError_t launch_nmi_final(const double *hx, const double *hy, double *out, hipStream_t st) {
    hipLaunchKernelGGL(nmi_final_kernel, dim3(1), dim3(64), 0, st, hx, hy, out);
    return hipGetLastError();
}

hipError_t launch_cover_check(const int32_t *ptr, const int32_t *mem, int32_t k, int64_t total, int32_t n,
                              uint32_t *bad, hipStream_t st) {
    hipError_t e = launch_zero_bytes(bad, 4, st);
    if (e != hipSuccess || k == 0)
        return e;
    hipLaunchKernelGGL(cover_check_kernel, dim3(grid_for(k, 4) < 4096 ? grid_for(k, 4) : 4096), dim3(256), 0, st,
                       ptr, mem, k, total, n, bad);
    return hipGetLastError();
}

hipError_t launch_nmi_windows(const double *pair, int32_t S, int32_t p, double *out, hipStream_t st) {
    if (p < 2 || p > S)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(nmi_windows_kernel, dim3((S - p + 1 + 255) / 256), dim3(256), 0, st, pair, S, p, out);
    return hipGetLastError();
}

hipError_t launch_counter_sum(const uint64_t *ctr, int64_t n_rec, unsigned long long *tot,
                              hipStream_t st) {
    if (n_rec == 0)
        return hipSuccess;
    hipLaunchKernelGGL(counter_sum_kernel, dim3(grid_for(n_rec, 256) < 512 ? grid_for(n_rec, 256) : 512),
                       dim3(256), 0, st, ctr, n_rec, tot);
    return hipGetLastError();
}

}  // namespace lcd
