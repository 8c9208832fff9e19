// HIP kernels (gfx950) for full-neighbourhood move evaluation, best-move
// reduction, move application and attribute rebuild.
//
// The paper evaluates moves by concatenating route subsequences whose
// attributes are precomputed (Section 4.1; distance: eq. dist; load: the
// zero-pickup form of the load concatenation; windows: Section 4.3.3), in
// five steps per operator (Section 5.1): extraction, concatenation,
// differencing, evaluation (argmin), update.  Here the five steps are fused
// per pair of positions: the attribute "tensor" is a set of per-slot arrays
// (route id and position, as the positional tensors of Section 5.3.1; prefix
// load; edge to the successor; earliest departure; latest feasible arrival
// at the successor), every concatenation is evaluated in registers, and the
// argmin is a running (delta, id) minimum per lane followed by a wavefront and
// workgroup reduction and one 64-bit atomicMin per solution.
//
// Time windows use the hard-window case of the time-warp algebra (Section
// 4.3.3: a concatenation is feasible exactly when its time-window violation
// T_V is zero): forward earliest service starts A, backward latest arrivals
// Z, and (duration, earliest finish, latest arrival) summaries for the middle
// segments of intra-route moves.

#include "tga_internal.h"
#include <type_traits>

namespace tga {

constexpr int kInterWaves = 8;      // wavefronts per inter-route workgroup
constexpr int kInterThreads = kInterWaves * 64;
constexpr int kColsPerWave = 62;    // lanes 1..62 own a column; 0 and 63 are halo
constexpr int kIntraThreads = 256;
constexpr int kApplyThreads = 1024;
constexpr int kTwOff = 1 << 28;     // due time standing for "no window" (CVRP)

// Loads through pointers kept in the solution descriptor: the pointee is
// global memory, so say so (global_load instead of a generic flat load).
template <class T>
__device__ __forceinline__ T gld(const T *p) {
    return *(const __attribute__((address_space(1))) T *)p;
}

__device__ __forceinline__ int4 gld(const int4 *p) {
    typedef int v4i __attribute__((ext_vector_type(4)));
    const v4i v = *(const __attribute__((address_space(1))) v4i *)p;
    return make_int4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ int2 gld(const int2 *p) {
    typedef int v2i __attribute__((ext_vector_type(2)));
    const v2i v = *(const __attribute__((address_space(1))) v2i *)p;
    return make_int2(v.x, v.y);
}

// Load of a value every lane of the wavefront reads at the same address,
// through the constant address space so that it becomes a scalar load into
// SGPRs.  Only for data no kernel of the same launch writes.
__device__ __forceinline__ int4 sld(const int4 *p) {
    typedef int v4i __attribute__((ext_vector_type(4)));
    const v4i v = *(const __attribute__((address_space(4))) v4i *)p;
    return make_int4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ int sld1(const int *p) { return *(const __attribute__((address_space(4))) int *)p; }

// The same at a byte offset from p (one scalar load with an offset register).
__device__ __forceinline__ int4 sld_at(const int4 *p, uint32_t byte_off) {
    typedef int v4i __attribute__((ext_vector_type(4)));
    const __attribute__((address_space(4))) char *b = (const __attribute__((address_space(4))) char *)p;
    const v4i v = *(const __attribute__((address_space(4))) v4i *)(b + byte_off);
    return make_int4(v.x, v.y, v.z, v.w);
}

template <class T>
__device__ __forceinline__ void gst(T *p, T v) {
    *(__attribute__((address_space(1))) T *)p = v;
}

__device__ __forceinline__ void gst(int4 *p, int4 v) {
    typedef int v4i __attribute__((ext_vector_type(4)));
    const v4i x = {v.x, v.y, v.z, v.w};
    *(__attribute__((address_space(1))) v4i *)p = x;
}

__device__ __forceinline__ void gst(int2 *p, int2 v) {
    typedef int v2i __attribute__((ext_vector_type(2)));
    const v2i x = {v.x, v.y};
    *(__attribute__((address_space(1))) v2i *)p = x;
}

__device__ __forceinline__ int nodeof(int x) { return x & 0xFFFF; }
__device__ __forceinline__ int flagsof(int x) { return x >> 16; }

// Deltas at or above this are not admissible (inter-route moves carry a
// penalty of 2^30; every admissible delta is far below 2^29).
constexpr int kAdmissibleBound = 1 << 29;

// Internal operator-mask bit: the evaluation feeds a local-search step, which
// applies the best move only when its delta is negative.  Lanes then start
// from the bound (delta 0, no id): moves with a positive delta are never
// evaluated in full, and the best improving move — the only one the step can
// apply — is found exactly as before.
constexpr uint32_t kImprovingOnly = 1u << 31;
// Operator-mask modifier (TGA_OP_COUNT_FULL, batched form): the evaluation
// launch is the instantiation that also counts the pairs evaluated in full.
constexpr uint32_t kCountFull = 1u << 17;
// Operator-mask modifier (TGA_OP_MULTI, general path): the evaluation also
// keeps, per pair of route slots, the best improving move touching exactly
// those routes (S.pairkey), for the selection of independent moves.
constexpr uint32_t kMulti = 1u << 18;

// Operator-mask modifier (TGA_OP_GRANULAR): inter-route operators restricted
// to the granular pairs of the instance.
constexpr uint32_t kGranular = 1u << 16;

__device__ __forceinline__ int initial_bound(uint32_t op_mask) {
    return (op_mask & kImprovingOnly) ? 0 : kAdmissibleBound;
}

// A local-search evaluation skips a solution that has converged (or reached
// its step cap); any other evaluation covers every solution, converged or not.
__device__ __forceinline__ bool skip_solution(const SolDev &S, uint32_t op_mask) {
    return (op_mask & kImprovingOnly) && S.state[kStDone];
}

__device__ __forceinline__ unsigned long long pack_key(int delta, uint32_t id) {
    return ((unsigned long long)((uint32_t)delta ^ 0x80000000u) << 32) | id;
}

__device__ __forceinline__ bool better(int d, uint32_t id, int bd, uint32_t bid) {
    return d < bd || (d == bd && id < bid);
}

__device__ __forceinline__ void consider(int d, uint32_t id, int &bd, uint32_t &bid) {
    if (d < kAdmissibleBound && better(d, id, bd, bid)) {
        bd = d;
        bid = id;
    }
}

__device__ __forceinline__ void wave_argmin(int &bd, uint32_t &bid) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const int od = __shfl_xor(bd, off);
        const uint32_t oid = (uint32_t)__shfl_xor((int)bid, off);
        if (better(od, oid, bd, bid)) {
            bd = od;
            bid = oid;
        }
    }
}

// One wavefront's best folded into the solution's key.
__device__ __forceinline__ void wave_argmin_commit(int bd, uint32_t bid, unsigned long long *key) {
    wave_argmin(bd, bid);
    if ((threadIdx.x & 63) == 0 && bd < kAdmissibleBound && bid != 0xFFFFFFFFu) atomicMin(key, pack_key(bd, bid));
}

// Reduce the per-lane bests of a workgroup and fold the result into the
// solution's key.  Every thread of the block must call it.
__device__ __forceinline__ void block_argmin_commit(int bd, uint32_t bid, unsigned long long *key,
                                    unsigned long long *red) {
    // (a wavefront that found nothing, most of them late in a search, has nothing to reduce)
    if (__builtin_amdgcn_ballot_w64(bid != 0xFFFFFFFFu)) wave_argmin(bd, bid);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) red[wave] = (bd >= kAdmissibleBound || bid == 0xFFFFFFFFu) ? ~0ull : pack_key(bd, bid);
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long m = ~0ull;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) m = red[w] < m ? red[w] : m;
        if (m != ~0ull) atomicMin(key, m);
    }
    __syncthreads();
}

// (duration, earliest finish, latest arrival) summary of a segment under hard
// windows: arriving at time a <= la, the segment is served and left at
// max(a + dur, ef).
struct Seg {
    int dur, ef, la;
    bool ok;
};

__device__ __forceinline__ Seg seg_node(int e, int l, int s) { return Seg{s, e + s, l, true}; }

// a then b, travelling c from the last node of a to the first node of b.
__device__ __forceinline__ Seg seg_cat(const Seg &a, int c, const Seg &b) {
    Seg r;
    r.dur = a.dur + c + b.dur;
    r.ef = max(a.ef + c + b.dur, b.ef);
    r.la = min(a.la, b.la - c - a.dur);
    r.ok = a.ok && b.ok && (a.ef + c <= b.la);
    return r;
}

// Arrive at `arr`; returns the departure time, or kInf when infeasible.
__device__ __forceinline__ int seg_pass(const Seg &g, int arr) {
    if (!g.ok || arr > g.la) return kInf;
    const int d = arr + g.dur;
    return d > g.ef ? d : g.ef;
}

// ------------------------------------------------------------ rebuild ------
// Segmented scans over the route-major slot array, one workgroup per
// solution.  Forward: prefix load and prefix distance (sums) and the earliest
// service start A (maps x -> x <= th ? max(x + al, be) : INF, closed under
// composition).  Backward: latest feasible arrival Z (maps
// y -> y >= th ? min(y + al, be) : NEG).  A reset flag marks a segment
// boundary (a route start for the forward scans, a route end for the
// backward scan).

struct FwdElem {
    int32_t rs;          // reset
    int32_t load, dist;  // additive parts
    int32_t th, al, be;  // A map
};

__device__ __forceinline__ FwdElem fwd_identity() { return FwdElem{0, 0, 0, kInf, 0, kNeg}; }

// apply a, then b
__device__ __forceinline__ FwdElem fwd_cat(const FwdElem &a, const FwdElem &b) {
    if (b.rs) return b;
    FwdElem r;
    r.rs = a.rs;
    r.load = a.load + b.load;
    r.dist = a.dist + b.dist;
    r.th = (a.be <= b.th) ? min(a.th, b.th - a.al) : -1;
    r.al = a.al + b.al;
    r.be = max(a.be + b.al, b.be);
    return r;
}

__device__ __forceinline__ int fwd_apply(const FwdElem &m, int x) {
    return (x <= m.th) ? max(x + m.al, m.be) : kInf;
}

struct BwdElem {
    int32_t rs, th, al, be;
};

__device__ __forceinline__ BwdElem bwd_identity() { return BwdElem{0, kNeg, 0, kInf}; }

// apply r (the part to the right) first, then l
__device__ __forceinline__ BwdElem bwd_cat(const BwdElem &l, const BwdElem &r) {
    if (l.rs) return l;
    BwdElem o;
    o.rs = r.rs;
    o.th = (r.be >= l.th) ? max(r.th, l.th - r.al) : kInf;
    o.al = r.al + l.al;
    o.be = min(r.be + l.al, l.be);
    return o;
}

__device__ __forceinline__ int bwd_apply(const BwdElem &m, int y) {
    return (y >= m.th) ? min(y + m.al, m.be) : kNeg;
}

struct ApplyShared {
    FwdElem fw[kApplyThreads / 64];
    BwdElem bw[kApplyThreads / 64];
    long long red[kApplyThreads / 64][8];
};

__device__ __forceinline__ FwdElem shfl_f(const FwdElem &e, int src) {
    return FwdElem{__shfl(e.rs, src), __shfl(e.load, src), __shfl(e.dist, src),
                   __shfl(e.th, src),  __shfl(e.al, src),   __shfl(e.be, src)};
}

__device__ __forceinline__ BwdElem shfl_b(const BwdElem &e, int src) {
    return BwdElem{__shfl(e.rs, src), __shfl(e.th, src), __shfl(e.al, src), __shfl(e.be, src)};
}

// Exclusive prefix (in thread order) of per-thread forward aggregates:
// wavefront shuffle scan, then a scan of the wavefront totals by wavefront 0.
__device__ __forceinline__ FwdElem block_prefix_fwd(FwdElem v, FwdElem *wtot) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    FwdElem x = v;
    for (int d = 1; d < 64; d <<= 1) {
        const FwdElem y = shfl_f(x, lane - d < 0 ? lane : lane - d);
        if (lane >= d) x = fwd_cat(y, x);
    }
    if (lane == 63) wtot[wave] = x;
    __syncthreads();
    if (wave == 0) {
        FwdElem w = lane < nw ? wtot[lane] : fwd_identity();
        for (int d = 1; d < 64; d <<= 1) {
            const FwdElem y = shfl_f(w, lane - d < 0 ? lane : lane - d);
            if (lane >= d) w = fwd_cat(y, w);
        }
        if (lane < nw) wtot[lane] = w;
    }
    __syncthreads();
    FwdElem ex = shfl_f(x, lane == 0 ? 0 : lane - 1);
    if (lane == 0) ex = fwd_identity();
    const FwdElem pre = wave > 0 ? wtot[wave - 1] : fwd_identity();
    const FwdElem r = fwd_cat(pre, ex);
    __syncthreads();
    return r;
}

// Exclusive suffix (aggregate of the threads after this one) of backward
// aggregates.
__device__ __forceinline__ BwdElem block_suffix_bwd(BwdElem v, BwdElem *wtot) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    BwdElem x = v;
    for (int d = 1; d < 64; d <<= 1) {
        const BwdElem y = shfl_b(x, lane + d > 63 ? lane : lane + d);
        if (lane + d < 64) x = bwd_cat(x, y);
    }
    if (lane == 0) wtot[wave] = x;
    __syncthreads();
    if (wave == 0) {
        BwdElem w = lane < nw ? wtot[lane] : bwd_identity();
        for (int d = 1; d < 64; d <<= 1) {
            const BwdElem y = shfl_b(w, lane + d > 63 ? lane : lane + d);
            if (lane + d < nw) w = bwd_cat(w, y);
        }
        if (lane < nw) wtot[lane] = w;
    }
    __syncthreads();
    BwdElem ex = shfl_b(x, lane == 63 ? 63 : lane + 1);
    if (lane == 63) ex = bwd_identity();
    const BwdElem post = wave < nw - 1 ? wtot[wave + 1] : bwd_identity();
    const BwdElem r = bwd_cat(ex, post);
    __syncthreads();
    return r;
}

// Forward element of slot s (reads what passes 1 and 2 wrote).
__device__ __forceinline__ FwdElem fwd_elem(const SolDev &S, const int32_t *roffn, int s) {
    const int4 a = gld(S.a4 + s);
    FwdElem e;
    if (s == gld(roffn + a.y)) {
        e = fwd_identity();
        e.rs = 1;
        return e;
    }
    const int4 ap = gld(S.a4 + s - 1);
    const int sp = gld(S.w4 + s - 1).z;
    const int4 w = gld(S.w4 + s);
    e.rs = 0;
    e.load = gld(S.b4 + s).x;
    e.dist = ap.z;
    e.al = sp + ap.z;
    e.th = w.y - e.al;
    e.be = w.x;
    return e;
}

__device__ __forceinline__ BwdElem bwd_elem(const SolDev &S, const int32_t *roffn, int s) {
    const int4 a = gld(S.a4 + s);
    const int4 w = gld(S.w4 + s);
    const int last = gld(roffn + a.y + 1) - 1;
    const int b = w.z + a.z;
    BwdElem e;
    e.rs = s == last;
    e.th = w.x + b;
    e.al = -b;
    e.be = w.y;
    return e;
}

// Terms a route of L customers adds to |N(S)| of RELOCATE, to twice that of
// 2OPT* (subtracted), to 2OPT and OR-OPT, and to the operator variants'
// counts (see kAccExtSeg).
struct RouteCounts {
    long long rel, star2, two, oropt, seg, k, k2;
};
__host__ __device__ __forceinline__ RouteCounts route_counts(long long L, long long Q) {
    RouteCounts c{L * (Q - L - 1), (L + 1) * (L + 1), L * (L - 1) / 2, 0, 0, 0, 0};
    for (int k = 1; k <= 3; ++k)
        if (k <= L) c.oropt += (L - k + 1) * (L - k);
    const long long more = L >= 2 ? 2 * L - 3 : 0;  // sum of k(x) - 1
    c.seg = more * (Q - L - 1);
    c.k = more + L;
    c.k2 = c.k * c.k - L * L;
    return c;
}

// Attributes of the slots [lo, hi) of the layout (nr, roffn), a union of
// whole routes, from their nodes (nr[ST * s] = {node, route} for slot s; it is
// then reused as scratch for the scans' A and Z), and those routes' distances.
// Requires blockDim.x == kApplyThreads.
template <int ST>
__device__ __forceinline__ void rebuild_range(const SolDev &S, int2 *nr, const int32_t *roffn, int lo, int hi,
                                              ApplyShared &sh) {
    const int n = S.n, np1 = S.np1;
    const int tid = threadIdx.x, T = blockDim.x;
    const int32_t *D = S.D;
    const int4 *nd = S.node4;
    const bool tw = S.has_tw;

    // pass 1: node, route, edge, per-node data, ref map
    for (int s = lo + tid; s < hi; s += T) {
        const int2 x = gld(nr + ST * s);
        const int node = x.x, r = x.y;
        const int first = gld(roffn + r), last = gld(roffn + r + 1) - 1;
        const int succ = s < last ? gld(nr + ST * (s + 1)).x : 0;
        int4 q = gld(nd + node);
        if (!tw) q = make_int4(q.x, 0, kTwOff, 0);
        const int edge = gld(D + (size_t)node * np1 + succ);
        const bool cust = s != first;
        gst(S.a4 + s, make_int4(node | ((cust ? kFlagCustomer : 0) << 16), r, edge, 0));
        gst(S.w4 + s, make_int4(q.y, q.z, q.w, S.pd && cust ? gld(S.pick + node) : 0));
        gst(S.b4 + s, make_int4(cust ? q.x : 0, 0, 0, 0));
        gst(S.ref2slot + (cust ? node - 1 : n + r), s);
    }
    __threadfence_block();
    __syncthreads();
    // pass 2: removal delta and incident-edge sums (customers)
    for (int s = lo + tid; s < hi; s += T) {
        int4 a = gld(S.a4 + s);
        if (s == gld(roffn + a.y)) continue;
        const int4 ap = gld(S.a4 + s - 1);
        const int succ = s + 1 < gld(roffn + a.y + 1) ? gld(nr + ST * (s + 1)).x : 0;
        const int dpw = gld(D + (size_t)nodeof(ap.x) * np1 + succ);
        a.w = dpw - ap.z - a.z;
        gst(S.a4 + s, a);
        int4 b = gld(S.b4 + s);
        b.w = ap.z + a.z;
        gst(S.b4 + s, b);
    }
    __threadfence_block();
    __syncthreads();

    const int C = (hi - lo + T - 1) / T;
    const int beg = min(hi, lo + tid * C), end = min(hi, beg + C);
    // forward scans: prefix load, prefix distance, earliest service start A
    {
        FwdElem agg = fwd_identity();
        for (int s = beg; s < end; ++s) agg = fwd_cat(agg, fwd_elem(S, roffn, s));
        FwdElem run = block_prefix_fwd(agg, sh.fw);
        const int e0 = tw ? gld(nd).y : 0;
        for (int s = beg; s < end; ++s) {
            run = fwd_cat(run, fwd_elem(S, roffn, s));
            int4 b = gld(S.b4 + s);
            b.y = run.load;
            gst(S.b4 + s, b);
            gst(S.pdist + s, run.dist);
            int2 z = gld(nr + ST * s);
            z.x = tw ? fwd_apply(run, e0) : 0;  // A[s]
            gst(nr + ST * s, z);
        }
    }
    __threadfence_block();
    __syncthreads();
    // backward scan: latest feasible arrival Z (windows only)
    if (!tw) {
        for (int s = beg; s < end; ++s) {
            int2 z = gld(nr + ST * s);
            z.y = kTwOff;
            gst(nr + ST * s, z);
        }
    } else {
        BwdElem agg = bwd_identity();
        for (int s = end - 1; s >= beg; --s) agg = bwd_cat(bwd_elem(S, roffn, s), agg);
        BwdElem run = block_suffix_bwd(agg, sh.bw);
        const int l0 = gld(nd).z;
        for (int s = end - 1; s >= beg; --s) {
            run = bwd_cat(bwd_elem(S, roffn, s), run);
            int2 z = gld(nr + ST * s);
            z.y = bwd_apply(run, l0);  // Z[s]
            gst(nr + ST * s, z);
        }
    }
    __threadfence_block();
    __syncthreads();
    // pass 3: route totals (by the thread owning each route's last slot)
    for (int s = lo + tid; s < hi; s += T) {
        const int r = gld(S.a4 + s).y;
        if (s == gld(roffn + r + 1) - 1) gst(S.rdist + r, gld(S.pdist + s) + gld(S.a4 + s).z);
    }
    // pass 4: derived per-slot values and flags
    const int l0 = tw ? gld(nd).z : kTwOff;
    const int cap = S.cap;
    for (int s = lo + tid; s < hi; s += T) {
        int4 a = gld(S.a4 + s);
        const int first = gld(roffn + a.y), last = gld(roffn + a.y + 1) - 1;
        const int rload = gld(S.b4 + last).y;
        const int4 w = gld(S.w4 + s);
        const int2 az = gld(nr + ST * s);
        const int A = az.x;
        const int dep = A >= kInf ? kInf : A + w.z;
        const int zn = s < last ? gld(nr + ST * (s + 1)).y : l0;
        int adp = kInf;
        int flags = flagsof(a.x);
        int4 b = gld(S.b4 + s);
        if (s != first) {
            const int Ap = gld(nr + ST * (s - 1)).x;
            adp = Ap >= kInf ? kInf : Ap + gld(S.w4 + s - 1).z;
            if (rload - b.x <= cap) flags |= kFlagRemCap;
            // without this node: predecessor departure + c(pred, succ) <= Z(succ)
            const int dpw = a.w + b.w;  // removal delta + incident edges = c(pred, succ)
            if (adp < kInf && adp + dpw <= zn) flags |= kFlagRemTw;
        }
        a.x = nodeof(a.x) | (flags << 16);
        gst(S.a4 + s, a);
        b.z = rload;
        gst(S.b4 + s, b);
        gst(S.t4 + s, make_int4(dep, zn, adp, az.y));
    }
    __threadfence_block();
    __syncthreads();
}

// Attributes of one slot of a route, as route_attr computes them.
struct SlotAttr {
    int4 a, b, t, w;
    int pdist, ref, rdist;  // rdist: the route's distance (lane L)
};

// The same attributes for one route of at most 64 slots, by one wavefront
// entirely in registers: lane p holds position p (p = 0 is the start depot,
// L customers follow; `node` is the lane's node).  The prefix load and
// distance and the two window maps are wavefront shuffle scans of the same
// elements the block scans use.  No memory is written.
__device__ __forceinline__ SlotAttr route_attr(const SolDev &S, int node, int r, int L) {
    const int lane = threadIdx.x & 63, np1 = S.np1;
    const int32_t *D = S.D;
    const bool tw = S.has_tw;
    const bool on = lane <= L;
    node = on ? node : 0;
    const int succ = __shfl(node, min(lane + 1, 63));
    const int nsucc = lane < L ? succ : 0;  // the route ends at the depot
    const int pred = __shfl(node, max(lane - 1, 0));
    const bool cust = lane >= 1 && on;
    int4 q = gld(S.node4 + node);
    const int4 q0 = gld(S.node4);
    const int edge = on ? gld(D + (size_t)node * np1 + nsucc) : 0;
    const int dpw = cust ? gld(D + (size_t)pred * np1 + nsucc) : 0;  // c(pred, succ)
    const int pick = S.pd && cust ? gld(S.pick + node) : 0;
    if (!tw) q = make_int4(q.x, 0, kTwOff, 0);
    const int demand = cust ? q.x : 0;
    const int epred = __shfl(edge, max(lane - 1, 0));
    const int spred = __shfl(q.w, max(lane - 1, 0));
    // forward elements (as fwd_elem): reset at the start depot
    FwdElem f;
    if (lane == 0 || !on) {
        f = fwd_identity();
        f.rs = lane == 0;
    } else {
        f.rs = 0;
        f.load = demand;
        f.dist = epred;
        f.al = spred + epred;
        f.th = q.z - f.al;
        f.be = q.y;
    }
    // a route of L + 1 slots needs only the scan steps below its length
    for (int d = 1; d <= L; d <<= 1) {
        const FwdElem y = shfl_f(f, lane - d < 0 ? lane : lane - d);
        if (lane >= d) f = fwd_cat(y, f);
    }
    int A = 0, Z = kTwOff;
    if (tw) {
        // backward elements (as bwd_elem): reset at the last slot
        BwdElem g;
        if (on) {
            const int b = q.w + edge;
            g.rs = lane == L;
            g.th = q.y + b;
            g.al = -b;
            g.be = q.z;
        } else {
            g = bwd_identity();
        }
        for (int d = 1; d <= L; d <<= 1) {
            const BwdElem y = shfl_b(g, lane + d > 63 ? lane : lane + d);
            if (lane + d < 64) g = bwd_cat(g, y);
        }
        A = fwd_apply(f, q0.y);
        Z = bwd_apply(g, q0.z);
    }
    const int l0 = tw ? q0.z : kTwOff;
    const int rload = __shfl(f.load, L);
    const int Zn = __shfl(Z, min(lane + 1, 63));
    const int Ap = __shfl(A, max(lane - 1, 0));
    const int dep = A >= kInf ? kInf : A + q.w;
    const int zn = lane < L ? Zn : l0;
    int adp = kInf;
    int flags = cust ? kFlagCustomer : 0;
    if (cust) {
        adp = Ap >= kInf ? kInf : Ap + spred;
        if (rload - demand <= S.cap) flags |= kFlagRemCap;
        if (adp < kInf && adp + dpw <= zn) flags |= kFlagRemTw;
    }
    SlotAttr x;
    x.a = make_int4(node | (flags << 16), r, edge, cust ? dpw - epred - edge : 0);
    x.b = make_int4(demand, f.load, rload, cust ? epred + edge : 0);
    x.w = make_int4(q.y, q.z, q.w, pick);
    x.t = make_int4(dep, zn, adp, Z);
    x.pdist = f.dist;
    x.ref = cust ? node - 1 : S.n + r;
    x.rdist = f.dist + edge;
    return x;
}

// Stores lane p's attributes (p <= L) at slot base + p, the reverse map and
// (lane L) the route's distance.
__device__ __forceinline__ void store_attr(const SolDev &S, const SlotAttr &x, int r, int base, int L) {
    const int lane = threadIdx.x & 63;
    if (lane > L) return;
    const int s = base + lane;
    gst(S.a4 + s, x.a);
    gst(S.b4 + s, x.b);
    gst(S.w4 + s, x.w);
    gst(S.t4 + s, x.t);
    gst(S.pdist + s, x.pdist);
    gst(S.ref2slot + x.ref, s);
    if (lane == L) gst(S.rdist + r, x.rdist);
}

// ------------------------------------------------------ penalised mode ---
// Time-warp summaries (Section 4.3.3): a subsequence sigma carries its
// duration T_D, earliest and latest start T_E / T_L and time warp T_V; a node
// is {s, e, l, 0}; two subsequences joined by an edge of travel time t
// concatenate as below (the garbled shift read as T_D(a) - T_V(a) + t).  A
// route's time warp is the T_V of depot, customers, depot.

struct Tw {
    int d, e, l, v;
};

__device__ __forceinline__ Tw tw_of(int4 x) { return Tw{x.x, x.y, x.z, x.w}; }
__device__ __forceinline__ int4 tw_pack(const Tw &x) { return make_int4(x.d, x.e, x.l, x.v); }
__device__ __forceinline__ Tw tw_node(int e, int l, int s) { return Tw{s, e, l, 0}; }

__device__ __forceinline__ Tw tw_cat(const Tw &a, int t, const Tw &b) {
    const int dt = a.d - a.v + t;
    const int dw = max(b.e - dt - a.l, 0);
    const int dv = max(a.e + dt - b.l, 0);
    return Tw{a.d + t + dw + b.d, max(a.e, b.e - dt) - dw, min(a.l, b.l - dt) + dv, a.v + dv + b.v};
}

__device__ __forceinline__ Tw tw_depot(const SolDev &S) {
    const int4 q = gld(S.node4);
    return tw_node(q.y, q.z, q.w);
}

// Load summaries (Section 4.3.2): {L_I delivered, L_O picked up, L_M the
// largest load on board}; a node is {d, p, max(d, p)}; concatenation keeps
// the later part's deliveries on board through the earlier part, and the
// earlier part's pickups through the later one.
struct Ld {
    int li, lo, lm;
};

__device__ __forceinline__ Ld ld_of(int4 x) { return Ld{x.x, x.y, x.z}; }
__device__ __forceinline__ int4 ld_pack(const Ld &x) { return make_int4(x.li, x.lo, x.lm, 0); }
__device__ __forceinline__ Ld ld_cat(const Ld &a, const Ld &b) {
    return Ld{a.li + b.li, a.lo + b.lo, max(a.lm + b.li, a.lo + b.lm)};
}
__device__ __forceinline__ Ld ld_node_at(const SolDev &S, int x) {
    const int d = gld(S.b4 + x).x, p = gld(S.w4 + x).w;
    return Ld{d, p, max(d, p)};
}

// The summaries of one route of at most 64 slots, by one wavefront in
// registers: lane p holds position p (`node` its node).  Concatenation is
// associative (exactly, in integers), so prefixes and suffixes are wavefront
// shuffle scans of single nodes, each carrying the edge that enters it.
__device__ __forceinline__ Tw shfl_tw(const Tw &x, int src) {
    return Tw{__shfl(x.d, src), __shfl(x.e, src), __shfl(x.l, src), __shfl(x.v, src)};
}

// Prefix (f) and suffix (b) time-warp summaries of the lanes 0..L.
__device__ __forceinline__ void tw_route_wave(const SolDev &S, int node, int L, Tw &f, Tw &b) {
    const int lane = threadIdx.x & 63, np1 = S.np1;
    const bool on = lane <= L;
    node = on ? node : 0;
    const int succ = __shfl(node, min(lane + 1, 63));
    const int4 q = gld(S.node4 + node), q0 = gld(S.node4);
    const int out = on ? gld(S.D + (size_t)node * np1 + (lane < L ? succ : 0)) : 0;  // edge leaving the lane's node
    int in = __shfl(out, max(lane - 1, 0));                                          // edge entering it
    const Tw dep = tw_node(q0.y, q0.z, q0.w);
    f = tw_node(q.y, q.z, q.w);
    b = lane == L ? tw_cat(f, out, dep) : f;  // the end depot closes the route
    int fin = in;
    for (int d = 1; d <= L; d <<= 1) {
        const int lo = max(lane - d, 0);
        const Tw y = shfl_tw(f, lo);
        const int yi = __shfl(fin, lo);
        if (lane >= d) {
            f = tw_cat(y, fin, f);
            fin = yi;
        }
    }
    for (int d = 1; d <= L; d <<= 1) {
        const int hi = min(lane + d, 63);
        const Tw y = shfl_tw(b, hi);
        const int yi = __shfl(in, hi);  // edge entering lane + d: the first node of the part to the right
        if (lane + d <= L) b = tw_cat(b, yi, y);
    }
}

// Prefix (f) and suffix (b) load summaries of the lanes 0..L (the start
// depot carries nothing).
__device__ __forceinline__ void ld_route_wave(const SolDev &S, int node, int L, Ld &f, Ld &b) {
    const int lane = threadIdx.x & 63;
    const bool cust = lane >= 1 && lane <= L;
    const int d0 = cust ? gld(S.node4 + node).x : 0, p0 = cust ? gld(S.pick + node) : 0;
    f = Ld{d0, p0, max(d0, p0)};
    b = f;
    for (int d = 1; d <= L; d <<= 1) {
        const int lo = max(lane - d, 0), hi = min(lane + d, 63);
        const Ld y{__shfl(f.li, lo), __shfl(f.lo, lo), __shfl(f.lm, lo)};
        const Ld z{__shfl(b.li, hi), __shfl(b.lo, hi), __shfl(b.lm, hi)};
        if (lane >= d) f = ld_cat(y, f);
        if (lane + d <= L) b = ld_cat(b, z);
    }
}

// Largest load on route r: the route load without pickups (kept in every
// slot's b4.z), the suffix summary's L_M at the start depot with them.
__device__ __forceinline__ int route_peak(const SolDev &S, int r) {
    const int off = gld(S.roff + r);
    return S.pd ? gld(S.ql4 + off).z : gld(S.b4 + off).z;
}

// Load excess of route r.
__device__ __forceinline__ int route_excess(const SolDev &S, int r) { return max(route_peak(S, r) - S.cap, 0); }

// Time warp of route r (the suffix summary at its start depot).
__device__ __forceinline__ int route_warp(const SolDev &S, int r) {
    return S.has_tw ? gld(S.pb4 + gld(S.roff + r)).w : 0;
}

// Removal deltas of the segments of two and three nodes that start at lane
// p's node (`node`, `edge`: the lanes' nodes and the edges leaving them; L
// customers follow the depot in lane 0); 0 where the route is too short.
__device__ __forceinline__ int2 segment_removal(const SolDev &S, int node, int edge, int L) {
    const int lane = threadIdx.x & 63, np1 = S.np1;
    const int pred = __shfl(node, max(lane - 1, 0)), epred = __shfl(edge, max(lane - 1, 0));
    const int n2 = __shfl(node, min(lane + 2, 63)), n3 = __shfl(node, min(lane + 3, 63));
    const int e1 = __shfl(edge, min(lane + 1, 63)), e2 = __shfl(edge, min(lane + 2, 63));
    int2 v = make_int2(0, 0);
    if (lane >= 1 && lane + 1 <= L) v.x = gld(S.D + (size_t)pred * np1 + (lane + 2 <= L ? n2 : 0)) - epred - e1;
    if (lane >= 1 && lane + 2 <= L) v.y = gld(S.D + (size_t)pred * np1 + (lane + 3 <= L ? n3 : 0)) - epred - e2;
    return v;
}

// The general path's summaries of route r (slots off .., L < 64 customers) by
// one wavefront: lane p's node and the edge leaving it, the route's load.
// peak and warp receive the route's largest load and time warp.
__device__ __forceinline__ void gen_route_wave(const SolDev &S, int off, int L, int node, int edge, int load, int &peak,
                                               int &warp) {
    const int lane = threadIdx.x & 63;
    const int2 rem = segment_removal(S, node, edge, L);
    peak = load;
    warp = 0;
    if (S.has_tw) {
        Tw f, b;
        tw_route_wave(S, node, L, f, b);
        if (lane <= L) {
            gst(S.pf4 + off + lane, tw_pack(f));
            gst(S.pb4 + off + lane, tw_pack(b));
        }
        warp = __shfl(b.v, 0);
    }
    if (S.pd) {
        Ld f, b;
        ld_route_wave(S, node, L, f, b);
        if (lane <= L) {
            gst(S.pl4 + off + lane, ld_pack(f));
            gst(S.ql4 + off + lane, ld_pack(b));
        }
        peak = __shfl(b.lm, 0);
    }
    if (lane <= L) gst(S.g4 + off + lane, make_int4(rem.x, rem.y, peak, warp));
}

// Removal deltas of the segments of two and three nodes that start at
// position p of the route whose slots begin at off (L customers), by one
// thread from the slots' attributes (as segment_removal).
__device__ __forceinline__ int2 slot_removal(const SolDev &S, int off, int p, int L) {
    int2 v = make_int2(0, 0);
    if (p < 1) return v;
    auto at = [&](int q) { return gld(S.a4 + off + min(q, L)); };
    const int4 ap = at(p - 1), a1 = at(p + 1), a2 = at(p + 2), a3 = at(p + 3);
    const int32_t *row = S.D + (size_t)nodeof(ap.x) * S.np1;
    const int d2 = gld(row + (p + 2 <= L ? nodeof(a2.x) : 0)), d3 = gld(row + (p + 3 <= L ? nodeof(a3.x) : 0));
    if (p + 1 <= L) v.x = d2 - ap.z - a1.z;
    if (p + 2 <= L) v.y = d3 - ap.z - a2.z;
    return v;
}

// gen_route_wave's prefix and suffix summaries of a route of 64 customers or
// more, by one wavefront: tiles of 64 positions, each scanned like a short
// route and joined to what the tiles before (after) it came to.  (One thread
// per route, a node after the other, took 1.3 ms for routes of 2000 customers
// and 0.1 ms for routes of 200.)
__device__ __forceinline__ void gen_route_long(const SolDev &S, int off, int L, int load, int &peak, int &warp) {
    const int lane = threadIdx.x & 63, last = L & ~63;
    peak = load;
    warp = 0;
    if (S.has_tw) {
        const Tw dep = tw_depot(S);
        Tw carry = dep;
        for (int t0 = 0; t0 <= L; t0 += 64) {
            const int p = min(t0 + lane, L);
            const int4 w = gld(S.w4 + off + p);
            int fin = gld(S.a4 + off + max(p - 1, 0)).z;  // edge entering the lane's node, then its tile's first
            Tw f = tw_node(w.x, w.y, w.z);
            for (int d = 1; d < 64; d <<= 1) {
                const int lo = max(lane - d, 0);
                const Tw y = shfl_tw(f, lo);
                const int yi = __shfl(fin, lo);
                if (lane >= d) {
                    f = tw_cat(y, fin, f);
                    fin = yi;
                }
            }
            if (t0 > 0) f = tw_cat(carry, fin, f);
            carry = shfl_tw(f, 63);
            if (t0 + lane <= L) gst(S.pf4 + off + p, tw_pack(f));
        }
        for (int t0 = last; t0 >= 0; t0 -= 64) {
            const int p = min(t0 + lane, L), end = min(63, L - t0);
            const int4 w = gld(S.w4 + off + p);
            const int in = gld(S.a4 + off + max(p - 1, 0)).z, out = gld(S.a4 + off + p).z;
            Tw b = tw_node(w.x, w.y, w.z);
            if (p == L) b = tw_cat(b, out, dep);  // the end depot closes the route
            for (int d = 1; d < 64; d <<= 1) {
                const int hi = min(lane + d, 63);
                const Tw y = shfl_tw(b, hi);
                const int yi = __shfl(in, hi);
                if (lane + d <= end) b = tw_cat(b, yi, y);
            }
            if (t0 < last) b = tw_cat(b, __shfl(out, 63), carry);
            carry = shfl_tw(b, 0);
            if (t0 + lane <= L) gst(S.pb4 + off + p, tw_pack(b));
        }
        warp = carry.v;
    }
    if (S.pd) {
        auto shfl_ld = [](const Ld &x, int src) { return Ld{__shfl(x.li, src), __shfl(x.lo, src), __shfl(x.lm, src)}; };
        Ld carry{0, 0, 0};
        for (int t0 = 0; t0 <= L; t0 += 64) {
            const int p = min(t0 + lane, L);
            Ld f = p ? ld_node_at(S, off + p) : Ld{0, 0, 0};
            for (int d = 1; d < 64; d <<= 1) {
                const Ld y = shfl_ld(f, max(lane - d, 0));
                if (lane >= d) f = ld_cat(y, f);
            }
            f = ld_cat(carry, f);
            carry = shfl_ld(f, 63);
            if (t0 + lane <= L) gst(S.pl4 + off + p, ld_pack(f));
        }
        carry = Ld{0, 0, 0};
        for (int t0 = last; t0 >= 0; t0 -= 64) {
            const int p = min(t0 + lane, L), end = min(63, L - t0);
            Ld b = p ? ld_node_at(S, off + p) : Ld{0, 0, 0};
            for (int d = 1; d < 64; d <<= 1) {
                const Ld z = shfl_ld(b, min(lane + d, 63));
                if (lane + d <= end) b = ld_cat(b, z);
            }
            b = ld_cat(b, carry);
            carry = shfl_ld(b, 0);
            if (t0 + lane <= L) gst(S.ql4 + off + p, ld_pack(b));
        }
        peak = carry.lm;
    }
}

// What gen_route_sums leaves for gen_slots and the totals: a route's largest
// load, time warp, first slot and customers.
struct GenRoute {
    int peak, warp, off, len;
};

// Summaries of route r by one wavefront, from its slots' attributes; g (LDS)
// receives its totals.  A long route's g4 is left to gen_slots.
__device__ __forceinline__ void gen_route_sums(const SolDev &S, int r, GenRoute &g) {
    const int lane = threadIdx.x & 63;
    const int off = gld(S.roff + r), L = gld(S.roff + r + 1) - off - 1, load = gld(S.b4 + off).z;
    int peak, warp;
    if (L < 64) {
        const int4 a = lane <= L ? gld(S.a4 + off + lane) : make_int4(0, 0, 0, 0);
        gen_route_wave(S, off, L, nodeof(a.x), a.z, load, peak, warp);
    } else {
        gen_route_long(S, off, L, load, peak, warp);
    }
    if (lane == 0) {
        g.peak = peak;
        g.warp = warp;
        g.off = off;
        g.len = L;
    }
}

// g4 of the slots [lo, hi) that belong to long routes (routes r0, r0 + 1, ..
// are entries 0, 1, .. of g), one thread per slot, four at a time.
__device__ __forceinline__ void gen_slots(const SolDev &S, const GenRoute *g, int r0, int lo, int hi) {
    constexpr int U = 4;
    const int T = blockDim.x;
    for (int s0 = lo + threadIdx.x; s0 < hi; s0 += T * U) {
        int4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = s0 + u * T;
            v[u].z = -1;
            if (s < hi) {
                const GenRoute &q = g[gld(S.a4 + s).y - r0];
                if (q.len >= 64) {
                    const int2 rem = slot_removal(S, q.off, s - q.off, q.len);
                    v[u] = make_int4(rem.x, rem.y, q.peak, q.warp);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (v[u].z >= 0) gst(S.g4 + s0 + u * T, v[u]);
    }
}

// Local-search state and counters of a solution, for a new run.
__device__ __forceinline__ void reset_run(const SolDev &S, int max_steps) {
    S.state[kStDone] = 0;
    S.state[kStSteps] = 0;
    S.state[kStStatus] = 0;
    S.state[kStMaxSteps] = max_steps;
    S.acc[kAccMoves] = 0;
    S.acc[kAccFullPairs] = 0;
    S.acc[kAccScreenPairs] = 0;
    S.acc[kAccMultiApplied] = 0;
    *S.best_key = ~0ull;
}

// Sums over the grid of the workgroups' sums (sum_sh, per wavefront): true for
// threads 0..2 of the last workgroup to finish, t their total; part[0] counts
// the workgroups and is back at zero then.  Every thread of the block calls it.
__device__ __forceinline__ bool grid_sums(const SolDev &S, long long (*sum_sh)[3], int &last_sh, long long &t) {
    __syncthreads();
    const int nb = gridDim.x;
    if (threadIdx.x == 0) {
        long long s[3] = {0, 0, 0};
        for (int w = 0; w < kBuildRoutes; ++w)
            for (int i = 0; i < 3; ++i) s[i] += sum_sh[w][i];
        for (int i = 0; i < 3; ++i) {
            sum_sh[0][i] = s[i];
            if (nb > 1)
                __hip_atomic_store(S.part + 1 + 3 * blockIdx.x + i, s[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        int last = 1;
        if (nb > 1) {
            __threadfence();
            last = atomicAdd((unsigned long long *)S.part, 1ull) == (unsigned long long)(nb - 1);
            __threadfence();
        }
        last_sh = last;
    }
    __syncthreads();
    if (!last_sh || threadIdx.x >= 3) return false;
    t = nb > 1 ? 0 : sum_sh[0][threadIdx.x];
    if (nb > 1)
        for (int b = 0; b < nb; ++b)
            t += __hip_atomic_load(S.part + 1 + 3 * b + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (threadIdx.x == 0) S.part[0] = 0;
    return true;
}

// Attributes of a new layout: route r holds cust[off[r] .. off[r + 1]).  One
// wavefront per route, every attribute in registers (route_attr) and, on the
// general path, the summaries; the totals are summed over the workgroup, and
// the last workgroup to finish adds up the others' (part[0] counts them).
// off and cust may lie in pinned host memory: each route is read once,
// straight from there, so that a new solution takes this one launch: 9 us (11
// with n up to 10^4) and one synchronisation, a reload 26 us of host time, in
// place of two copies, three launches and one workgroup that scanned all slots
// (20 us, 58 us), a reload 50 us.
// A workgroup that holds a route of 64 customers or more builds its slots by
// the block scans instead (rebuild_range, with the slots' own entries of pf4,
// which are not set yet, as scratch); the other workgroups' routes keep to
// their wavefronts.  A reload of 10^4 customers with one route of 64: 44 us
// (203 before the wavefront form, 242 when one workgroup took every slot and
// looked its route up in host memory).
// fresh: a solution set or reloaded by the host, which gives |N(S)|; its state
// and the route distance-block cache start empty.  Otherwise a multi-move
// step's layout (its launch keeps the counts), if there is one.  LONG: some
// route may hold 64 customers or more (the other instance has no code for
// that, which costs a reload of short routes 0.8 of its 29 us).
struct BuildCounts {
    long long cnt[5], seg, k, k2;
};

template <bool LONG>
__global__ __launch_bounds__(kBuildRoutes * 64) void k_build_routes(const SolDev S, const int32_t *__restrict__ off,
                                                                    const int32_t *__restrict__ cust, int fresh,
                                                                    const BuildCounts c) {
    __shared__ long long sum_sh[kBuildRoutes][3];
    __shared__ int last_sh;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = blockIdx.x * kBuildRoutes + wave, R = S.R, Q = S.Q;
    const bool gen = S.pen || S.pd || S.gen;
    const int build = fresh ? (LONG ? 2 : 1) : S.state[kStBuild];
    if (!build) return;  // uniform for the grid
    long long cost = 0, excess = 0, warps = 0;
    int c0 = 0, L = 0;
    if (r < R) {
        c0 = __builtin_amdgcn_readfirstlane(off[r]);
        L = __builtin_amdgcn_readfirstlane(off[r + 1]) - c0;
    }
    const int base = c0 + r;  // one start depot per route before it, and its own
    if (!LONG || build < 2 || !__syncthreads_or(L >= 64)) {
        if (r < R) {
            const int node = lane >= 1 && lane <= L ? cust[c0 + lane - 1] : 0;
            const SlotAttr x = route_attr(S, node, r, L);
            store_attr(S, x, r, base, L);
            cost = __shfl(x.rdist, L);
            if (gen) {
                int peak, warp;
                gen_route_wave(S, base, L, node, x.a.z, x.b.z, peak, warp);
                excess = max(peak - S.cap, 0);
                warps = warp;
            }
            if (lane == 0) gst(S.roff + r, base);
        }
    } else if constexpr (LONG) {
        __shared__ ApplyShared sh;
        __shared__ int base_sh[kBuildRoutes + 1];
        const int r0 = blockIdx.x * kBuildRoutes, r1 = min(r0 + kBuildRoutes, R);
        int2 *nr = (int2 *)S.pf4;
        if (r < R && lane == 0) {
            base_sh[wave] = base;
            gst(S.roff + r, base);
            if (r == r1 - 1) {
                base_sh[wave + 1] = base + L + 1;
                gst(S.roff + r1, base + L + 1);  // (the next workgroup writes the same)
            }
        }
        __syncthreads();
        const int lo = base_sh[0], hi = base_sh[r1 - r0];
        for (int s = lo + threadIdx.x; s < hi; s += kBuildRoutes * 64) {
            int k = 0;  // the slot's route, r0 + k
            for (int u = 1; u < r1 - r0; ++u) k += base_sh[u] <= s;
            gst(nr + 2 * s, make_int2(s == base_sh[k] ? 0 : cust[s - (r0 + k) - 1], r0 + k));
        }
        __threadfence_block();
        __syncthreads();
        rebuild_range<2>(S, nr, S.roff, lo, hi, sh);
        if (r < R) cost = gld(S.rdist + r);
        if (gen) {
            __shared__ GenRoute g[kBuildRoutes];
            if (r < R) {
                gen_route_sums(S, r, g[wave]);
                excess = max(g[wave].peak - S.cap, 0);
                warps = g[wave].warp;
            }
            __syncthreads();
            gen_slots(S, g, r0, lo, hi);
        }
    }
    if (r < R && lane == 0 && fresh) gst(S.rblk + (size_t)r * kRouteBlockWords, -1);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const bool tw = S.has_tw;
        const int4 q = gld(S.node4);
        gst(S.roff + R, Q);
        gst(S.a4 + Q, make_int4(0, R, 0, 0));
        gst(S.b4 + Q, make_int4(0, 0, 0, 0));
        gst(S.w4 + Q, make_int4(tw ? q.y : 0, tw ? q.z : kTwOff, 0, 0));
        gst(S.t4 + Q, make_int4(kInf, kNeg, kInf, kNeg));
        gst(S.pdist + Q, 0);
        if (fresh) {
            reset_run(S, 0);
            for (int i = 0; i < 5; ++i) S.acc[kAccCnt0 + i] = c.cnt[i];
            S.acc[kAccExtSeg] = c.seg;
            S.acc[kAccExtK] = c.k;
            S.acc[kAccExtK2] = c.k2;
            S.acc[kAccGranInter] = 0;
        }
    }
    if (lane == 0) {
        sum_sh[wave][0] = cost;
        sum_sh[wave][1] = excess;
        sum_sh[wave][2] = warps;
    }
    long long t;
    if (!grid_sums(S, sum_sh, last_sh, t)) return;
    if (threadIdx.x == 0) {
        S.acc[kAccCost] = t;
        S.state[kStBuild] = 0;
    } else if (gen) {
        S.acc[threadIdx.x == 1 ? kAccLoadExcess : kAccTimeWarp] = t;
    }
}

// Switch the general path on for a solution whose descriptor now says so:
// summaries of every route and the totals, kBuildRoutes routes a workgroup.
__global__ __launch_bounds__(kBuildRoutes * 64) void k_pen_init(const SolDev S) {
    __shared__ long long sum_sh[kBuildRoutes][3];
    __shared__ GenRoute g[kBuildRoutes];
    __shared__ int last_sh;
    if (!(S.pen || S.pd || S.gen)) return;  // uniform for the grid
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r0 = blockIdx.x * kBuildRoutes, r = r0 + wave, r1 = min(r0 + kBuildRoutes, S.R);
    if (r < S.R) gen_route_sums(S, r, g[wave]);
    if ((threadIdx.x & 63) == 0) {
        sum_sh[wave][0] = 0;
        sum_sh[wave][1] = r < S.R ? max(g[wave].peak - S.cap, 0) : 0;
        sum_sh[wave][2] = r < S.R ? g[wave].warp : 0;
    }
    if (__syncthreads_or(r < S.R && g[wave].len >= 64)) gen_slots(S, g, r0, gld(S.roff + r0), gld(S.roff + r1));
    long long t;
    if (grid_sums(S, sum_sh, last_sh, t) && threadIdx.x > 0) S.acc[threadIdx.x == 1 ? kAccLoadExcess : kAccTimeWarp] = t;
}

// The current routes as the caller's arrays: offsets (R + 1), customers (n),
// and the cost in front of them; out may lie in pinned host memory.
__global__ __launch_bounds__(256) void k_export(const SolDev S, int32_t *__restrict__ out) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    int32_t *offsets = out + 2, *customers = offsets + S.R + 1;
    if (s == 0) {
        *(long long *)out = S.acc[kAccCost];
        offsets[S.R] = S.n;
    }
    if (s >= S.Q) return;
    const int4 a = gld(S.a4 + s);
    if (flagsof(a.x) & kFlagCustomer) customers[s - a.y - 1] = nodeof(a.x);
    else offsets[a.y] = s - a.y;
}

// ------------------------------------------------------ inter-route eval ---
// One work item = rows [s0, s1) (slots, route-major) against every column
// slot of a later route.  For each unordered pair of slots (s, t) in
// different routes, route(s) < route(t), the fused pass evaluates
// RELOCATE s->after t, RELOCATE t->after s, SWAP s<->t and 2OPT*(s, t) (the
// node-based extraction of Section 5.3.1, eq. node_based1 and
// eq. node_based2, over the positional attributes).
//
// Rows stream through LDS in sub-blocks of S.tile_rows rows plus one halo row
// on each side, copied straight from HBM into LDS (global_load_lds).  A lane
// owns one column of a 62-column chunk and keeps its attributes in
// registers; per row it gathers D[row][node(t)] from LDS once and takes
// D[row][succ(t)] and D[row][pred(t)] from its neighbour lanes (DPP
// wavefront shifts), D[pred(s)][t] and D[succ(s)][t] from the previous and
// next row of a register window.

typedef __attribute__((address_space(3))) void *lds_void_ptr;
typedef __attribute__((address_space(1))) void *global_void_ptr;

// lane i receives lane i+1 (lane 63 receives 0)
__device__ __forceinline__ int from_next_lane(int v) { return __builtin_amdgcn_mov_dpp(v, 0x130, 0xF, 0xF, true); }
// lane i receives lane i-1 (lane 0 receives 0)
__device__ __forceinline__ int from_prev_lane(int v) { return __builtin_amdgcn_mov_dpp(v, 0x138, 0xF, 0xF, true); }

constexpr int kPenalty = 1 << 30;     // added to the delta of an inadmissible move
constexpr int kAdmissible = 1 << 29;  // every admissible delta is below this

// Column-side (lane) values of one chunk, kept in registers while the
// wavefront walks rows against it.  Every feasibility condition below is
// written as a difference that must be >= 0; "bad" values are 0 when a
// condition holds and negative otherwise, so OR-ing them keeps the sign of
// "any condition fails".
struct LaneCol {
    int4 ta, tb, tt, tw;
    int node;      // LDS gather index (node of slot t)
    int refT;
    int tyOwn;     // route(t) - 1 if the lane owns its column, else very negative
    int tInval;    // t is a start depot (cannot move): negative
    int tRemCap;   // t's route would exceed capacity without it... negative if not ok
    int tRemTw;    // t's route is late without it: negative
    int negTz, negTw;  // -edge(t), -(incident edges of t)
    int zx, zy;        // route load - demand, route load - prefix load of t
    // delta terms of the four moves with kPenalty added for a disabled
    // operator, for the delta-only pass
    int cRel, cRel2, cSwap, c2s;
};

// Raw column attributes of the chunk whose first owned column is slot cb
// (lanes 1..kColsPerWave own cb..cb+61; lanes 0 and 63 hold the
// neighbours), fetched ahead of their use.
struct ColRaw {
    int4 ta, tb, tt, tw;
};

// The slot arrays, their addresses read once per item.
struct SlotPtrs {
    const int4 *a4, *b4, *t4, *w4;
};

template <bool TW>
__device__ __forceinline__ ColRaw col_fetch(const SlotPtrs &P, int Q, int cb) {
    const int lane = threadIdx.x & 63;
    const int tc = min(max(cb - 1 + lane, 0), Q);
    ColRaw c;
    c.ta = gld(P.a4 + tc);
    c.tb = gld(P.b4 + tc);
    if (TW) {
        c.tt = gld(P.t4 + tc);
        c.tw = gld(P.w4 + tc);
    } else {
        c.tt = make_int4(0, 0, 0, 0);
        c.tw = make_int4(0, 0, 0, 0);
    }
    return c;
}

// Lane values of the chunk at cb from its raw attributes.  routeLast: route
// of the last owned column (-1 if none), wave-uniform.
__device__ __forceinline__ void col_setup(int Q, int n, int cb, const ColRaw &c, uint32_t op_mask, LaneCol &L,
                                          int &routeLast) {
    const int lane = threadIdx.x & 63;
    const int t = cb - 1 + lane;
    L.ta = c.ta;
    L.tb = c.tb;
    L.tt = c.tt;
    L.tw = c.tw;
    L.node = nodeof(L.ta.x);
    const int fl = flagsof(L.ta.x);
    const bool cust = fl & kFlagCustomer;
    const bool own = lane >= 1 && lane <= kColsPerWave && t < Q;
    L.refT = cust ? L.node - 1 : n + L.ta.y;
    L.tyOwn = own ? L.ta.y - 1 : -(1 << 30);
    L.tInval = cust ? 0 : (int)0x80000000;
    L.tRemCap = (fl & kFlagRemCap) ? 0 : (int)0x80000000;
    L.tRemTw = (fl & kFlagRemTw) ? 0 : (int)0x80000000;
    L.negTz = -L.ta.z;
    L.negTw = -L.tb.w;
    L.zx = L.tb.z - L.tb.x;
    L.zy = L.tb.z - L.tb.y;
    const int offRel = (op_mask & 1) ? 0 : (1 << 30);
    const int offSwap = (op_mask & 2) ? 0 : (1 << 30);
    const int off2s = (op_mask & 4) ? 0 : (1 << 30);
    L.cRel = L.negTz + offRel;
    L.cRel2 = L.ta.w + offRel;
    L.cSwap = L.negTw + offSwap;
    L.c2s = L.negTz + off2s;
    const int lastLane = min(kColsPerWave, Q - cb);
    routeLast = lastLane >= 1 ? __builtin_amdgcn_readlane(L.ta.y, lastLane) : -1;
}

// ---- LDS block of distance rows of an inter-route item.  While the rows of
// a sub-block starting at row sb are evaluated, slot x (sb - 1 <= x <= the
// sub-block's last row + 1) sits at row position x - sb + 1; slots outside
// [0, Q] are read clamped.

// Distance rows of slots [x0, x0 + cnt) copied straight from HBM into the
// block (global_load_lds, four dwords per lane for 16-bit rows, else one),
// slot `base` at position 0,
// from the 16-bit copy of D when W16.  The issuing wavefront must wait
// (vmcnt) before a barrier publishes them.  `wave` is the wavefront index
// (uniform).
template <bool W16>
__device__ __forceinline__ void drow_issue(const SolDev &S, const int4 *a4, int Q, void *rows, int base, int x0,
                                           int cnt, int wave) {
    const int lane = threadIdx.x & 63;
    const int stride = W16 ? S.stride16 : S.np1;  // elements per row
    const int words = W16 ? stride / 2 : stride;  // dwords per row
    const char *const D = W16 ? (const char *)S.D16 : (const char *)S.D;
    // lane k: the node of this wavefront's k-th row (cnt <= 64 * kInterWaves),
    // read together: a scalar read per row had each row wait for the last
    const int nodes = nodeof(gld(&a4[min(max(x0 + min(wave + lane * kInterWaves, cnt - 1), 0), Q)].x));
    for (int r = wave, k = 0; r < cnt; r += kInterWaves, ++k) {
        const int x = x0 + r;
        const int node = __builtin_amdgcn_readlane(nodes, k);
        const int *src = (const int *)(D + (size_t)node * stride * (W16 ? 2 : 4));
        int *dst = (int *)rows + (x - base) * words;
        if (W16) {  // rows are 16-byte aligned multiples of 16 bytes: four dwords per lane
            for (int c = 0; c < words; c += 256) {
                if (c + 4 * lane < words)
                    __builtin_amdgcn_global_load_lds((global_void_ptr)(src + c + 4 * lane), (lds_void_ptr)(dst + c), 16,
                                                     0, 0);
            }
        } else {
            for (int c = 0; c < words; c += 64) {
                if (c + lane < words)
                    __builtin_amdgcn_global_load_lds((global_void_ptr)(src + c + lane), (lds_void_ptr)(dst + c), 4, 0,
                                                     0);
            }
        }
    }
}

template <bool W16> struct DistElem { typedef int type; };
template <> struct DistElem<true> { typedef uint16_t type; };

constexpr int kSign = (int)0x80000000;

// delta, plus kPenalty when viol < 0
__device__ __forceinline__ int penalise(int d, int viol) {
    return d + (int)(((uint32_t)viol >> 31) << 30);
}

// Row-side (scalar) values of one row slot s.
struct RowVals {
    int rs, refS;
    int sInval, sRemCap, sRemTw;   // 0 or negative, as the lane's
    int capA, capB, capC, capD, capE;
    int rw_ra, rz;                 // removal delta of s, edge(s)
    int rbw;                       // incident edges of s
};

__device__ __forceinline__ RowVals row_vals(const int4 &ra, const int4 &rb, int cap, int n) {
    RowVals R;
    const int fl = flagsof(ra.x);
    const bool cust = fl & kFlagCustomer;
    R.rs = ra.y;
    R.refS = cust ? nodeof(ra.x) - 1 : n + ra.y;
    R.sInval = cust ? 0 : kSign;
    R.sRemCap = (fl & kFlagRemCap) ? 0 : kSign;
    R.sRemTw = (fl & kFlagRemTw) ? 0 : kSign;
    R.capA = cap - rb.x;          // relocate s->t: load(t) <= capA; swap: load(t) - dem(t) <= capA
    R.capB = cap - rb.z;          // relocate t->s: dem(t) <= capB
    R.capC = cap - rb.z + rb.x;   // swap: dem(t) <= capC
    R.capD = cap - rb.y;          // 2-opt*: load(t) - prefix(t) <= capD
    R.capE = cap - rb.z + rb.y;   // 2-opt*: prefix(t) <= capE
    R.rw_ra = ra.w;
    R.rz = ra.z;
    R.rbw = rb.w;
    return R;
}

// The four inter-route moves of row slot s against the lane's column slot t:
// RELOCATE s -> after t, RELOCATE t -> after s, SWAP s <-> t, 2OPT*(s, t).
// g = D[s][t], gp = D[pred(s)][t], gn = D[succ(s)][t], gR = D[s][succ(t)],
// gL = D[s][pred(t)].  rt / rw: the row's time values and window (TW only).
template <bool TW, bool DUMP>
__device__ __forceinline__ void pair_moves(const LaneCol &L, const RowVals &R, const int4 &rt, const int4 &rw,
                                           int gp, int g, int gn, int gR, int gL, uint32_t uQ, bool opRel,
                                           bool opSwap, bool op2s, int32_t *__restrict__ dump_delta,
                                           uint8_t *__restrict__ dump_feas, int &bd, uint32_t &bid) {
    const int4 ta = L.ta, tb = L.tb, tt = L.tt, tw = L.tw;
    const int pairViol = L.tyOwn - R.rs;  // >= 0 iff the lane owns t and route(t) > route(s)

    // RELOCATE s -> right after t
    const int d1 = g + gR + L.negTz + R.rw_ra;
    const int cap1 = R.capA - tb.z;
    int tw1 = 0;
    if (TW) {
        const int arr = tt.x + g;
        const int st = max(arr, rw.x);
        tw1 = (rw.y - arr) | ((tt.y - rw.z) - (st + gR)) | R.sRemTw;
    }
    const int v1 = pairViol | R.sInval;
    const int e1 = penalise(d1, v1 | cap1 | R.sRemCap | tw1);

    // RELOCATE t -> right after s
    const int d2 = g + gn + ta.w - R.rz;
    const int cap2 = R.capB - tb.x;
    int tw2 = 0;
    if (TW) {
        const int arr = rt.x + g;
        const int st = max(arr, tw.x);
        tw2 = (tw.y - arr) | (rt.y - (st + tw.z + gn)) | L.tRemTw;
    }
    const int v2 = pairViol | L.tInval;
    const int e2 = penalise(d2, v2 | cap2 | L.tRemCap | tw2);

    // SWAP s <-> t
    const int d3 = gp + gn + gL + gR + L.negTw - R.rbw;
    const int cap3 = (R.capC - tb.x) | (R.capA - L.zx);
    int tw3 = 0;
    if (TW) {
        const int arrS = rt.z + gp;  // t placed where s was
        const int stS = max(arrS, tw.x);
        const int arrT = tt.z + gL;  // s placed where t was
        const int stT = max(arrT, rw.x);
        tw3 = (tw.y - arrS) | (rt.y - (stS + tw.z + gn)) | (rw.y - arrT) | (tt.y - (stT + rw.z + gR));
    }
    const int v3 = pairViol | R.sInval | L.tInval;
    const int e3 = penalise(d3, v3 | cap3 | tw3);

    // 2OPT*(s, t): heads keep their slots, tails are exchanged
    const int d4 = gR + gn + L.negTz - R.rz;
    const int cap4 = (R.capD - L.zy) | (R.capE - tb.y);
    int tw4 = 0;
    if (TW) tw4 = ((tt.y - gR) - rt.x) | ((rt.y - gn) - tt.x);
    const int e4 = penalise(d4, pairViol | cap4 | tw4);

    const uint32_t lo = min((uint32_t)R.refS, (uint32_t)L.refT), hi = max((uint32_t)R.refS, (uint32_t)L.refT);
    if (DUMP) {
        // exact feasibility bits of every valid move
        if (opRel && v1 >= 0) {
            const uint32_t id = (uQ + R.refS) * uQ + L.refT;
            dump_delta[id] = d1;
            dump_feas[id] = (uint8_t)(((cap1 | R.sRemCap) >= 0) | ((tw1 >= 0) << 1));
        }
        if (opRel && v2 >= 0) {
            const uint32_t id = (uQ + L.refT) * uQ + R.refS;
            dump_delta[id] = d2;
            dump_feas[id] = (uint8_t)(((cap2 | L.tRemCap) >= 0) | ((tw2 >= 0) << 1));
        }
        if (opSwap && v3 >= 0) {
            const uint32_t id = (5u * uQ + lo) * uQ + hi;
            dump_delta[id] = d3;
            dump_feas[id] = (uint8_t)((cap3 >= 0) | ((tw3 >= 0) << 1));
        }
        if (op2s && pairViol >= 0) {
            const uint32_t id = (8u * uQ + lo) * uQ + hi;
            dump_delta[id] = d4;
            dump_feas[id] = (uint8_t)((cap4 >= 0) | ((tw4 >= 0) << 1));
        }
    }
    const int m1 = opRel ? e1 : kNoDelta;
    const int m2 = opRel ? e2 : kNoDelta;
    const int m3 = opSwap ? e3 : kNoDelta;
    const int m4 = op2s ? e4 : kNoDelta;
    const int m = min(min(m1, m2), min(m3, m4));
    if (m <= bd) {  // rare: only an admissible move can reach bd (< kAdmissible)
        consider(m1, (uQ + R.refS) * uQ + L.refT, bd, bid);
        consider(m2, (uQ + L.refT) * uQ + R.refS, bd, bid);
        consider(m3, (5u * uQ + lo) * uQ + hi, bd, bid);
        consider(m4, (8u * uQ + lo) * uQ + hi, bd, bid);
    }
}

// Delta of the best admissible move committed so far for S (kAdmissibleBound
// if none): every workgroup working on S may skip moves that cannot beat it.
__device__ __forceinline__ int committed_delta(const SolDev &S) {
    const unsigned long long k = __hip_atomic_load(S.best_key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return k == ~0ull ? kAdmissibleBound : (int)((uint32_t)(k >> 32) ^ 0x80000000u);
}

// Whole-workgroup evaluation of one inter-route item: the row slots
// [s0, s1) against every column slot after the row.  The distance rows
// (16-bit when W16) are staged in LDS in sub-blocks of h = S.tile_rows rows
// plus a halo row on each side (one sub-block per item by default); row
// attributes are wave-uniform and come through the scalar cache, one row
// ahead of their use.  The (column chunk, row) pairs of a
// sub-block are split into kInterWaves equal contiguous runs, chunk-major, so
// every wavefront gets the same work whatever the shape of the triangle; the
// column attributes of a wavefront's next run are fetched while the current
// one is evaluated.
//
// Each pair first gets the deltas of its four moves only; the feasibility
// conditions and move ids are evaluated only where some delta is <= the
// run's threshold: the best any wavefront of the workgroup has published in
// LDS (thr_sh, read at the start of a run; each wavefront publishes its own
// best at the end of a run) or the solution has committed, bounded by the
// initial bound.  Every threshold is the delta of an admissible move of this
// neighbourhood (or the bound), so no move that could be the minimum (or tie
// with it) is ever skipped.
// With dump arrays every move is evaluated.  smem4 is the dynamic LDS area,
// free when the call starts; red holds kInterWaves keys (BATCH: unused).
//
// Per item the time goes to chains, not to bytes or instructions: of 12 us for
// about 18 rows of 2000 columns, 2.7 until the rows are in LDS, 6 for some 40
// passes per wavefront, 2.5 for its barriers and the commit.  Hence the rows'
// nodes in one read (each row's own scalar read waited for the one before),
// the next chunk's columns fetched on one path only (where two paths met, the
// wait for this run's columns became one for the next run's), no read for the
// rows' routes, and for a batch a commit without barriers: the evaluation
// launch of 256 solutions of 100..2000 customers 165 -> 150 us, of one of
// 1000 (CVRP) 11.1 -> 10.7 us.  (Fewer instructions per pass gained nothing:
// four rows at a time without a branch 164 us, 13 instead of 17 vector
// instructions 154.)
template <bool TW, bool DUMP, bool W16, bool CNT = false, bool BATCH = false>
__device__ __forceinline__ void inter_item(const SolDev &S, const InterItem &item, uint32_t op_mask,
                           int32_t *__restrict__ dump_delta, uint8_t *__restrict__ dump_feas,
                           int4 *smem4, unsigned long long *red, int *thr_sh) {
    typedef typename DistElem<W16>::type DT;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const bool opRel = op_mask & 1, opSwap = op_mask & 2, op2s = op_mask & 4;
    const int Q = S.Q, np1 = S.np1, n = S.n, cap = S.cap, h = S.tile_rows;
    const uint32_t uQ = (uint32_t)Q;
    const SlotPtrs P{S.a4, S.b4, S.t4, S.w4};
    const int s0 = item.s0, s1 = item.s1;
    const int nsb = (s1 - s0 + h - 1) / h;
    const int NB = h + 2;
    const int rs = W16 ? S.stride16 : np1;  // row stride in LDS (elements)
    DT *rows = (DT *)smem4;
    const DT *rowsLast = rows + (NB - 1) * rs;  // the last row position

    int bd = initial_bound(op_mask);
    uint32_t bid = 0xFFFFFFFFu;
    uint32_t nfull = 0;  // CNT: this wavefront's pairs evaluated in full (wave-uniform)

    // this wavefront's share of the sub-block: (chunk, row) pairs from chunk j,
    // row r0 on, `left` of them; the first chunk's column attributes; lane k:
    // the route of the sub-block's k-th row (at most 64 rows)
    int j = 0, r0 = 0, left = 0, rowRoute = 0;
    ColRaw nxt;
    // everything a sub-block reads besides its distance rows, together with them
    auto sub_block = [&](int sb, int nr) {
        const int T = max(0, (Q - sb - 1 + kColsPerWave - 1) / kColsPerWave) * nr;  // below 2^14
        const int lo = T * wave / kInterWaves;
        left = T * (wave + 1) / kInterWaves - lo;
        j = lo / nr;
        r0 = lo - j * nr;
        rowRoute = gld(&P.a4[sb + min(lane, nr - 1)].y);
        nxt = col_fetch<TW>(P, Q, sb + 1 + j * kColsPerWave);
    };

    // prologue: the distance rows of sub-block 0 (with its halo rows)
    if (!DUMP && threadIdx.x == 0) *thr_sh = committed_delta(S);
    drow_issue<W16>(S, P.a4, Q, rows, s0 - 1, s0 - 1, min(h, s1 - s0) + 2, wave);
    sub_block(s0, min(h, s1 - s0));
    __builtin_amdgcn_s_waitcnt(0);
    for (int i = 0; i < nsb; ++i) {
        const int sb = s0 + i * h;
        const int nr = min(h, s1 - sb);  // rows of this sub-block
        __syncthreads();                 // rows of sub-block i resident (i = 0), or i - 1 consumed
        if (i > 0) {
            // The previous sub-block (h rows) ended with rows sb - 1 and sb
            // at positions h and h + 1: they become this one's first halo
            // row and first row, so only rows sb + 1 .. sb + nr come from
            // memory and a strip of sub-blocks reads each row once.
            {
                const int words = (int)((size_t)rs * sizeof(DT) / 4);  // dwords per row
                int *blk = (int *)rows;
                const int *from = blk + h * words;
                if (h >= 2) {  // positions h, h + 1 and 0, 1 do not overlap
                    for (int w = threadIdx.x; w < 2 * words; w += blockDim.x) blk[w] = from[w];
                } else {  // position 1 is source and destination: read a chunk, wait, write it
                    for (int w0 = 0; w0 < 2 * words; w0 += blockDim.x) {
                        const int w = w0 + threadIdx.x;
                        const int v = w < 2 * words ? from[w] : 0;
                        __syncthreads();
                        if (w < 2 * words) blk[w] = v;
                        __syncthreads();
                    }
                }
            }
            __syncthreads();
            drow_issue<W16>(S, P.a4, Q, rows, sb - 1, sb + 1, nr, wave);
            sub_block(sb, nr);
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
        }
        // columns: every slot after the sub-block's first row (pairs in the
        // same route are skipped per pair).  Runs = (chunk j, rows [r0, r1));
        // every run after the first of a share starts the next chunk at row 0.
        if (left > 0) {
            for (; left > 0; ++j, r0 = 0) {
                const int r1 = min(nr, r0 + left);
                left -= r1 - r0;
                const int cb = sb + 1 + j * kColsPerWave;
                // the next run's chunk is fetched while this one is evaluated
                const ColRaw cur = nxt;
                if (left > 0) nxt = col_fetch<TW>(P, Q, cb + kColsPerWave);
                LaneCol L;
                int routeLast;
                col_setup(Q, n, cb, cur, op_mask, L, routeLast);
                int x = sb + r0;  // row slot
                // rows whose route precedes the chunk's last route (slots are
                // route-major, so they come first), at most up to the end of
                // the run
                const int before = (int)__builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < nr && rowRoute < routeLast));
                const int xlim = sb + min(r1, before);
                // register window over the distance rows: x - 1, x, x + 1
                const DT *pp = rows + (x - sb) * rs;
                int gp = pp[L.node];
                pp += rs;
                int g = pp[L.node];
                pp += rs;
                int gn = pp[L.node];
                uint32_t ro = (uint32_t)x * 16u;  // byte offset of row x's slot attributes
                int4 ra = sld_at(P.a4, ro), rb = sld_at(P.b4, ro);
                const int thrRun = DUMP ? 0 : __hip_atomic_load(thr_sh, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                // The passes screen against the run's threshold alone (the delta
                // of an admissible move, or the initial bound): a lane's own
                // better move found during the run tightens it only from the
                // next run, which saves an instruction per pass and lets a few
                // more pairs into the full evaluation.
                const int thrScreen = min(thrRun, initial_bound(op_mask));
                // Each pass first consumes what the previous one fetched, then
                // fetches row x + 1 (attributes) and the gather of row x + 2,
                // then evaluates row x from registers (the rare full
                // evaluation also reads the row's time attributes).  Passes
                // go in fours so that the two sets of row attributes and the
                // four window registers take turns without copies.
                auto pass = [&](const int4 &rA, const int4 &rB, int4 &rAn, int4 &rBn, int wp, int w0, int wn,
                                int &wnn) {
                    pp = min(pp + rs, rowsLast);
                    wnn = pp[L.node];  // row x + 2 (past the halo on the last row: unused)
                    rAn = sld_at(P.a4, ro + 16u);  // x + 1 <= Q
                    rBn = sld_at(P.b4, ro + 16u);
                    const int gR = from_next_lane(w0);  // D[s][succ(t)]
                    const int gL = from_prev_lane(w0);  // D[s][pred(t)]
                    bool full = true;
                    if (!DUMP) {
                        const int thr = thrScreen;
                        const int wz = wn - rA.z;  // shared by RELOCATE t -> s and 2OPT*
                        const int d1 = w0 + gR + (L.cRel + rA.w);
                        const int d2 = w0 + wz + L.cRel2;
                        const int d3 = (wp + wn) + gL + (gR + (L.cSwap - rB.w));
                        const int d4 = gR + wz + L.c2s;
                        const int m = min(min(d1, d2), min(d3, d4));
                        full = m <= thr && L.tyOwn >= rA.y;
                        if (full) {
                            // capacity screen: a move whose capacity condition
                            // fails is inadmissible whatever its delta (most
                            // screened-in moves late in a search are such)
                            const int capA = cap - rB.x, capB = cap - rB.z;
                            const int e1 = (capA - L.tb.z) >= 0 ? d1 : kNoDelta;
                            const int e2 = (capB - L.tb.x) >= 0 ? d2 : kNoDelta;
                            const int e3 = ((capB + rB.x - L.tb.x) | (capA - L.zx)) >= 0 ? d3 : kNoDelta;
                            const int e4 = ((cap - rB.y - L.zy) | (capB + rB.y - L.tb.y)) >= 0 ? d4 : kNoDelta;
                            full = min(min(e1, e2), min(e3, e4)) <= thr;
                        }
                        if (CNT) nfull += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(full));
                    }
                    if (full) {
                        int4 rt = make_int4(0, 0, 0, 0), rw = make_int4(0, 0, 0, 0);
                        if (TW) {
                            rt = sld_at(P.t4, ro);
                            rw = sld_at(P.w4, ro);
                        }
                        const RowVals R = row_vals(rA, rB, cap, n);
                        pair_moves<TW, DUMP>(L, R, rt, rw, wp, w0, wn, gR, gL, uQ, opRel, opSwap, op2s, dump_delta,
                                             dump_feas, bd, bid);
                    }
                    ++x;
                    ro += 16u;
                };
                int4 ra2, rb2;
                int g3 = 0;
                // four passes per iteration: the four window registers take
                // turns, so the window is back in gp, g, gn without copies
                for (int q = (xlim - x) >> 2; q > 0; --q) {  // whole groups of four rows
                    pass(ra, rb, ra2, rb2, gp, g, gn, g3);  // rows x - 1, x, x + 1; fetches x + 2
                    pass(ra2, rb2, ra, rb, g, gn, g3, gp);
                    pass(ra, rb, ra2, rb2, gn, g3, gp, g);
                    pass(ra2, rb2, ra, rb, g3, gp, g, gn);
                }
                if (x < xlim) {  // the last one to three rows
                    pass(ra, rb, ra2, rb2, gp, g, gn, g3);
                    if (x < xlim) {
                        pass(ra2, rb2, ra, rb, g, gn, g3, gp);
                        if (x < xlim) pass(ra, rb, ra2, rb2, gn, g3, gp, g);
                    }
                }
                // publish this wavefront's best to the workgroup (one lane, one
                // LDS atomic, only when some lane improved on the shared value)
                if (!DUMP && __builtin_amdgcn_ballot_w64(bd < thrRun)) {
                    int wmin = bd;
#pragma unroll
                    for (int off = 32; off >= 1; off >>= 1) wmin = min(wmin, __shfl_xor(wmin, off));
                    if (lane == 0) atomicMin(thr_sh, wmin);
                }
            }
        }
    }
    if (CNT && !DUMP && (op_mask & kImprovingOnly) && lane == 0 && nfull)
        atomicAdd((unsigned long long *)(S.acc + kAccFullPairs), (unsigned long long)nfull);
    if (BATCH) {
        // an item of many: a wavefront commits by itself, without the
        // workgroup's barriers, and only what is still the workgroup's best
        const int best = __hip_atomic_load(thr_sh, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (__builtin_amdgcn_ballot_w64(bid != 0xFFFFFFFFu && bd <= best)) wave_argmin_commit(bd, bid, S.best_key);
    } else {
        block_argmin_commit(bd, bid, S.best_key, red);
    }
}

// ------------------------------------------- granular inter-route eval ---
// Edge-based extraction (Section 5.3.1): only the node pairs kept by the
// granular mask, the symmetric closure of each node's theta nearest
// neighbours, get their inter-route moves evaluated.  The mask is a list of
// pairs of customers, each pair once, and of the customers paired with the
// depot, which stands for the start depot of every route.  One thread per
// pair (u, v): the slot of the route that comes first is the row (as in the
// full kernel, row route < column route); one thread per (customer paired
// with the depot, route): the customer against that route's start depot.
// Attributes are gathered per thread (no LDS staging): E is small next to
// the Q^2 pairs of the full neighbourhood.

// Column attributes of slot t for one thread (the fields pair_moves reads).
__device__ __forceinline__ void lane_col_single(const SolDev &S, int t, LaneCol &L) {
    L.ta = gld(S.a4 + t);
    L.tb = gld(S.b4 + t);
    if (S.has_tw) {
        L.tt = gld(S.t4 + t);
        L.tw = gld(S.w4 + t);
    } else {
        L.tt = make_int4(0, 0, 0, 0);
        L.tw = make_int4(0, 0, 0, 0);
    }
    L.node = nodeof(L.ta.x);
    const int fl = flagsof(L.ta.x);
    const bool cust = fl & kFlagCustomer;
    L.refT = cust ? L.node - 1 : S.n + L.ta.y;
    L.tyOwn = L.ta.y - 1;
    L.tInval = cust ? 0 : (int)0x80000000;
    L.tRemCap = (fl & kFlagRemCap) ? 0 : (int)0x80000000;
    L.tRemTw = (fl & kFlagRemTw) ? 0 : (int)0x80000000;
    L.negTz = -L.ta.z;
    L.negTw = -L.tb.w;
    L.zx = L.tb.z - L.tb.x;
    L.zy = L.tb.z - L.tb.y;
}

// The four inter-route moves of row slot x against column slot t (route(x)
// < route(t)), with every attribute gathered from the slot arrays and D.
// Returns the number of moves of N_theta(S) the pair stands for.
template <bool TW, bool DUMP>
__device__ __forceinline__ int gran_pair(const SolDev &S, int x, int t, uint32_t op_mask,
                                         int32_t *__restrict__ dump_delta, uint8_t *__restrict__ dump_feas,
                                         int &bd, uint32_t &bid) {
    const bool opRel = op_mask & 1, opSwap = op_mask & 2, op2s = op_mask & 4;
    LaneCol L;
    lane_col_single(S, t, L);
    const int4 ra = gld(S.a4 + x), rb = gld(S.b4 + x);
    int4 rt = make_int4(0, 0, 0, 0), rw = make_int4(0, 0, 0, 0);
    if (TW) {
        rt = gld(S.t4 + x);
        rw = gld(S.w4 + x);
    }
    const RowVals R = row_vals(ra, rb, S.cap, S.n);
    const int np1 = S.np1;
    const int nx = nodeof(ra.x), npx = nodeof(gld(S.a4 + max(x - 1, 0)).x), nsx = nodeof(gld(S.a4 + x + 1).x);
    const int nt = L.node, npt = nodeof(gld(S.a4 + t - 1).x), nst = nodeof(gld(S.a4 + t + 1).x);
    const int32_t *D = S.D;
    const int g = gld(D + (size_t)nx * np1 + nt), gp = gld(D + (size_t)npx * np1 + nt),
              gn = gld(D + (size_t)nsx * np1 + nt), gR = gld(D + (size_t)nx * np1 + nst),
              gL = gld(D + (size_t)nx * np1 + npt);
    pair_moves<TW, DUMP>(L, R, rt, rw, gp, g, gn, gR, gL, (uint32_t)S.Q, opRel, opSwap, op2s, dump_delta,
                         dump_feas, bd, bid);
    const bool cx = R.sInval == 0, ct = L.tInval == 0;
    return (opRel ? (int)cx + (int)ct : 0) + (opSwap && cx && ct ? 1 : 0) + (op2s ? 1 : 0);
}

// The granular pairs of an instance (device lists).
struct GranPairs {
    const int32_t *src, *adj, *dep;  // gcc pairs of customers; gdep customers paired with the depot
    int gcc, gdep;
};

// Work items: e < gcc, a pair of customers; gcc <= e < gcc + gdep * R,
// customer dep[(e - gcc) / R] against the start depot of route
// (e - gcc) % R, so that no thread walks every route.  The inter-route moves
// of N_theta(S) evaluated are added to S.acc[kAccGranInter].
// One block of work items, item e for this thread (every thread of the
// block calls it; red holds blockDim / 64 keys).
template <bool TW, bool DUMP>
__device__ __forceinline__ void gran_block(const SolDev &S, const GranPairs &P, int e, uint32_t op_mask,
                                           int32_t *__restrict__ dump_delta, uint8_t *__restrict__ dump_feas,
                                           unsigned long long *red, long long *cnt_sh) {
    if (threadIdx.x == 0) *cnt_sh = 0;
    __syncthreads();
    int bd = DUMP ? kAdmissibleBound : initial_bound(op_mask);
    uint32_t bid = 0xFFFFFFFFu;
    long long cnt = 0;
    int x = 0, t = 0;
    if (e < P.gcc) {
        x = gld(S.ref2slot + gld(P.src + e) - 1);
        t = gld(S.ref2slot + gld(P.adj + e) - 1);
    } else if (e - P.gcc < P.gdep * S.R) {
        const int k = (e - P.gcc) / S.R, r = (e - P.gcc) - k * S.R;
        x = gld(S.ref2slot + gld(P.dep + k) - 1);
        t = gld(S.roff + r);  // start depot slot of route r
    }
    if (x != t && gld(S.a4 + x).y != gld(S.a4 + t).y)
        cnt += gran_pair<TW, DUMP>(S, min(x, t), max(x, t), op_mask, dump_delta, dump_feas, bd, bid);
    for (int off = 32; off >= 1; off >>= 1) cnt += __shfl_xor(cnt, off);
    if ((threadIdx.x & 63) == 0 && cnt) atomicAdd((unsigned long long *)cnt_sh, (unsigned long long)cnt);
    block_argmin_commit(bd, bid, S.best_key, red);  // its barriers also order cnt_sh
    if (threadIdx.x == 0 && *cnt_sh) atomicAdd((unsigned long long *)(S.acc + kAccGranInter), (unsigned long long)*cnt_sh);
}

// theta nearest neighbours of every node (distance, then node id; the node
// itself excluded), one workgroup per node.  The row of D is read once into
// LDS; the theta-th smallest key (d << 14 | j) is found digit by digit from
// the top: a histogram of the next eight bits of the keys that share the
// digits found so far, then the bin that holds the theta-th.  It ends when
// every key of the bin is wanted.  (Bisecting the key range instead read the
// row some 38 times: 206 us at n = 2500 against 21.)
// out: theta node ids per node, in no order; bound: per node a value that
// exactly its theta neighbours' keys do not exceed.  Requires theta <= n;
// dynamic LDS of np1 ints.
constexpr int kKnnMax = 512;

__global__ __launch_bounds__(256) void k_knn(const int32_t *__restrict__ D, int np1, int theta,
                                             int32_t *__restrict__ out, unsigned long long *__restrict__ bound) {
    extern __shared__ int row[];
    __shared__ int hist[256];
    __shared__ int max_w[4], bin_sh, below_sh, nsel;
    const int i = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int mx = 0;
    for (int j = tid; j < np1; j += 256) {
        const int d = gld(D + (size_t)i * np1 + j);
        row[j] = d;
        mx = max(mx, d);
    }
    for (int off = 32; off >= 1; off >>= 1) mx = max(mx, __shfl_xor(mx, off));
    if (lane == 0) max_w[wave] = mx;
    if (tid == 0) nsel = 0;
    __syncthreads();
    mx = max(max(max_w[0], max_w[1]), max(max_w[2], max_w[3]));
    auto key = [&](int j) { return ((unsigned long long)(uint32_t)row[j] << 14) | (unsigned)j; };
    int bits = 32 - __clz(mx | 1) + 14, rem = theta;  // bits still to be found, rank among the keys that share the rest
    unsigned long long prefix = 0, limit = 0;
    while (true) {
        const int w = min(8, bits), shift = bits - w;
        hist[tid] = 0;
        __syncthreads();
        for (int j = tid; j < np1; j += 256) {
            const unsigned long long k = key(j);
            if (j != i && (k >> bits) == prefix) atomicAdd(&hist[(int)(k >> shift) & ((1 << w) - 1)], 1);
        }
        __syncthreads();
        if (wave == 0) {  // four bins per lane
            int c[4], t = 0;
            for (int u = 0; u < 4; ++u) t += c[u] = hist[4 * lane + u];
            int incl = t;
            for (int off = 1; off < 64; off <<= 1) {
                const int v = __shfl_up(incl, off);
                if (lane >= off) incl += v;
            }
            int below = incl - t;
            for (int u = 0; u < 4; ++u) {
                if (below < rem && rem <= below + c[u]) {
                    bin_sh = 4 * lane + u;
                    below_sh = below;
                }
                below += c[u];
            }
        }
        __syncthreads();
        const int bin = bin_sh, inbin = hist[bin];
        rem -= below_sh;
        prefix = (prefix << w) | (unsigned)bin;
        bits = shift;
        limit = ((prefix + 1) << shift) - 1;
        if (inbin == rem || shift == 0) break;  // the same for the whole workgroup
        __syncthreads();
    }
    for (int j = tid; j < np1; j += 256)
        if (j != i && key(j) <= limit) out[(size_t)i * theta + atomicAdd(&nsel, 1)] = j;
    if (tid == 0) bound[i] = limit;
}

// The granular pairs: the symmetric closure of the neighbour lists, every
// pair of customers once (src, adj), the customers paired with the depot in
// dep; cnt[0] and cnt[1] (zero before) receive how many.  One thread per list
// entry (i, j): a pair that is in both lists is emitted by its lower node's
// entry, which i's key against j's bound tells.  One atomic per workgroup.
__global__ __launch_bounds__(1024) void k_gran_pairs(const int32_t *__restrict__ D, int np1, int theta,
                                                     const int32_t *__restrict__ nn,
                                                     const unsigned long long *__restrict__ bound,
                                                     int32_t *__restrict__ src, int32_t *__restrict__ adj,
                                                     int32_t *__restrict__ dep, int *__restrict__ cnt) {
    __shared__ int n_sh[16][2], base_sh[2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long long e = (long long)blockIdx.x * 1024 + tid;
    int u = 0, v = 0;
    bool pair = false, depot = false;
    if (e < (long long)np1 * theta) {
        const int i = (int)(e / theta), j = nn[e];
        const unsigned long long k = ((unsigned long long)(uint32_t)gld(D + (size_t)j * np1 + i) << 14) | (unsigned)i;
        const bool mutual = k <= bound[j];
        u = i;
        v = j;
        depot = j == 0 || (i == 0 && !mutual);
        pair = i != 0 && j != 0 && (!mutual || i < j);
        if (i == 0) u = j;  // the customer of a depot pair
    }
    const unsigned long long mp = __builtin_amdgcn_ballot_w64(pair), md = __builtin_amdgcn_ballot_w64(depot);
    if (lane == 0) {
        n_sh[wave][0] = __builtin_popcountll(mp);
        n_sh[wave][1] = __builtin_popcountll(md);
    }
    __syncthreads();
    if (tid < 2) {
        int t = 0;
        for (int w = 0; w < 16; ++w) {
            const int c = n_sh[w][tid];
            n_sh[w][tid] = t;
            t += c;
        }
        base_sh[tid] = t ? atomicAdd(cnt + tid, t) : 0;
    }
    __syncthreads();
    const auto rank = [&](unsigned long long m) {
        return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
    };
    if (pair) {
        const int at = base_sh[0] + n_sh[wave][0] + rank(mp);
        src[at] = u;
        adj[at] = v;
    }
    if (depot) dep[base_sh[1] + n_sh[wave][1] + rank(md)] = u;
}

// ------------------------------------------------------ intra-route eval ---
// One wavefront per route (the route-based extraction of Section 5.3.1,
// eq. 2_opt, eq. ext_intra_relocate, eq. ext_intra_swap).  Lane i takes the
// first position i; the second position j walks the route while the
// summaries of the middle segments grow by one node per step, so every move
// costs O(1).  Positions p = 0..L+1 index the route (0 and L+1 are the
// depot).  A route that fits the wavefront's LDS region is staged there
// first (per-position data and the (L+2)^2 distance sub-block), so the walks
// never wait on global memory; a longer route reads the same values from
// the slot arrays and D directly.

constexpr int kIntraRegionBytes = 8192;  // LDS per wavefront in the intra phase

// Staged view: seven per-position arrays and the distance sub-block.
struct RouteLds {
    const int *pn, *pe, *pdep, *pz, *pe_, *pl, *ps, *dm;
    int stride;
    __device__ int node(int p) const { return pn[p]; }
    __device__ int edge(int p) const { return pe[p]; }
    __device__ int dep(int p) const { return pdep[p]; }
    __device__ int z(int p) const { return pz[p]; }
    __device__ int e(int p) const { return pe_[p]; }
    __device__ int l(int p) const { return pl[p]; }
    __device__ int s(int p) const { return ps[p]; }
    __device__ int dd(int p, int q) const { return dm[p * stride + q]; }
};

// Direct view over the slot arrays of route r.
struct RouteGlobal {
    const SolDev *S;
    int off, L, l0;
    __device__ int node(int p) const { return p <= L ? nodeof(gld(S->a4 + off + p).x) : 0; }
    __device__ int edge(int p) const { return gld(S->a4 + off + p).z; }
    __device__ int dep(int p) const { return gld(S->t4 + off + p).x; }
    __device__ int z(int p) const { return p <= L ? gld(S->t4 + off + p).w : l0; }
    __device__ int e(int p) const { return gld(S->w4 + off + p).x; }
    __device__ int l(int p) const { return gld(S->w4 + off + p).y; }
    __device__ int s(int p) const { return gld(S->w4 + off + p).z; }
    __device__ int dd(int p, int q) const { return gld(S->D + (size_t)node(p) * S->np1 + node(q)); }
};

// Moves of route r (L customers, view V) whose first position is i, for
// i = i0, i0 + di, ... <= L.  Without SPLIT: all of them; with it only walk per
// first position: 0 the 2-opt / same-route swap walk, 1..3 the forward and
// 4..6 the backward or-opt walk of segment length 1..3 (the seven walks
// cover each move exactly once).  A step reads everything it may need at its
// start, so that it waits for the staged values once, not once per test.
template <bool TW, bool DUMP, bool SPLIT, class RV>
__device__ __forceinline__ void intra_moves(const SolDev &S, const RV &V, int r, int L, int i0, int di,
                                            bool capOK, uint32_t op_mask, int walk_arg,
                                            int32_t *__restrict__ dump_delta, uint8_t *__restrict__ dump_feas, int &bd,
                                            uint32_t &bid) {
    const int walk = SPLIT ? walk_arg : -1;  // a compile-time -1 without the split
    const bool opSwap = op_mask & 2, op2o = op_mask & 8, opOr = op_mask & 16;
    if (SPLIT && walk > 6) return;
    const int n = S.n;
    const uint32_t uQ = (uint32_t)S.Q;
    auto ref = [&](int p) { return p == 0 ? (uint32_t)(n + r) : (uint32_t)(V.node(p) - 1); };
    auto segAt = [&](int p) { return seg_node(V.e(p), V.l(p), V.s(p)); };
#pragma unroll 1
    for (int i = i0; i <= L; i += di) {
        const int eP = V.edge(i - 1);  // c(c_{i-1}, c_i)
        const int eI = V.edge(i);      // c(c_i, c_{i+1})
        const int depP = TW ? V.dep(i - 1) : 0;
        const uint32_t refI = ref(i);
        const int bI = TW ? V.e(i) : 0, lI = TW ? V.l(i) : 0, sI = TW ? V.s(i) : 0;
        // Every step computes the deltas (and carries the segment summaries
        // along); feasibility, ids and the running minimum are evaluated
        // only where a delta can still reach the lane's best.
        // ---- 2OPT(i, j) and SWAP(i, j), j > i
        if ((op2o || opSwap) && walk <= 0) {
            Seg rev = TW ? seg_node(bI, lI, sI) : Seg{0, 0, 0, true};
            Seg mid = Seg{0, 0, 0, true};
            int ejm = eI;
#pragma unroll 1
            for (int j = i + 1; j <= L; ++j) {
                const int ej = V.edge(j);
                const int d1 = V.dd(i - 1, j), d2 = V.dd(i, j + 1);
                const int dA = V.dd(j, i + 1), dB = V.dd(j - 1, i);
                const uint32_t refJ = ref(j);
                const int bJ = TW ? V.e(j) : 0, lJ = TW ? V.l(j) : 0, sJ = TW ? V.s(j) : 0, zJ1 = TW ? V.z(j + 1) : 0;
                const Seg nj = seg_node(bJ, lJ, sJ);
                if (TW) rev = seg_cat(nj, ejm, rev);
                const int dlt2 = d1 + d2 - eP - ej;
                const int dS = j > i + 1 ? d1 + dA + dB + d2 - eP - eI - ejm - ej : dlt2;
                if (DUMP || (capOK && min(op2o ? dlt2 : kNoDelta, opSwap ? dS : kNoDelta) <= bd)) {
                    bool tw2 = true;
                    if (TW) tw2 = seg_pass(rev, depP + d1) + d2 <= zJ1;
                    bool twS = tw2;
                    if (TW && j > i + 1) {
                        const int arr0 = depP + d1;
                        bool ok = arr0 <= lJ;
                        const int t0 = max(arr0, bJ) + sJ;
                        const int dM = seg_pass(mid, t0 + dA);
                        const int arrI = dM + dB;
                        ok = ok && dM < kInf && arrI <= lI;
                        const int t2 = max(arrI, bI) + sI;
                        twS = ok && (t2 + d2 <= zJ1);
                    }
                    const uint32_t lo = min(refI, refJ), hi = max(refI, refJ);
                    if (op2o) {
                        const uint32_t id = (12u * uQ + lo) * uQ + hi;
                        if (DUMP) {
                            dump_delta[id] = dlt2;
                            dump_feas[id] = (uint8_t)(capOK | (tw2 << 1));
                        }
                        if (capOK && tw2) consider(dlt2, id, bd, bid);
                    }
                    if (opSwap) {
                        const uint32_t id = (5u * uQ + lo) * uQ + hi;
                        if (DUMP) {
                            dump_delta[id] = dS;
                            dump_feas[id] = (uint8_t)(capOK | (twS << 1));
                        }
                        if (capOK && twS) consider(dS, id, bd, bid);
                    }
                }
                // middle c_{i+1} .. c_j for the next j
                if (TW) mid = (j == i + 1) ? nj : seg_cat(mid, ejm, nj);
                ejm = ej;
            }
        }
        if (!opOr || walk == 0) continue;
#pragma unroll 1
        for (int k = 1; k <= 3; ++k) {
            if (walk > 0 && k != (walk <= 3 ? walk : walk - 3)) continue;
            if (i + k - 1 > L) break;
            // segment c_i..c_{i+k-1} (first f = i, last g = i+k-1), followed by w = i+k
            const int g = i + k - 1, w = i + k;
            const int eG = V.edge(g);  // c(g, w)
            const int dPW = V.dd(i - 1, w);
            const int base = dPW - eP - eG;
            Seg sig = Seg{0, 0, 0, true};
            if (TW) {
                sig = seg_node(bI, lI, sI);
#pragma unroll 1
                for (int q = 1; q < k; ++q) sig = seg_cat(sig, V.edge(i + q - 1), segAt(i + q));
            }
            // ---- forward: right after c_j, j >= i+k (middle c_{i+k} .. c_j)
            Seg mid = Seg{0, 0, 0, true};
            int ejm = eG;
#pragma unroll 1
            for (int j = w; j <= (walk <= 3 ? L : w - 1); ++j) {
                const int ej = V.edge(j), dVF = V.dd(j, i), dGV = V.dd(g, j + 1);
                const uint32_t refJ = ref(j);
                const int zJ1 = TW ? V.z(j + 1) : 0;
                if (TW) mid = (j == w) ? segAt(j) : seg_cat(mid, ejm, segAt(j));
                ejm = ej;
                const int dlt = base + dVF + dGV - ej;
                if (DUMP || (capOK && dlt <= bd)) {
                    bool tw = true;
                    if (TW) {
                        const int dm = seg_pass(mid, depP + dPW);
                        const int ds = dm >= kInf ? kInf : seg_pass(sig, dm + dVF);
                        tw = ds < kInf && ds + dGV <= zJ1;
                    }
                    const uint32_t id = ((16u + k) * uQ + refI) * uQ + refJ;
                    if (DUMP) {
                        dump_delta[id] = dlt;
                        dump_feas[id] = (uint8_t)(capOK | (tw << 1));
                    }
                    if (capOK && tw) consider(dlt, id, bd, bid);
                }
            }
            // ---- backward: right after c_j, j <= i-2 (middle c_{j+1} .. c_{i-1})
            const int zW = TW ? V.z(w) : 0;
            mid = Seg{0, 0, 0, true};
            int ej1 = 0;  // c(c_{j+1}, c_{j+2})
#pragma unroll 1
            for (int j = i - 2; j >= (walk < 0 || walk >= 4 ? 0 : i - 1); --j) {
                const int ej = V.edge(j), dVF = V.dd(j, i), dGV = V.dd(g, j + 1);
                const uint32_t refJ = ref(j);
                const int depJ = TW ? V.dep(j) : 0;
                if (TW) mid = (j == i - 2) ? segAt(i - 1) : seg_cat(segAt(j + 1), ej1, mid);
                ej1 = ej;
                const int dlt = base + dVF + dGV - ej;
                if (DUMP || (capOK && dlt <= bd)) {
                    bool tw = true;
                    if (TW) {
                        const int ds = seg_pass(sig, depJ + dVF);
                        const int dmm = ds >= kInf ? kInf : seg_pass(mid, ds + dGV);
                        tw = dmm < kInf && dmm + dPW <= zW;
                    }
                    const uint32_t id = ((16u + k) * uQ + refI) * uQ + refJ;
                    if (DUMP) {
                        dump_delta[id] = dlt;
                        dump_feas[id] = (uint8_t)(capOK | (tw << 1));
                    }
                    if (capOK && tw) consider(dlt, id, bd, bid);
                }
            }
        }
    }
}

// Stage route r (P = L + 2 positions) at `base` in LDS: seven per-position
// arrays followed by the P x P distance sub-block.  Returns the view.
template <bool TW>
__device__ __forceinline__ RouteLds stage_route(const SolDev &S, int off, int L, int l0, int *base) {
    const int lane = threadIdx.x & 63;
    const int P = L + 2;
    int *pn = base, *pe = pn + P, *pdep = pe + P, *pz = pdep + P, *pe_ = pz + P, *pl = pe_ + P, *ps = pl + P,
        *dm = ps + P;
    for (int p = lane; p < P; p += 64) {
        if (p <= L) {
            const int4 a = gld(S.a4 + off + p);
            pn[p] = nodeof(a.x);
            pe[p] = a.z;
            if (TW) {
                const int4 t = gld(S.t4 + off + p);
                const int4 w = gld(S.w4 + off + p);
                pdep[p] = t.x;
                pz[p] = t.w;
                pe_[p] = w.x;
                pl[p] = w.y;
                ps[p] = w.z;
            }
        } else {
            pn[p] = 0;
            pe[p] = 0;
            pz[p] = l0;
        }
    }
    return RouteLds{pn, pe, pdep, pz, pe_, pl, ps, dm, P};
}

constexpr int kIntraMaxGroup = 8;  // routes per intra-route work item
constexpr int kGatherBatch = 8;    // distance gathers in flight per lane while staging

// The P x P distance sub-blocks of G staged routes (route k = r0 + k: P[k]
// positions, staged at word offset at[k] of the region, nodes first):
// element y of route k's block is D[node(y / P)][node(y % P)].  A route whose
// cache entry holds the same P and nodes copies its block from there (LDS
// DMA) and any other route gathers it from D and, when P <= kRouteBlockMaxP,
// rewrites its entry.  Each lane keeps up to kGatherBatch loads in flight
// before it stores them, so a group costs a couple of memory round trips.
__device__ __forceinline__ void gather_dist_blocks(const SolDev &S, int *region, const int (&P)[kIntraMaxGroup],
                                                   const int (&at)[kIntraMaxGroup], int G, int r0, uint32_t hit,
                                                   uint32_t fill);

__device__ __forceinline__ void stage_dist_blocks(const SolDev &S, int *region, const int (&P)[kIntraMaxGroup],
                                                  const int (&at)[kIntraMaxGroup], int G, int r0) {
    const int lane = threadIdx.x & 63;
    // which routes' cached blocks are current (bit k), and which entries to rewrite
    uint32_t hit = 0, fill = 0;
#pragma unroll
    for (int k = 0; k < kIntraMaxGroup; ++k) {
        if (k < G && P[k] <= kRouteBlockMaxP) {
            const int *c = S.rblk + (size_t)(r0 + k) * kRouteBlockWords;
            const bool same = lane >= P[k] || gld(c + kRouteBlockNodes + lane) == region[at[k] + lane];
            const bool ok = __builtin_amdgcn_readfirstlane(gld(c)) == P[k] && __builtin_amdgcn_ballot_w64(!same) == 0;
            hit |= (ok ? 1u : 0u) << k;
            fill |= (ok ? 0u : 1u) << k;
        }
    }
    // current cached blocks: straight from the cache into LDS (LDS DMA, no
    // register round trip)
#pragma unroll
    for (int k = 0; k < kIntraMaxGroup; ++k) {
        if ((hit >> k) & 1) {
            const int *src = S.rblk + (size_t)(r0 + k) * kRouteBlockWords + kRouteBlockData;
            int *dst = region + at[k] + 7 * P[k];
            const int PP = P[k] * P[k];
            for (int c = 0; c < PP; c += 64)
                if (c + lane < PP)
                    __builtin_amdgcn_global_load_lds((global_void_ptr)(src + c + lane), (lds_void_ptr)(dst + c), 4, 0, 0);
        }
    }
    gather_dist_blocks(S, region, P, at, G, r0, hit, fill);
}

// The P x P blocks of the routes of the group not in `hit`, gathered from D
// into the region (and, for the routes in `fill`, into their cache
// entries); then, once every load issued before has landed, the nodes and
// P of the rewritten entries.
__device__ __forceinline__ void gather_dist_blocks(const SolDev &S, int *region, const int (&P)[kIntraMaxGroup],
                                                   const int (&at)[kIntraMaxGroup], int G, int r0, uint32_t hit,
                                                   uint32_t fill) {
    const int lane = threadIdx.x & 63;
    int cum[kIntraMaxGroup + 1];
    cum[0] = 0;
#pragma unroll
    for (int k = 0; k < kIntraMaxGroup; ++k) cum[k + 1] = cum[k] + (k < G ? P[k] * P[k] : 0);
    const int E = cum[kIntraMaxGroup];
    if (hit != (1u << G) - 1u) {
        for (int x0 = 0; x0 < E; x0 += 64 * kGatherBatch) {
            int val[kGatherBatch], dst[kGatherBatch], cst[kGatherBatch];
#pragma unroll
            for (int u = 0; u < kGatherBatch; ++u) {
                const int x = x0 + u * 64 + lane;
                dst[u] = -1;
                cst[u] = -1;
                val[u] = 0;
                if (x < E) {
                    int k = 0, c = 0, pk = P[0], ak = at[0];
#pragma unroll
                    for (int kk = 1; kk < kIntraMaxGroup; ++kk) {
                        if (kk < G && x >= cum[kk]) {
                            k = kk;
                            c = cum[kk];
                            pk = P[kk];
                            ak = at[kk];
                        }
                    }
                    if (!((hit >> k) & 1)) {
                        const int y = x - c;
                        const int pp = y / pk, qq = y - pp * pk;
                        const int *pn = region + ak;
                        val[u] = gld(S.D + (size_t)pn[pp] * S.np1 + pn[qq]);
                        if ((fill >> k) & 1) cst[u] = (r0 + k) * kRouteBlockWords + kRouteBlockData + y;
                        dst[u] = ak + 7 * pk + y;
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < kGatherBatch; ++u) {
                if (dst[u] >= 0) region[dst[u]] = val[u];
                if (cst[u] >= 0) S.rblk[cst[u]] = val[u];
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(0);  // the gathers and the caller's LDS DMA have landed (the caller then syncs the wavefront)
    // entries rewritten above: their nodes, then P
#pragma unroll
    for (int k = 0; k < kIntraMaxGroup; ++k) {
        if ((fill >> k) & 1) {
            int *c = S.rblk + (size_t)(r0 + k) * kRouteBlockWords;
            if (lane < P[k]) c[kRouteBlockNodes + lane] = region[at[k] + lane];
            if (lane == 0) c[0] = P[k];
        }
    }
}

__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wavefront evaluates every intra-route move of routes [r0, r1) of one
// solution and commits the best to the solution's key (the batched form's
// path for a group that intra_group_flat does not stage).  When all their
// positions fit (sum of L <= 64 first positions, staged data within the
// wavefront's LDS region), lane l takes one (route, first position) pair of
// the whole group; otherwise routes are taken one at a time.
template <bool TW>
__device__ __forceinline__ void intra_group(const SolDev &S, const IntraItem &item, uint32_t op_mask, int *region) {
    const int lane = threadIdx.x & 63;
    int bd = initial_bound(op_mask);
    uint32_t bid = 0xFFFFFFFFu;
    const int l0 = S.has_tw ? S.node4[0].z : kTwOff;
    const int G = min(item.r1 - item.r0, kIntraMaxGroup);
    int offs[kIntraMaxGroup + 1];
    offs[0] = gld(S.roff + item.r0);
    int sumL = 0, words = 0;
#pragma unroll
    for (int k = 0; k < kIntraMaxGroup; ++k) {
        if (k < G) {
            offs[k + 1] = gld(S.roff + item.r0 + k + 1);
            const int L = offs[k + 1] - offs[k] - 1, P = L + 2;
            sumL += L;
            words += 7 * P + P * P;
        }
    }
    if (sumL <= 64 && words <= kIntraRegionBytes / 4) {
        // stage every route of the group, then one lane per (route, first position)
        int *base = region;
#pragma unroll
        for (int k = 0; k < kIntraMaxGroup; ++k) {
            if (k < G) {
                const int L = offs[k + 1] - offs[k] - 1;
                stage_route<TW>(S, offs[k], L, l0, base);
                base += 7 * (L + 2) + (L + 2) * (L + 2);
            }
        }
        wave_lds_sync();
        {
            int Pk[kIntraMaxGroup], at[kIntraMaxGroup], w = 0;
#pragma unroll
            for (int k = 0; k < kIntraMaxGroup; ++k) {
                Pk[k] = k < G ? offs[k + 1] - offs[k] + 1 : 0;
                at[k] = w;
                w += 7 * Pk[k] + Pk[k] * Pk[k];
            }
            stage_dist_blocks(S, region, Pk, at, G, item.r0);
        }
        wave_lds_sync();
        // lane -> (route k, first position i) and that route's staged view
        int myk = -1, myi = 0, myL = 0, myOff = 0, myBase = 0, cum = 0, words2 = 0;
#pragma unroll
        for (int k = 0; k < kIntraMaxGroup; ++k) {
            if (k < G) {
                const int L = offs[k + 1] - offs[k] - 1, P = L + 2;
                if (myk < 0 && lane < cum + L) {
                    myk = k;
                    myi = lane - cum + 1;
                    myL = L;
                    myOff = offs[k];
                    myBase = words2;
                }
                cum += L;
                words2 += 7 * P + P * P;
            }
        }
        if (myk >= 0) {
            const int P = myL + 2;
            int *b = region + myBase;
            const RouteLds V{b, b + P, b + 2 * P, b + 3 * P, b + 4 * P, b + 5 * P, b + 6 * P, b + 7 * P, P};
            const bool capOK = gld(S.b4 + myOff).z <= S.cap;
            intra_moves<TW, false, false>(S, V, item.r0 + myk, myL, myi, 1 << 30, capOK, op_mask, -1, nullptr, nullptr, bd,
                                          bid);
        }
        wave_lds_sync();
    } else {
        for (int k = 0; k < G; ++k) {
            const int r = item.r0 + k;
            const int off = gld(S.roff + r);
            const int L = gld(S.roff + r + 1) - off - 1;
            const bool capOK = gld(S.b4 + off).z <= S.cap;
            const int P = L + 2;
            if (7 * P + P * P <= kIntraRegionBytes / 4) {
                const RouteLds V = stage_route<TW>(S, off, L, l0, region);
                wave_lds_sync();
                {
                    int Pk[kIntraMaxGroup], at[kIntraMaxGroup];
#pragma unroll
                    for (int k = 0; k < kIntraMaxGroup; ++k) {
                        Pk[k] = k == 0 ? P : 0;
                        at[k] = 0;
                    }
                    stage_dist_blocks(S, region, Pk, at, 1, r);
                }
                wave_lds_sync();
                intra_moves<TW, false, false>(S, V, r, L, lane + 1, 64, capOK, op_mask, -1, nullptr, nullptr, bd, bid);
                wave_lds_sync();
            } else {
                const RouteGlobal V{&S, off, L, l0};
                intra_moves<TW, false, false>(S, V, r, L, lane + 1, 64, capOK, op_mask, -1, nullptr, nullptr, bd, bid);
            }
        }
    }
    wave_argmin_commit(bd, bid, S.best_key);
}

// The intra-route moves of one (i, j) cell of route r (L customers, staged
// view V, 1 <= i <= L, 0 <= j <= L) without windows: 2OPT(i, j) and
// SWAP(i, j) when i < j, and the or-opt moves of the segments of length
// k = 1..3 that start at c_i to right after c_j (j >= i + k forward,
// j <= i - 2 backward).  The cells of the grid hold every intra-route move
// exactly once, with the deltas and ids of intra_moves (every position
// clamped into the route, invalid moves masked).
template <bool DUMP>
__device__ __forceinline__ void intra_cell(const SolDev &S, const RouteLds &V, int r, int L, int i, int j, bool capOK,
                                           bool opSwap, bool op2o, bool opOr, int32_t *__restrict__ dump_delta,
                                           uint8_t *__restrict__ dump_feas, int &bd, uint32_t &bid) {
    const int jm = max(j - 1, 0);
    const int eP = V.edge(i - 1), eI = V.edge(i), eJ = V.edge(j), eJm = V.edge(jm);
    const int d1 = V.dd(i - 1, j), d2 = V.dd(i, j + 1);  // j + 1 <= L + 1
    const int dA = V.dd(j, i + 1), dB = V.dd(jm, i);
    const int dVF = V.dd(j, i);
    const bool up = j > i;
    const int dlt2 = d1 + d2 - eP - eJ;
    const int dS = j > i + 1 ? d1 + dA + dB + d2 - eP - eI - eJm - eJ : dlt2;
    int m = kNoDelta;
    if (up && op2o) m = min(m, dlt2);
    if (up && opSwap) m = min(m, dS);
    int dOr[3];
    bool vOr[3];
#pragma unroll
    for (int k = 1; k <= 3; ++k) {
        const int g = min(i + k - 1, L);  // last node of the segment (clamped when it does not fit)
        dOr[k - 1] = V.dd(i - 1, g + 1) - eP - V.edge(g) + dVF + V.dd(g, j + 1) - eJ;
        vOr[k - 1] = opOr && i + k - 1 <= L && (j >= i + k || j <= i - 2);
        if (vOr[k - 1]) m = min(m, dOr[k - 1]);
    }
    if (!DUMP && m > bd) return;  // rare late in a search: no move of the cell can reach the lane's best

    const uint32_t uQ = (uint32_t)S.Q;
    const uint32_t refI = (uint32_t)(V.node(i) - 1);
    const uint32_t refJ = j == 0 ? (uint32_t)(S.n + r) : (uint32_t)(V.node(j) - 1);
    auto record = [&](int d, uint32_t id) {
        if (DUMP) {
            dump_delta[id] = d;
            dump_feas[id] = (uint8_t)(capOK | 2);
        }
        if (capOK) consider(d, id, bd, bid);
    };
    if (up) {
        const uint32_t lo = min(refI, refJ), hi = max(refI, refJ);
        if (op2o) record(dlt2, (12u * uQ + lo) * uQ + hi);
        if (opSwap) record(dS, (5u * uQ + lo) * uQ + hi);
    }
#pragma unroll
    for (int k = 1; k <= 3; ++k)
        if (vOr[k - 1]) record(dOr[k - 1], ((16u + k) * uQ + refI) * uQ + refJ);
}

// A route staged in a region has fewer than 64 positions, so a row of its
// cell grid (L + 1 cells) fits the wavefront.
static_assert(7 * 64 + 64 * 64 > kIntraRegionBytes / 4, "staged route within one wavefront row");

// The moves of intra_moves (no dump, every walk) whose first position is i,
// in two walks of the second position instead of seven: forward (j = i + 1
// .. L) the 2-opt and same-route swap moves together with the forward or-opt
// moves of the three segment lengths, backward (j = i - 2 .. 0) the backward
// or-opt moves, whose middle c_{j+1} .. c_{i-1} is the same for the three
// lengths.  The walks share their reads of position j; the segment summaries
// they carry are the ones intra_moves carries (the swap's middle
// c_{i+1} .. c_{j-1} is the length-1 or-opt middle of the step before), and
// concatenation is associative, so every feasibility test is the same.
template <bool TW>
__device__ __forceinline__ void intra_moves_joint(const SolDev &S, const RouteLds &V, int r, int L, int i,
                                                  bool capOK, uint32_t op_mask, int &bd, uint32_t &bid) {
    if (!capOK) return;  // over capacity: no admissible move
    const bool opSwap = op_mask & 2, op2o = op_mask & 8, opOr = op_mask & 16;
    const uint32_t uQ = (uint32_t)S.Q;
    auto ref = [&](int p) { return p == 0 ? (uint32_t)(S.n + r) : (uint32_t)(V.node(p) - 1); };
    auto segAt = [&](int p) { return seg_node(V.e(p), V.l(p), V.s(p)); };
    const int eP = V.edge(i - 1), eI = V.edge(i);
    const int depP = TW ? V.dep(i - 1) : 0;
    const uint32_t refI = ref(i);
    // or-opt segments c_i .. c_g (g = i + k - 1), then w = i + k
    bool okK[3];
    int baseK[3], dPW[3], zW[3];
    Seg sig[3];
#pragma unroll
    for (int k = 1; k <= 3; ++k) {
        const int g = min(i + k - 1, L);
        okK[k - 1] = opOr && i + k - 1 <= L;
        dPW[k - 1] = V.dd(i - 1, g + 1);
        baseK[k - 1] = dPW[k - 1] - eP - V.edge(g);
        zW[k - 1] = TW ? V.z(g + 1) : 0;
        if (TW) sig[k - 1] = k == 1 ? segAt(i) : seg_cat(sig[k - 2], V.edge(g - 1), segAt(g));
    }
    // ---- forward: j = i + 1 .. L.  The step is written once; the first
    // three steps (where the or-opt middles start) are peeled with their
    // offset PH = j - i known at compile time, so that the main loop updates
    // every summary unconditionally.
    Seg rev = TW ? segAt(i) : Seg{0, 0, 0, true};  // c_i .. c_j reversed
    Seg m1 = Seg{0, 0, 0, true}, m2 = m1, m3 = m1;  // c_{i+k} .. c_j (k = 1, 2, 3)
    auto fwd = [&](int j, auto phc) {
        constexpr int PH = decltype(phc)::value;  // j - i, or 4 for any j >= i + 4
        const int ej = V.edge(j), ejm = V.edge(j - 1);
        Seg sj = Seg{0, 0, 0, true};
        if (TW) {
            sj = segAt(j);
            rev = seg_cat(sj, ejm, rev);
        }
        const uint32_t refJ = ref(j);
        if (op2o || opSwap) {
            const int d1 = V.dd(i - 1, j), d2 = V.dd(i, j + 1);
            const int dlt2 = d1 + d2 - eP - ej;
            int dS = dlt2, dA = 0, dB = 0;
            if (PH > 1) {
                dA = V.dd(j, i + 1);
                dB = V.dd(j - 1, i);
                dS = d1 + dA + dB + d2 - eP - eI - ejm - ej;
            }
            if (min(op2o ? dlt2 : kNoDelta, opSwap ? dS : kNoDelta) <= bd) {
                bool tw2 = true;
                if (TW) tw2 = seg_pass(rev, depP + d1) + d2 <= V.z(j + 1);
                bool twS = tw2;
                if (TW && PH > 1) {
                    const int arr0 = depP + d1;
                    bool ok = arr0 <= V.l(j);
                    const int t0 = max(arr0, V.e(j)) + V.s(j);
                    const int dM = seg_pass(m1, t0 + dA);  // m1 is c_{i+1} .. c_{j-1} here
                    const int arrI = dM + dB;
                    ok = ok && dM < kInf && arrI <= V.l(i);
                    const int t2 = max(arrI, V.e(i)) + V.s(i);
                    twS = ok && (t2 + d2 <= V.z(j + 1));
                }
                const uint32_t lo = min(refI, refJ), hi = max(refI, refJ);
                if (op2o && tw2) consider(dlt2, (12u * uQ + lo) * uQ + hi, bd, bid);
                if (opSwap && twS) consider(dS, (5u * uQ + lo) * uQ + hi, bd, bid);
            }
        }
        if (TW) {
            m1 = PH == 1 ? sj : seg_cat(m1, ejm, sj);
            if (PH >= 2) m2 = PH == 2 ? sj : seg_cat(m2, ejm, sj);
            if (PH >= 3) m3 = PH == 3 ? sj : seg_cat(m3, ejm, sj);
        }
        if (opOr) {
            const int dVF = V.dd(j, i);
#pragma unroll
            for (int k = 1; k <= 3; ++k) {
                if (!okK[k - 1] || PH < k) continue;
                const int dGV = V.dd(i + k - 1, j + 1);
                const int dlt = baseK[k - 1] + dVF + dGV - ej;
                if (dlt > bd) continue;
                bool tw = true;
                if (TW) {
                    const Seg &mid = k == 1 ? m1 : (k == 2 ? m2 : m3);
                    const int dm = seg_pass(mid, depP + dPW[k - 1]);
                    const int ds = dm >= kInf ? kInf : seg_pass(sig[k - 1], dm + dVF);
                    tw = ds < kInf && ds + dGV <= V.z(j + 1);
                }
                if (tw) consider(dlt, ((16u + k) * uQ + refI) * uQ + refJ, bd, bid);
            }
        }
    };
    if (i + 1 <= L) fwd(i + 1, std::integral_constant<int, 1>{});
    if (i + 2 <= L) fwd(i + 2, std::integral_constant<int, 2>{});
    if (i + 3 <= L) fwd(i + 3, std::integral_constant<int, 3>{});
#pragma unroll 1
    for (int j = i + 4; j <= L; ++j) fwd(j, std::integral_constant<int, 4>{});
    if (!opOr) return;
    // ---- backward: j = i - 2 .. 0, middle c_{j+1} .. c_{i-1} (the first
    // step, where the middle is c_{i-1} alone, peeled as above)
    Seg mid = Seg{0, 0, 0, true};
    auto bwd = [&](int j, auto firstc) {
        if (TW) mid = decltype(firstc)::value ? segAt(i - 1) : seg_cat(segAt(j + 1), V.edge(j + 1), mid);
        const int dVF = V.dd(j, i), ej = V.edge(j);
        const int depJ = TW ? V.dep(j) : 0;
        const uint32_t refJ = ref(j);
#pragma unroll
        for (int k = 1; k <= 3; ++k) {
            if (!okK[k - 1]) continue;
            const int dGV = V.dd(i + k - 1, j + 1);
            const int dlt = baseK[k - 1] + dVF + dGV - ej;
            if (dlt > bd) continue;
            bool tw = true;
            if (TW) {
                const int ds = seg_pass(sig[k - 1], depJ + dVF);
                const int dmm = ds >= kInf ? kInf : seg_pass(mid, ds + dGV);
                tw = dmm < kInf && dmm + dPW[k - 1] <= zW[k - 1];
            }
            if (tw) consider(dlt, ((16u + k) * uQ + refI) * uQ + refJ, bd, bid);
        }
    };
    if (i - 2 >= 0) bwd(i - 2, std::true_type{});
#pragma unroll 1
    for (int j = i - 3; j >= 0; --j) bwd(j, std::false_type{});
}

// bits [lo, hi) of a 64-bit word (lo and hi clamped to [0, 64])
__device__ __forceinline__ unsigned long long bit_range(int lo, int hi) {
    lo = max(lo, 0);
    hi = min(hi, 64);
    if (lo >= hi) return 0ull;
    const unsigned long long top = hi >= 64 ? ~0ull : ((1ull << hi) - 1ull);
    return top & ~((1ull << lo) - 1ull);
}

// intra_group for the batched local-search launch (no dump, every walk of
// every route of the group in one wavefront).  A group that fits the region
// is staged with every load issued at once: the routes' per-position
// attributes and loads, their cache entries' P and nodes, and the cached
// distance blocks themselves (LDS DMA, before it is known whether they are
// current; a route whose entry turns out stale is then gathered from D over
// it).  With current entries the staging thus costs one memory round trip
// after the route offsets instead of several per route.  The moves of a
// VRPTW route are then taken by one lane per first position (the joint
// walks of intra_moves_joint), those of a CVRP route one (i, j) cell per
// lane (intra_cell), the cells laid over the wavefront as rows of L + 1
// lanes.  Any other group goes to intra_group.
template <bool TW>
__device__ __forceinline__ void intra_group_flat(const SolDev &S, const IntraItem &item, uint32_t op_mask,
                                                 int *region) {
    const int lane = threadIdx.x & 63;
    const int G = min(item.r1 - item.r0, kIntraMaxGroup);
    int offs[kIntraMaxGroup + 1];
#pragma unroll
    for (int k = 0; k <= kIntraMaxGroup; ++k) offs[k] = sld1(S.roff + min(item.r0 + k, item.r1));
    int P[kIntraMaxGroup], at[kIntraMaxGroup], cumP[kIntraMaxGroup + 1];
    int sumL = 0, words = 0;
    cumP[0] = 0;
#pragma unroll
    for (int k = 0; k < kIntraMaxGroup; ++k) {
        P[k] = k < G ? offs[k + 1] - offs[k] + 1 : 0;
        at[k] = words;
        if (k < G) {
            sumL += P[k] - 2;
            words += 7 * P[k] + P[k] * P[k];
        }
        cumP[k + 1] = cumP[k] + P[k];
    }
    if (!(sumL <= 64 && words <= kIntraRegionBytes / 4)) {
        intra_group<TW>(S, item, op_mask, region);
        return;
    }
    const int l0 = TW ? S.node4[0].z : kTwOff;
    const int NP = cumP[kIntraMaxGroup];  // positions of the group, <= 64 + 2 * kIntraMaxGroup
    // flat position f = lane + 64 u -> route k, position p: every load first
    int4 va[2], vt[2], vw[2];
    int cn[2], hd[2], ld[2], fk[2], fp[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int f = lane + 64 * u;
        int k = 0, pk = P[0], ok = offs[0], ck = 0;
#pragma unroll
        for (int kk = 1; kk < kIntraMaxGroup; ++kk) {
            if (kk < G && f >= cumP[kk]) {
                k = kk;
                pk = P[kk];
                ok = offs[kk];
                ck = cumP[kk];
            }
        }
        const int p = f - ck;
        fk[u] = f < NP ? k : -1;
        fp[u] = p;
        va[u] = vt[u] = vw[u] = make_int4(0, 0, 0, 0);
        cn[u] = hd[u] = -2;
        ld[u] = 0;
        if (f < NP) {
            const int *c = S.rblk + (size_t)(item.r0 + k) * kRouteBlockWords;
            if (p <= pk - 2) {
                va[u] = gld(S.a4 + ok + p);
                if (TW) {
                    vt[u] = gld(S.t4 + ok + p);
                    vw[u] = gld(S.w4 + ok + p);
                }
            }
            if (pk <= kRouteBlockMaxP) cn[u] = gld(c + kRouteBlockNodes + p);
            if (p == 0) {
                hd[u] = gld(c);
                ld[u] = gld(S.b4 + ok).z;
            }
        }
    }
    // the cached blocks, copied whether or not they are current
#pragma unroll
    for (int k = 0; k < kIntraMaxGroup; ++k) {
        if (k < G && P[k] <= kRouteBlockMaxP) {
            const int *src = S.rblk + (size_t)(item.r0 + k) * kRouteBlockWords + kRouteBlockData;
            int *dst = region + at[k] + 7 * P[k];
            const int PP = P[k] * P[k];
            for (int c = 0; c < PP; c += 64)
                if (c + lane < PP)
                    __builtin_amdgcn_global_load_lds((global_void_ptr)(src + c + lane), (lds_void_ptr)(dst + c), 4, 0, 0);
        }
    }
    __builtin_amdgcn_s_waitcnt(0);  // the DMA has landed before any of it is overwritten or read
    // per-position arrays (as stage_route), and per route: cache entry
    // current, route load within capacity (bits at the route's first
    // flat position)
    unsigned long long mism[2], hdok[2], capok[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        bool bad = false, hok = false, cok = false;
        if (fk[u] >= 0) {
            int k = 0;
#pragma unroll
            for (int kk = 1; kk < kIntraMaxGroup; ++kk) k = fk[u] == kk ? kk : k;
            int pk = P[0], ak = at[0];
#pragma unroll
            for (int kk = 1; kk < kIntraMaxGroup; ++kk) {
                if (k == kk) {
                    pk = P[kk];
                    ak = at[kk];
                }
            }
            const int p = fp[u];
            int *b = region + ak;
            int node;
            if (p <= pk - 2) {
                node = nodeof(va[u].x);
                b[p] = node;
                b[pk + p] = va[u].z;
                if (TW) {
                    b[2 * pk + p] = vt[u].x;
                    b[3 * pk + p] = vt[u].w;
                    b[4 * pk + p] = vw[u].x;
                    b[5 * pk + p] = vw[u].y;
                    b[6 * pk + p] = vw[u].z;
                }
            } else {
                node = 0;
                b[p] = 0;
                b[pk + p] = 0;
                b[3 * pk + p] = l0;
            }
            bad = pk <= kRouteBlockMaxP && cn[u] != node;
            hok = p == 0 && hd[u] == pk;
            cok = p == 0 && ld[u] <= S.cap;
        }
        mism[u] = __builtin_amdgcn_ballot_w64(bad);
        hdok[u] = __builtin_amdgcn_ballot_w64(hok);
        capok[u] = __builtin_amdgcn_ballot_w64(cok);
    }
    uint32_t hit = 0, fill = 0, capOK = 0;
#pragma unroll
    for (int k = 0; k < kIntraMaxGroup; ++k) {
        if (k < G) {
            const int c0 = cumP[k], c1 = cumP[k + 1];
            const bool stale = ((mism[0] & bit_range(c0, c1)) | (mism[1] & bit_range(c0 - 64, c1 - 64))) != 0ull;
            const bool hdr = ((c0 < 64 ? hdok[0] >> c0 : hdok[1] >> (c0 - 64)) & 1ull) != 0ull;
            const bool cap = ((c0 < 64 ? capok[0] >> c0 : capok[1] >> (c0 - 64)) & 1ull) != 0ull;
            if (P[k] <= kRouteBlockMaxP) {
                const bool cur = hdr && !stale;
                hit |= (cur ? 1u : 0u) << k;
                fill |= (cur ? 0u : 1u) << k;
            }
            capOK |= (cap ? 1u : 0u) << k;
        }
    }
    wave_lds_sync();  // the nodes are in place for the gathers
    gather_dist_blocks(S, region, P, at, G, item.r0, hit, fill);
    wave_lds_sync();

    int bd = initial_bound(op_mask);
    uint32_t bid = 0xFFFFFFFFu;
    if (TW) {
        // Time windows: most moves with a negative delta break a window, and
        // the walks carry the segment summaries from one move to the next,
        // so their check is O(1) where a cell's would be O(L): one lane per
        // (route, first position), as intra_group.
        int myk = -1, myi = 0, cum = 0;
#pragma unroll
        for (int k = 0; k < kIntraMaxGroup; ++k) {
            const int L = P[k] - 2;
            if (k < G && myk < 0 && lane < cum + L) {
                myk = k;
                myi = lane - cum + 1;
            }
            cum += k < G ? L : 0;
        }
        if (myk >= 0) {
            int pk = P[0], ak = at[0];
#pragma unroll
            for (int kk = 1; kk < kIntraMaxGroup; ++kk) {
                if (myk == kk) {
                    pk = P[kk];
                    ak = at[kk];
                }
            }
            int *b = region + ak;
            const RouteLds V{b, b + pk, b + 2 * pk, b + 3 * pk, b + 4 * pk, b + 5 * pk, b + 6 * pk, b + 7 * pk, pk};
            intra_moves_joint<TW>(S, V, item.r0 + myk, pk - 2, myi, (capOK >> myk) & 1, op_mask, bd, bid);
        }
        wave_lds_sync();
        wave_argmin_commit(bd, bid, S.best_key);
        return;
    }
    const bool opSwap = op_mask & 2, op2o = op_mask & 8, opOr = op_mask & 16;
    // route k's P and region offset sit in lane k (read back uniformly below,
    // so that the route loop is not unrolled)
    int laneP = 0, laneAt = 0;
#pragma unroll
    for (int k = 0; k < kIntraMaxGroup; ++k) {
        laneP = lane == k ? P[k] : laneP;
        laneAt = lane == k ? at[k] : laneAt;
    }
#pragma unroll 1
    for (int k = 0; k < G; ++k) {
        const int Pk = __builtin_amdgcn_readlane(laneP, k), L = Pk - 2;
        if (L < 1 || !((capOK >> k) & 1)) continue;  // over capacity: no admissible move
        int *b = region + __builtin_amdgcn_readlane(laneAt, k);
        const RouteLds V{b, b + Pk, b + 2 * Pk, b + 3 * Pk, b + 4 * Pk, b + 5 * Pk, b + 6 * Pk, b + 7 * Pk, Pk};
        // cells per row, rows per pass (W <= 62, see above)
        const int W = L + 1, rpi = 64 / W;
        const int di = lane / W, j = lane - di * W;
#pragma unroll 1
        for (int i0 = 1; i0 <= L; i0 += rpi) {
            const int i = i0 + di;
            if (di < rpi && i <= L)
                intra_cell<false>(S, V, item.r0 + k, L, i, j, true, opSwap, op2o, opOr, nullptr, nullptr, bd, bid);
        }
    }
    wave_lds_sync();  // the region is free for the next group
    wave_argmin_commit(bd, bid, S.best_key);
}

// A group of consecutive routes staged in LDS by a whole workgroup: route k
// (P[k] positions) at word offset at[k] of the region, NA per-position
// arrays (seven, more on the general path) and its P x P distance sub-block.
struct GroupStage {
    int offs[kIntraMaxGroup + 1], P[kIntraMaxGroup], at[kIntraMaxGroup];
    int NP, sumL, words;
};

// Layout of the routes [r0, r0 + G) (G <= kIntraMaxGroup), uniform.
template <int NA = 7>
__device__ __forceinline__ void group_layout(const SolDev &S, int r0, int G, GroupStage &g) {
#pragma unroll
    for (int k = 0; k <= kIntraMaxGroup; ++k) g.offs[k] = sld1(S.roff + r0 + min(k, G));
    g.NP = g.sumL = g.words = 0;
#pragma unroll
    for (int k = 0; k < kIntraMaxGroup; ++k) {
        g.P[k] = k < G ? g.offs[k + 1] - g.offs[k] + 1 : 0;
        g.at[k] = g.words;
        g.NP += g.P[k];
        g.sumL += k < G ? g.P[k] - 2 : 0;
        g.words += NA * g.P[k] + g.P[k] * g.P[k];
    }
}

// Per-position arrays of a group staged for the general path: the seven with
// deliveries and pickups in the place of departures and latest arrivals, then
// the time-warp (TW) and load (PD) summaries of prefix and suffix.
template <bool TW, bool PD>
constexpr int gen_arrays() { return 7 + (TW ? 8 : 0) + (PD ? 6 : 0); }

// Stages the group: every position's attributes at once, then every distance
// at once (the workgroup's eight wavefronts share them, so a group of 48
// customers takes two memory round trips after its offsets).  Every thread
// of the block calls it; it ends with a barrier.
template <bool TW, bool GEN = false, bool PD = false>
__device__ __forceinline__ void stage_group(const SolDev &S, const GroupStage &g, int *region) {
    constexpr int NA = GEN ? gen_arrays<TW, PD>() : 7;
    const int T = blockDim.x;
    const int l0 = TW ? sld(S.node4).z : kTwOff;
    for (int f = threadIdx.x; f < g.NP; f += T) {
        int pk = g.P[0], ak = g.at[0], ok = g.offs[0], c = 0, ck = 0;
#pragma unroll
        for (int k = 1; k < kIntraMaxGroup; ++k) {
            c += g.P[k - 1];
            if (g.P[k] && f >= c) {
                pk = g.P[k];
                ak = g.at[k];
                ok = g.offs[k];
                ck = c;
            }
        }
        const int p = f - ck, x = ok + p;
        int *b = region + ak + p;
        if (p <= pk - 2) {
            const int4 a = gld(S.a4 + x);
            if (TW || PD) {
                const int4 w = gld(S.w4 + x);
                if (TW && !GEN) {
                    const int4 t = gld(S.t4 + x);
                    b[2 * pk] = t.x;
                    b[3 * pk] = t.w;
                }
                if (PD) {
                    b[2 * pk] = gld(S.b4 + x).x;
                    b[3 * pk] = w.w;
                }
                b[4 * pk] = w.x;
                b[5 * pk] = w.y;
                b[6 * pk] = w.z;
            }
            b[0] = nodeof(a.x);
            b[pk] = a.z;
        } else {
            b[0] = 0;
            b[pk] = 0;
            if (!GEN) b[3 * pk] = l0;
        }
        if (GEN && TW) {
            const bool in = p <= pk - 2;
            const int4 q = gld(S.node4);
            const int4 f4 = in ? gld(S.pf4 + x) : make_int4(0, 0, 0, 0);
            const int4 b4 = in ? gld(S.pb4 + x) : make_int4(q.w, q.y, q.z, 0);  // the end depot
            b[7 * pk] = f4.x;
            b[8 * pk] = f4.y;
            b[9 * pk] = f4.z;
            b[10 * pk] = f4.w;
            b[11 * pk] = b4.x;
            b[12 * pk] = b4.y;
            b[13 * pk] = b4.z;
            b[14 * pk] = b4.w;
        }
        if (GEN && PD) {
            constexpr int o = TW ? 15 : 7;
            const bool in = p <= pk - 2;
            const int4 f4 = in ? gld(S.pl4 + x) : make_int4(0, 0, 0, 0);
            const int4 b4 = in ? gld(S.ql4 + x) : make_int4(0, 0, 0, 0);
            b[o * pk] = f4.x;
            b[(o + 1) * pk] = f4.y;
            b[(o + 2) * pk] = f4.z;
            b[(o + 3) * pk] = b4.x;
            b[(o + 4) * pk] = b4.y;
            b[(o + 5) * pk] = b4.z;
        }
    }
    __syncthreads();
    int E = 0;
#pragma unroll
    for (int k = 0; k < kIntraMaxGroup; ++k) E += g.P[k] * g.P[k];
    constexpr int U = 4;  // gathers in flight per thread
    for (int x0 = threadIdx.x; x0 < E; x0 += T * U) {
        int val[U], dst[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int x = x0 + u * T;
            dst[u] = -1;
            if (x < E) {
                int pk = g.P[0], ak = g.at[0], c = 0, ck = 0;
#pragma unroll
                for (int k = 1; k < kIntraMaxGroup; ++k) {
                    c += g.P[k - 1] * g.P[k - 1];
                    if (g.P[k] && x >= c) {
                        pk = g.P[k];
                        ak = g.at[k];
                        ck = c;
                    }
                }
                const int y = x - ck, pp = y / pk, qq = y - pp * pk;
                val[u] = gld(S.D + (size_t)region[ak + pp] * S.np1 + region[ak + qq]);
                dst[u] = ak + NA * pk + y;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (dst[u] >= 0) region[dst[u]] = val[u];
    }
    __syncthreads();
}

// Single-solution form: one workgroup evaluates the intra-route moves of the
// routes [r0, r1) and commits the best.  The group is staged once for all its
// wavefronts (one staging per wavefront gathered every distance seven times,
// in two rounds).  Without windows every (i, j) cell is then a thread's own;
// with them wavefront w takes walk w of every first position (see
// intra_moves), the segment summaries carried along: the launch waits for its
// longest chain, and for CVRP routes of about 20 customers the cells end
// 2.8 us after the staging where the walks took 5.6.  (With windows, tables of
// every segment's summary in LDS and cells that read them took as long as the
// walks, 8 us.)  A group that does not fit the region, or has more first
// positions than lanes, is taken route by route; a route that does not fit
// reads the slot arrays directly.
template <bool TW, bool DUMP>
__device__ __forceinline__ void intra_block(const SolDev &S, int r0, int r1, uint32_t op_mask,
                                            int32_t *__restrict__ dump_delta, uint8_t *__restrict__ dump_feas,
                                            int *region) {
    const int lane = threadIdx.x & 63;
    const int walk = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int bd = initial_bound(op_mask);
    uint32_t bid = 0xFFFFFFFFu;
    GroupStage g;
    for (int ra = r0; ra < r1;) {
        // the rest of the group when it fits, else its next route
        int G = r1 - ra;
        group_layout(S, ra, G, g);
        if (G > 1 && (g.sumL > 64 || g.words > kIntraRegionBytes / 4)) {
            G = 1;
            group_layout(S, ra, 1, g);
        }
        if (ra != r0) __syncthreads();  // the previous route is done with the region
        const int load = lane < G ? gld(S.b4 + gld(S.roff + ra + lane)).z : 0;
        if (g.words > kIntraRegionBytes / 4) {
            const int L = g.P[0] - 2;
            const RouteGlobal V{&S, g.offs[0], L, S.has_tw ? sld(S.node4).z : kTwOff};
            intra_moves<TW, DUMP, true>(S, V, ra, L, lane + 1, 64, __builtin_amdgcn_readfirstlane(load) <= S.cap, op_mask,
                                        walk, dump_delta, dump_feas, bd, bid);
            ra += G;
            continue;
        }
        stage_group<TW>(S, g, region);
        const unsigned long long caps = __builtin_amdgcn_ballot_w64(load <= S.cap);  // bit k: route ra + k
        // element f of the group (first positions with windows, else cells) ->
        // route k and the index within it; one pass, or several
        auto per_route = [&](int P) { return P == 0 ? 0 : (TW ? P - 2 : (P - 1) * (P - 2)); };
        int count = 0;
#pragma unroll
        for (int k = 0; k < kIntraMaxGroup; ++k) count += per_route(g.P[k]);
        for (int f = TW ? lane : (int)threadIdx.x; f < count; f += TW ? 64 : (int)blockDim.x) {
            int pk = g.P[0], ak = g.at[0], kk = 0, c = 0, ck = 0;
#pragma unroll
            for (int k = 1; k < kIntraMaxGroup; ++k) {
                c += per_route(g.P[k - 1]);
                if (g.P[k] && f >= c) {
                    pk = g.P[k];
                    ak = g.at[k];
                    kk = k;
                    ck = c;
                }
            }
            int *b = region + ak;
            const RouteLds V{b, b + pk, b + 2 * pk, b + 3 * pk, b + 4 * pk, b + 5 * pk, b + 6 * pk, b + 7 * pk, pk};
            const bool capOK = caps >> kk & 1;
            const int W = pk - 1;
            if constexpr (TW) {
                intra_moves<TW, DUMP, true>(S, V, ra + kk, W - 1, f - ck + 1, 1 << 30, capOK, op_mask, walk, dump_delta,
                                            dump_feas, bd, bid);
            } else if (DUMP || capOK) {
                const int i = (f - ck) / W + 1, j = f - ck - (i - 1) * W;
                intra_cell<DUMP>(S, V, ra + kk, W - 1, i, j, capOK, op_mask & 2, op_mask & 8, op_mask & 16, dump_delta,
                                 dump_feas, bd, bid);
            }
        }
        ra += G;
    }
    wave_argmin_commit(bd, bid, S.best_key);
}

// Single-solution form: workgroups below nintra take the intra-route groups
// (G routes each, the launch's longest chains, dispatched first), the others
// the inter-route items (strips of S.tile_rows rows), so both run at once in
// one launch.  With only one kind of operator enabled the other count is 0.
// The launch is bound by its chains of dependent reads, not by its work, so
// the descriptor comes by value (its pointers are there with the kernel's
// arguments) and the items are computed instead of read.  Per launch, with
// the groups staged by the whole workgroup: n = 1000 CVRP 11.1 us (18.8 with
// descriptor and items in memory and a staging per wavefront; 11.8 with walks
// for the intra-route moves), n = 201 VRPTW 12.3 (18.3), granular n = 1000
// VRPTW 13.2 (21.3).  The dynamic LDS is the larger of the two needs.
template <bool TW, bool DUMP>
__global__ __launch_bounds__(kInterThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_eval_solution(
    const SolDev S, int nintra, int G, uint32_t op_mask, int32_t *__restrict__ dump_delta,
    uint8_t *__restrict__ dump_feas) {
    extern __shared__ int4 smem4[];
    __shared__ unsigned long long red[kInterWaves];
    __shared__ int thr_sh;
    if (skip_solution(S, op_mask)) return;  // uniform for the grid
    if ((int)blockIdx.x < nintra) {
        const int r0 = blockIdx.x * G;
        intra_block<TW, DUMP>(S, r0, min(S.R, r0 + G), op_mask, dump_delta, dump_feas, (int *)smem4);
        return;
    }
    const int s0 = ((int)blockIdx.x - nintra) * S.tile_rows;
    const InterItem item{0, s0, min(S.Q, s0 + S.tile_rows), 0};
    if (S.D16)
        inter_item<TW, DUMP, true>(S, item, op_mask, dump_delta, dump_feas, smem4, red, &thr_sh);
    else
        inter_item<TW, DUMP, false>(S, item, op_mask, dump_delta, dump_feas, smem4, red, &thr_sh);
}

// Granular mode (as k_eval_solution): workgroups below nintra take the
// intra-route groups, the others kInterThreads granular work items each.
template <bool TW, bool DUMP>
__global__ __launch_bounds__(kInterThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_eval_gran(
    const SolDev S, const GranPairs P, int nintra, int G, uint32_t op_mask, int32_t *__restrict__ dump_delta,
    uint8_t *__restrict__ dump_feas) {
    extern __shared__ int4 smem4[];
    __shared__ unsigned long long red[kInterWaves];
    __shared__ long long cnt_sh;
    if (skip_solution(S, op_mask)) return;  // uniform for the grid
    if ((int)blockIdx.x < nintra) {
        const int r0 = blockIdx.x * G;
        intra_block<TW, DUMP>(S, r0, min(S.R, r0 + G), op_mask, dump_delta, dump_feas, (int *)smem4);
        return;
    }
    gran_block<TW, DUMP>(S, P, ((int)blockIdx.x - nintra) * blockDim.x + threadIdx.x, op_mask, dump_delta, dump_feas,
                         red, &cnt_sh);
}

// ------------------------------------------------------- general path ---
// Penalised mode, pickups, the operator variants and multi-move steps: new
// routes are concatenations of the stored prefix / suffix summaries with the
// moved nodes (Section 4.3.2, Section 4.3.3).  Penalised mode (feasible and
// infeasible search, Alg. A2): every move is admissible and scores
// dD + w_L dL_V + w_T dT_V over the touched routes (Section 5.3.3 attribute
// deltas, eq. scoring_tensor).  The dumps hold the score (penalised) or the
// delta, and the hard capacity / window bits of the touched routes.
//
// As on the plain path the deltas come first and the concatenations only
// where a move can still be the best: a score is at least
// dD - w_L L_V - w_T T_V of the routes as they are (new excess and warp are
// >= 0), and the deliveries of a new route bound its largest load from
// below.

__device__ __forceinline__ Tw tw_node_at(const SolDev &S, int x) {
    const int4 w = gld(S.w4 + x);
    return tw_node(w.x, w.y, w.z);
}

// Record one move of the general path.  Penalised mode: every move is
// admissible.  Otherwise the distance delta, admissible when the touched
// routes have no load excess and no time warp.
__device__ __forceinline__ void gen_record(const SolDev &S, int dD, int dlv, int dtv, bool capok, bool twok, uint32_t id,
                                           int32_t *dd, uint8_t *df, int &bd, uint32_t &bid) {
    const int feas = (capok ? 1 : 0) | (twok ? 2 : 0);
    const int score = S.pen ? dD + S.wL * dlv + S.wT * dtv : dD;
    if (dd) {
        dd[id] = score;
        df[id] = (uint8_t)feas;
    }
    consider(S.pen || feas == 3 ? score : score + kPenalty, id, bd, bid);
}

// An inter-route move as a queue entry: cx customers starting at slot x and
// ct customers starting at slot t leave their routes and take each other's
// place (a side that gives nothing receives right after its slot); rev: the
// moved segment is reversed; star: 2OPT*, the tails after x and t change
// places.
constexpr int kGenTBits = 14;  // t < 2^14 (TGA_MAX_Q)
constexpr int gen_code(int cx, int ct, int rev, int star) { return cx | (ct << 2) | (rev << 4) | (star << 5); }
constexpr int kGenStar = gen_code(0, 0, 0, 1);

// One side's new route: the prefix ending at slot p, then the c customers
// that start at slot y (reversed when rev), then what follows slot q.
// Returns its time warp; peak receives its largest load, del the deliveries
// of the inserted customers.
template <bool TW, bool PD>
__device__ __forceinline__ int gen_new_route(const SolDev &S, int p, int y, int c, bool rev, int q, const Tw &dep,
                                             int &peak, int &del) {
    const int32_t *D = S.D;
    const int np1 = S.np1;
    int last = nodeof(gld(S.a4 + p).x);
    const int after = nodeof(gld(S.a4 + q + 1).x);  // node 0 when the route ends at q
    Tw f{};
    Ld lf{};
    if (TW) f = tw_of(gld(S.pf4 + p));
    if (PD) lf = ld_of(gld(S.pl4 + p));
    del = 0;
#pragma unroll
    for (int u = 0; u < 3; ++u) {
        if (u < c) {
            const int s = rev ? y + c - 1 - u : y + u;
            const int node = nodeof(gld(S.a4 + s).x);
            del += gld(S.b4 + s).x;
            if (TW) f = tw_cat(f, gld(D + (size_t)last * np1 + node), tw_node_at(S, s));
            if (PD) lf = ld_cat(lf, ld_node_at(S, s));
            last = node;
        }
    }
    if (PD) peak = ld_cat(lf, after ? ld_of(gld(S.ql4 + q + 1)) : Ld{0, 0, 0}).lm;
    if (!TW) return 0;
    const Tw b = after ? tw_of(gld(S.pb4 + q + 1)) : dep;
    return tw_cat(f, gld(D + (size_t)last * np1 + after), b).v;
}

// The move `code` of the slot pair (x, t), distance delta dD.
template <bool TW, bool PD>
__device__ __forceinline__ void gen_eval_move(const SolDev &S, int x, int t, int code, int dD, int32_t *dd, uint8_t *df,
                                              int &bd, uint32_t &bid) {
    const int cx = code & 3, ct = (code >> 2) & 3;
    const bool rev = code & 16, star = code & 32;
    const int4 ax = gld(S.a4 + x), at = gld(S.a4 + t), bx = gld(S.b4 + x), bt = gld(S.b4 + t), gx = gld(S.g4 + x),
               gt = gld(S.g4 + t);
    const int px = cx ? x - 1 : x, qx = cx ? x + cx - 1 : x, pt = ct ? t - 1 : t, qt = ct ? t + ct - 1 : t;
    const Tw dep = TW ? tw_depot(S) : Tw{};
    int lx = 0, lt = 0, intoX, intoT;
    const int tvx = gen_new_route<TW, PD>(S, px, t, ct, rev, star ? t : qx, dep, lx, intoX);
    const int tvt = gen_new_route<TW, PD>(S, pt, x, cx, rev, star ? x : qt, dep, lt, intoT);
    if (!PD) {  // loads: what leaves one route enters the other
        lx = star ? bx.y + (bt.z - bt.y) : bx.z - intoT + intoX;
        lt = star ? bt.y + (bx.z - bx.y) : bt.z - intoX + intoT;
    }
    const int cap = S.cap, lv = max(lx - cap, 0) + max(lt - cap, 0);
    const int lvOld = max(gx.z - cap, 0) + max(gt.z - cap, 0);
    const uint32_t uQ = (uint32_t)S.Q;
    const uint32_t refX = (flagsof(ax.x) & kFlagCustomer) ? nodeof(ax.x) - 1 : S.n + ax.y;
    const uint32_t refT = (flagsof(at.x) & kFlagCustomer) ? nodeof(at.x) - 1 : S.n + at.y;
    const uint32_t lo = min(refX, refT), hi = max(refX, refT);
    uint32_t opk, a = lo, b = hi;
    if (star) {
        opk = 8u;
    } else if (!cx || !ct) {  // relocation of a segment: op 0, or op 5 / op 6
        const uint32_t k = (uint32_t)(cx + ct);
        opk = (k == 1 ? 0u : (rev ? 24u : 20u)) + k;
        a = cx ? refX : refT;
        b = cx ? refT : refX;
    } else if (cx == 1 && ct == 1) {
        opk = 5u;
    } else {  // cross-exchange, the lower ref's segment length in the operator
        opk = (6u + (uint32_t)(refX < refT ? cx : ct)) * 4u + (uint32_t)(refX < refT ? ct : cx);
    }
    gen_record(S, dD, lv - lvOld, tvx + tvt - gx.w - gt.w, lv == 0, tvx + tvt == 0, (opk * uQ + a) * uQ + b, dd, df, bd,
               bid);
}

// A wavefront's remaining steps go to gen_dense once it has queued so many
// moves in all, a quarter of them in the last step (256 is every move of a
// step of 64 pairs).  Fewer, and steps after which the threshold screens the
// rest pay for both sides' summaries for nothing (with 128 in one step a
// query of 1000 customers with pickups 53 us, 50 without); more, and the gain
// on 2000 empty routes goes (192 in one step: 320 us).
constexpr int kGenDense = 256, kGenDenseExt = 768;

// Per wavefront: moves waiting to be evaluated (slots and code, lower bound of
// the score, distance delta).
constexpr int kGenQueue = 192, kGenSteps = 64;
struct GenQueue {
    int move[kGenQueue], bound[kGenQueue], delta[kGenQueue];
    int step_min[kGenSteps];  // least lower bound of each of the wavefront's steps
};
static_assert(kInterWaves * sizeof(GenQueue) == kGenQueueBytes, "move queues");

// One side of a slot pair as gen_dense reads it: summaries of the prefixes
// that end before and at the slot, of the suffixes that start 1 .. M after it,
// and of the segments of 1 .. M customers that start at it, both ways round.
template <bool TW, bool PD, int M>
struct GenSide {
    Tw f0, f1, b[M + 1], seg[M + 1], rev[M + 1];
    Ld lf0, lf1, lb[M + 1], lseg[M + 1], lrev[M + 1];

    // at(array, slot): the slot's entry; node[k], e[k]: the node k slots on and
    // the edge leaving it
    template <class At>
    __device__ __forceinline__ void read(const SolDev &S, int x, const Tw &dep, At at, const int *node, const int *e) {
        const int Q = S.Q, xm = max(x - 1, 0);
#pragma unroll
        for (int k = 1; k <= M; ++k) {
            const int y = min(x + k, Q);
            if (TW) b[k] = node[k] ? tw_of(at(S.pb4, y)) : dep;
            if (PD) lb[k] = node[k] ? ld_of(at(S.ql4, y)) : Ld{0, 0, 0};
        }
        if (TW) {
            f0 = tw_of(at(S.pf4, xm));
            f1 = tw_of(at(S.pf4, x));
        }
        if (PD) {
            lf0 = ld_of(at(S.pl4, xm));
            lf1 = ld_of(at(S.pl4, x));
        }
        if (!TW && !PD) return;
#pragma unroll
        for (int k = 1; k <= M; ++k) {
            const int y = min(x + k - 1, Q);
            const int4 w = at(S.w4, y);
            if (TW) {
                const Tw nd = tw_node(w.x, w.y, w.z);
                seg[k] = k == 1 ? nd : tw_cat(seg[k - 1], e[k - 2], nd);
                rev[k] = k == 1 ? nd : tw_cat(nd, e[k - 2], rev[k - 1]);
            }
            if (PD) {
                const int dem = at(S.b4, y).x;
                const Ld nd{dem, w.w, max(dem, w.w)};
                lseg[k] = k == 1 ? nd : ld_cat(lseg[k - 1], nd);
                lrev[k] = k == 1 ? nd : ld_cat(nd, lrev[k - 1]);
            }
        }
    }
    // The new route made of this side's prefix (before the slot, or with it),
    // the other side's segment k (0: none) and `after`: its time warp (d1, d2:
    // the distances that join the parts) and its largest load.
    __device__ __forceinline__ int warp(bool before, const GenSide &o, int k, bool r, int d1, int d2, const Tw &after) const {
        if (!TW) return 0;
        const Tw &f = before ? f0 : f1;
        return k ? tw_cat(tw_cat(f, d1, r ? o.rev[k] : o.seg[k]), d2, after).v : tw_cat(f, d1, after).v;
    }
    __device__ __forceinline__ int peak(bool before, const GenSide &o, int k, bool r, const Ld &after) const {
        const Ld &f = before ? lf0 : lf1;
        return ld_cat(k ? ld_cat(f, r ? o.lrev[k] : o.lseg[k]) : f, after).lm;
    }
};

// The steps [idx, end) of a wavefront of gen_strip (its run begins at `first`)
// where most moves pass the screens: far from feasible, with ties of many
// empty routes, and in dumps.  Lane = column, row uniform, every move of a step
// evaluated in place: both sides' summaries are read once for all moves of the
// pair (coalesced or uniform), the distances come from the staged rows.  A
// queue entry's 30 scattered reads are worth it only where few lanes pass:
// 1000 customers in 60 routes and 2000 empty ones, windows broken, penalised
// 195 us a step against 592 (264 with one thread per pair), with the variants
// 660 against 1420 (450); 60 routes, windows broken, a penalised query 73
// against 92 (79), with the variants 126 against 188 (134).
template <bool TW, bool PD, bool EXT, bool W16>
__device__ __forceinline__ void gen_dense(const SolDev &S, int s0, int s1, int first, int idx, int end, uint32_t op_mask,
                                          int32_t *__restrict__ dd, uint8_t *__restrict__ df, const uint16_t *rows,
                                          int *thr_sh, const int *step_min, int &bd, uint32_t &bid) {
    constexpr int M = EXT ? 3 : 1;  // longest segment
    const int lane = threadIdx.x & 63;
    const int Q = S.Q, cap = S.cap, wL = S.wL, nr = s1 - s0;
    const bool pen = S.pen, multi = op_mask & kMulti;
    const uint32_t uQ = (uint32_t)Q;
    const Tw dep = TW ? tw_depot(S) : Tw{};
    auto threshold = [&]() {
        if (dd) return 0x7FFFFFFF;
        const int v = min(__hip_atomic_load(thr_sh, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP),
                          initial_bound(op_mask));
        return multi ? max(v, 0) : v;
    };
    // a step none of whose moves can be the best any more
    auto screened = [&]() {
        return !dd && !multi && idx - first < kGenSteps && step_min[idx - first] > threshold();
    };
    while (true) {
        while (idx < end && screened()) ++idx;
        if (idx >= end) return;
        const int j0 = idx / nr, t = s0 + 1 + 64 * j0 + lane, tc = min(t, Q);
        const int4 ta = gld(S.a4 + tc), tb = gld(S.b4 + tc), tg = gld(S.g4 + tc);
        int nt[M + 2], et[M], lt[M + 1] = {};  // nodes of t - 1 .. t + M; edges; deliveries of t's first k customers
#pragma unroll
        for (int k = -1; k <= M; ++k) nt[k + 1] = nodeof(gld(S.a4 + min(max(t + k, 0), Q)).x);
#pragma unroll
        for (int k = 0; k < M; ++k) {
            et[k] = gld(S.a4 + min(t + k, Q)).z;
            lt[k + 1] = gld(S.b4 + min(t + k, Q)).y - tb.y + tb.x;
        }
        GenSide<TW, PD, M> T;
        bool have = false;  // T is read
        const bool ct = flagsof(ta.x) & kFlagCustomer;
        int kt = ct ? 1 : 0;  // longest segment that starts at t
#pragma unroll
        for (int k = 2; k <= M; ++k) kt += kt == k - 1 && nt[k] != 0;
        const int ept = tb.w - ta.z;
        const uint32_t refT = ct ? nodeof(ta.x) - 1 : S.n + ta.y;
#pragma unroll 1
        for (const int stop = min(end, (j0 + 1) * nr); idx < stop; ++idx) {
            if (screened()) continue;
            const int thr = threshold();
            const int x = s0 + idx - j0 * nr;
            const int4 ra = sld(S.a4 + x), rb = sld(S.b4 + x), rg = sld(S.g4 + x);
            const bool valid = t < Q && ta.y > ra.y;
            if (!__builtin_amdgcn_ballot_w64(valid)) continue;
            int nx[M + 2], ex[M], lx[M + 1] = {};
#pragma unroll
            for (int k = -1; k <= M; ++k) nx[k + 1] = nodeof(sld(S.a4 + min(max(x + k, 0), Q)).x);
#pragma unroll
            for (int k = 0; k < M; ++k) {
                ex[k] = sld(S.a4 + min(x + k, Q)).z;
                lx[k + 1] = sld(S.b4 + min(x + k, Q)).y - rb.y + rb.x;
            }
            const bool cx = flagsof(ra.x) & kFlagCustomer;
            int kx = cx ? 1 : 0;
#pragma unroll
            for (int k = 2; k <= M; ++k) kx += kx == k - 1 && nx[k] != 0;
            const int epx = rb.w - ra.z;
            int w[M + 2][M + 2];  // w[1 + a][1 + b]: between x + a and t + b
#pragma unroll
            for (int a = 0; a < M + 2; ++a)
#pragma unroll
                for (int b = 0; b < M + 2; ++b)
                    if (EXT || a == 1 || b == 1)
                        w[a][b] = W16 ? rows[(x + a - s0) * S.stride16 + nt[b]] : gld(S.D + (size_t)nx[a] * S.np1 + nt[b]);
            // every move of the pair: f(gx, gt, rev, star), gx customers from x
            // and gt from t change sides
            auto each_move = [&](auto f) {
                if (op_mask & 1) {
                    f(1, 0, false, false);
                    f(0, 1, false, false);
                }
                if (op_mask & 2) f(1, 1, false, false);
                if (op_mask & 4) f(0, 0, false, true);
                if constexpr (EXT) {
                    if (op_mask & 32) {
                        f(2, 0, false, false);
                        f(3, 0, false, false);
                        f(0, 2, false, false);
                        f(0, 3, false, false);
                    }
                    if (op_mask & 64) {
                        f(2, 0, true, false);
                        f(3, 0, true, false);
                        f(0, 2, true, false);
                        f(0, 3, true, false);
                    }
                    if (op_mask & 128) {
                        f(1, 2, false, false);
                        f(1, 3, false, false);
                        f(2, 1, false, false);
                        f(2, 2, false, false);
                        f(2, 3, false, false);
                        f(3, 1, false, false);
                        f(3, 2, false, false);
                        f(3, 3, false, false);
                    }
                }
            };
            // the distances that join the new routes, and the delta
            struct Join {
                int dx1, dx2, dt1, dt2, delta;
            };
            auto join = [&](int gx, int gt, bool rev, bool star) {
                Join q{0, 0, 0, 0, 0};
                if (star) {
                    q.dx1 = w[1][2];
                    q.dt1 = w[2][1];
                    q.delta = q.dx1 + q.dt1 - ex[0] - et[0];
                    return q;
                }
                const int ax = gx ? gx : 1, at = gt ? gt : 1;  // what follows on each side, slots on
                if (gt) {
                    q.dx1 = w[gx ? 0 : 1][rev ? gt : 1];
                    q.dx2 = w[1 + ax][rev ? 1 : gt];
                } else {
                    q.dx1 = (gx == 1 ? ra.w : (gx == 2 ? rg.x : rg.y)) + epx + ex[ax - 1];
                }
                if (gx) {
                    q.dt1 = w[rev ? gx : 1][gt ? 0 : 1];
                    q.dt2 = w[rev ? 1 : gx][1 + at];
                } else {
                    q.dt1 = (gt == 1 ? ta.w : (gt == 2 ? tg.x : tg.y)) + ept + et[at - 1];
                }
                q.delta = q.dx1 + q.dx2 + q.dt1 + q.dt2 - (gx ? epx + ex[ax - 1] : ex[0]) - (gt ? ept + et[at - 1] : et[0]);
                return q;
            };
            const int Lx = rb.z, Lt = tb.z, lvOld = max(rg.z - cap, 0) + max(tg.z - cap, 0), tvOld = rg.w + tg.w;
            const int slack = pen ? wL * lvOld + S.wT * tvOld : 0;
            // whether a move can matter (lower bounds as in gen_strip)
            auto passes = [&](int gx, int gt, bool star, int delta) {
                const int load = star ? (Lt - tb.y) - (Lx - rb.y) : lt[gt] - lx[gx];
                const int over = max(Lx + load - cap, 0) + max(Lt - load - cap, 0);
                return valid && gx <= kx && gt <= kt &&
                       (dd || (pen ? delta - slack + wL * over <= thr : !over && delta <= thr));
            };
            bool some = false;
            each_move([&](int gx, int gt, bool rev, bool star) { some |= passes(gx, gt, star, join(gx, gt, rev, star).delta); });
            if (!__builtin_amdgcn_ballot_w64(some)) continue;
            if (!have) {
                T.read(S, tc, dep, [&](const int4 *p, int y) { return gld(p + y); }, nt + 1, et);
                have = true;
            }
            GenSide<TW, PD, M> X;
            X.read(S, x, dep, [&](const int4 *p, int y) { return sld(p + y); }, nx + 1, ex);
            const uint32_t refX = cx ? nodeof(ra.x) - 1 : S.n + ra.y;
            const uint32_t lo = min(refX, refT), hi = max(refX, refT);
            int b1 = multi ? kAdmissibleBound : bd;
            uint32_t i1 = multi ? 0xFFFFFFFFu : bid;
            each_move([&](int gx, int gt, bool rev, bool star) {
                const Join q = join(gx, gt, rev, star);
                const bool p = passes(gx, gt, star, q.delta);
                if (!__builtin_amdgcn_ballot_w64(p)) return;
                const int ax = gx ? gx : 1, at = gt ? gt : 1;
                const int tv = X.warp(gx, T, gt, rev, q.dx1, q.dx2, star ? T.b[1] : X.b[ax]) +
                               T.warp(gt, X, gx, rev, q.dt1, q.dt2, star ? X.b[1] : T.b[at]);
                const int load = star ? (Lt - tb.y) - (Lx - rb.y) : lt[gt] - lx[gx];
                int px = Lx + load, pt = Lt - load;
                if (PD) {
                    px = X.peak(gx, T, gt, rev, star ? T.lb[1] : X.lb[ax]);
                    pt = T.peak(gt, X, gx, rev, star ? X.lb[1] : T.lb[at]);
                }
                const int lv = max(px - cap, 0) + max(pt - cap, 0);
                uint32_t opk, a = lo, b = hi;  // ids as in gen_eval_move
                if (star) {
                    opk = 8u;
                } else if (!gx || !gt) {
                    opk = (gx + gt == 1 ? 0u : (rev ? 24u : 20u)) + (uint32_t)(gx + gt);
                    a = gx ? refX : refT;
                    b = gx ? refT : refX;
                } else if (gx == 1 && gt == 1) {
                    opk = 5u;
                } else {
                    opk = refX < refT ? (6u + gx) * 4u + gt : (6u + gt) * 4u + gx;
                }
                if (p) gen_record(S, q.delta, lv - lvOld, tv - tvOld, lv == 0, tv == 0, (opk * uQ + a) * uQ + b, dd, df, b1, i1);
            });
            if (multi) {  // the best improving move of each pair of routes
                if (b1 < 0 && i1 != 0xFFFFFFFFu) atomicMin(S.pairkey + (size_t)ra.y * S.R + ta.y, pack_key(b1, i1));
                if (i1 != 0xFFFFFFFFu) consider(b1, i1, bd, bid);
            } else {
                bd = b1;
                bid = i1;
            }
            if (!dd && __builtin_amdgcn_ballot_w64(bd < thr)) {  // publish what was found
                int wmin = bd;
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) wmin = min(wmin, __shfl_xor(wmin, off));
                if (lane == 0) atomicMin(thr_sh, wmin);
            }
        }
    }
}

// Whole-workgroup evaluation of the inter-route moves of the row slots
// [s0, s1) (fewer than 256) against every column slot of a later route.
// The (64-column chunk, row) steps are dealt to the wavefronts in equal
// contiguous runs, chunk-major; lane = column, the distances between the slots x - 1 .. x + 3 and
// t - 1 .. t + 3 in a register window (x - 1 .. x + 1 and t - 1 .. t + 1
// without the operator variants), one row of it gathered per step: from the
// rows staged in LDS (16-bit distances), else from D.
//
// A step forms the deltas of every move of the pair (4, with the variants up
// to 20).  The wavefront goes over its steps twice, because evaluating a move
// costs some 30 scattered reads per lane, which the compute unit's address
// path takes one lane at a time: with thresholds that start at 0 the 90,000
// improving moves of an early step were evaluated, 20 us of the launch.
// First each lane keeps the move with the least lower bound (delta, the
// loads' exact or least excess, less what the pair's routes could shed), and
// the best of every eight lanes is evaluated: the workgroup's 64 candidates
// give a threshold that hardly any move passes the second time.  The second
// pass takes only the steps whose least lower bound reaches it; in them the
// least delta of the pair is compared with the threshold; only where some
// lane passes are the moves taken one by one and those that can still be the
// best queued.  The queue is evaluated 64 moves at a time, one per lane, so
// the long concatenations run on full wavefronts whatever the share of lanes
// that passed.  A queue that fills up in the middle of a step is drained and
// the step taken again from the move that did not fit.  A wavefront that has
// queued as many moves as a whole step holds leaves its remaining steps to
// gen_dense.  Dumps and multi-move steps (which need every improving move)
// start with the second pass.
//
// The evaluation launch (with the intra-route groups) against one thread per
// pair evaluating all of its moves, and one per walk gathering from memory, in
// two launches: n = 1000 VRPTW penalised 21.8 us (58.7), n = 997 CVRP with the
// variants 22.8 (77.3), n = 603 with pickups 17.2 (43.4); multi-move, where
// nothing is screened against the best, 18.8 (57.4).  The first pass is bound
// by its arithmetic, the rest by the latency of one batch and by the longest
// intra-route walk (16 us).
template <bool TW, bool PD, bool EXT, bool W16>
__device__ __forceinline__ void gen_strip(const SolDev &S, int s0, int s1, uint32_t op_mask, int32_t *__restrict__ dd,
                                          uint8_t *__restrict__ df, int4 *smem4, unsigned long long *red, int *thr_sh,
                                          GenQueue *queues) {
    constexpr int A = EXT ? 3 : 1;  // slots read ahead of x and t
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int Q = S.Q, cap = S.cap, wL = S.wL;
    const bool pen = S.pen, multi = op_mask & kMulti;
    const uint16_t *rows = (const uint16_t *)smem4;
    const int rs = S.stride16;
    if (threadIdx.x == 0) *thr_sh = committed_delta(S);
    if (W16) drow_issue<true>(S, S.a4, S.Q, smem4, s0 - 1, s0 - 1, s1 - s0 + 1 + A, wave);
    int bd = initial_bound(op_mask);
    uint32_t bid = 0xFFFFFFFFu;
    GenQueue &q = queues[wave];
    int cnt = 0;  // queued moves
    auto threshold = [&]() {
        if (dd) return 0x7FFFFFFF;
        const int v = min(__hip_atomic_load(thr_sh, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP),
                          initial_bound(op_mask));
        return multi ? max(v, 0) : v;  // multi-move: every improving move counts, for its pair of routes
    };
    auto node_at = [&](int s) { return nodeof(gld(S.a4 + min(max(s, 0), Q)).x); };
    // added to the delta of a move that does not exist (at most three times);
    // real deltas are below 2^27 in magnitude
    constexpr int big = kAdmissibleBound, exists = big / 2;
    const int offRel = (op_mask & 1) ? 0 : big, offSwap = (op_mask & 2) ? 0 : big, offStar = (op_mask & 4) ? 0 : big,
              offKept = (op_mask & 32) ? 0 : big, offRev = (op_mask & 64) ? 0 : big,
              offCross = (op_mask & 128) ? 0 : big;
    // the wavefront's steps, and the columns of the current chunk
    const int nr = s1 - s0, T = ((Q - s0 - 1 + 63) / 64) * nr;
    const int first = T * wave / kInterWaves, last = T * (wave + 1) / kInterWaves;
    int idx = first, end = last;
    int pushed = 0, queued = 0;  // moves the current step has queued, and the steps before it
    int cb = s0 + 1 + first / nr * 64;
    int nd[A + 2];  // nodes of t - 1 .. t + A
    int4 ta, tb, tg;
    int et1 = 0, et2 = 0, lt1 = 0, lt2 = 0, slackT = 0;  // edges leaving t + 1, t + 2; deliveries of t's first 2 / 3 customers
    auto columns = [&]() {
        const int t = cb + lane, tc = min(t, Q);
        ta = gld(S.a4 + tc);
        tb = gld(S.b4 + tc);
        tg = gld(S.g4 + tc);
        nd[0] = node_at(t - 1);
        nd[1] = nodeof(ta.x);
        nd[2] = node_at(t + 1);
        if (EXT) {
            nd[3] = node_at(t + 2);
            nd[A + 1] = node_at(t + 3);
            et1 = gld(S.a4 + min(t + 1, Q)).z;
            et2 = gld(S.a4 + min(t + 2, Q)).z;
            lt1 = gld(S.b4 + min(t + 1, Q)).y - tb.y + tb.x;
            lt2 = gld(S.b4 + min(t + 2, Q)).y - tb.y + tb.x;
        }
        slackT = pen ? wL * max(tg.z - cap, 0) + S.wT * tg.w : 0;
    };
    if (idx < end) columns();
    // row attributes, read one step ahead
    int4 ra = sld(S.a4 + s0 + first % nr), rb = sld(S.b4 + s0 + first % nr), rg = sld(S.g4 + s0 + first % nr);
    if (W16) __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();  // rows and threshold in place
    // D between slot x + a (uniform) and the lane's node
    auto dist = [&](int x, int node) -> int {
        if (W16) return rows[(x - s0 + 1) * rs + node];
        const int rn = nodeof(sld(S.a4 + min(max(x, 0), Q)).x);
        return gld(S.D + (size_t)rn * S.np1 + node);
    };
    int w[A + 2][A + 2];  // w[1 + a][1 + b]: between x + a and t + b
    int x = s0 + first % nr, m0 = 0;  // row; first move of the step still to be taken
    bool fresh = true;       // the window and the row attributes are not those of row x yet
    bool fresh_cols = false;  // the columns are not those of chunk cb yet
    bool scan = !dd && !multi;
    int scan_lb = threshold(), scan_d = big, scan_mv = 0;  // the lane's most promising move of the first pass
    while (true) {
        const bool fin = idx >= end;
        const bool visit = !fin && (scan || dd || multi || m0 != 0 || idx - first >= kGenSteps ||
                                    q.step_min[idx - first] <= threshold());
        if (!fin && !visit) {  // no move of the step can be the best any more
            ++idx;
            fresh = true;
            if (++x == s1) {
                x = s0;
                cb += 64;
                fresh_cols = true;
            }
        }
        if (visit) {
            if (fresh_cols) {
                columns();
                fresh_cols = false;
            }
            if (fresh) {
                ra = sld(S.a4 + x);
                rb = sld(S.b4 + x);
                rg = sld(S.g4 + x);
#pragma unroll
                for (int a = 0; a <= A; ++a)
#pragma unroll
                    for (int b = 0; b < A + 2; ++b)
                        if (EXT || a == 1 || b == 1) w[a][b] = dist(x - 1 + a, nd[b]);
                fresh = false;
            }
            if (m0 == 0) {
#pragma unroll
                for (int b = 0; b < A + 2; ++b)
                    if (EXT || b == 1) w[A + 1][b] = dist(x + A, nd[b]);
            }
            const int xn = x + 1 == s1 ? s0 : x + 1;
            const int4 na = sld(S.a4 + xn), nb = sld(S.b4 + xn), ng = sld(S.g4 + xn);
            const bool cx = flagsof(ra.x) & kFlagCustomer, ctv = flagsof(ta.x) & kFlagCustomer;
            const int bx = cx ? 0 : big, bt = ctv ? 0 : big;
            const int ex = ra.z, et = ta.z;
            const bool valid = cb + lane < Q && ta.y > ra.y;
            const int thr = threshold();
            const int slack = slackT + (pen ? wL * max(rg.z - cap, 0) + S.wT * rg.w : 0);
            int d[20];
            d[0] = w[1][1] + w[1][2] - et + (ra.w + bx + offRel);
            d[1] = w[1][1] + w[2][1] + (ta.w + bt) + (offRel - ex);
            d[2] = w[0][1] + w[2][1] + w[1][0] + w[1][2] - tb.w + bt + (bx + offSwap - rb.w);
            d[3] = w[1][2] + w[2][1] - et + (offStar - ex);
            int lx1 = 0, lx2 = 0;  // deliveries of x's first 2 / 3 customers
            int m = min(min(d[0], d[1]), min(d[2], d[3]));
            if constexpr (EXT) {
                const int4 r1 = sld(S.a4 + min(x + 1, Q)), r2 = sld(S.a4 + min(x + 2, Q));
                const int kx = cx ? (nodeof(r1.x) == 0 ? 1 : (nodeof(r2.x) == 0 ? 2 : 3)) : 0;
                const int kt = ctv ? (nd[2] == 0 ? 1 : (nd[3] == 0 ? 2 : 3)) : 0;
                lx1 = sld(S.b4 + min(x + 1, Q)).y - rb.y + rb.x;
                lx2 = sld(S.b4 + min(x + 2, Q)).y - rb.y + rb.x;
                const int x2 = rg.x - et + (kx >= 2 ? 0 : big), x3 = rg.y - et + (kx >= 3 ? 0 : big);
                const int t2 = tg.x - ex + (kt >= 2 ? 0 : big), t3 = tg.y - ex + (kt >= 3 ? 0 : big);
                d[4] = w[1][1] + w[2][2] + x2 + offKept;
                d[5] = w[2][1] + w[1][2] + x2 + offRev;
                d[6] = w[1][1] + w[3][2] + x3 + offKept;
                d[7] = w[3][1] + w[1][2] + x3 + offRev;
                d[8] = w[1][1] + w[2][2] + t2 + offKept;
                d[9] = w[1][2] + w[2][1] + t2 + offRev;
                d[10] = w[1][1] + w[2][3] + t3 + offKept;
                d[11] = w[1][3] + w[2][1] + t3 + offRev;
                const int c0 = w[0][1] + w[1][0] + offCross;
                const int epx = rb.w - ra.z, ept = tb.w - ta.z;  // edges entering x and t
                const int ox[3] = {-epx - ex + bx, -epx - r1.z + (kx >= 2 ? 0 : big), -epx - r2.z + (kx >= 3 ? 0 : big)};
                const int ot[3] = {-ept - et + bt, -ept - et1 + (kt >= 2 ? 0 : big), -ept - et2 + (kt >= 3 ? 0 : big)};
#pragma unroll
                for (int j = 1; j <= 8; ++j) {
                    const int ka = j / 3 + 1, kb = j % 3 + 1;
                    d[11 + j] = c0 + w[1 + ka][kb] + w[ka][1 + kb] + ox[ka - 1] + ot[kb - 1];
                }
#pragma unroll
                for (int j = 4; j < 20; ++j) m = min(m, d[j]);
            }
            int next = 0x7FFFFFFF;  // the move to resume from when the queue is full
            const int Lx = rb.z, Lt = tb.z;
            // every move of the pair: f(j, deliveries that x's route gains from t's, code)
            auto each_move = [&](auto f) {
                f(0, -rb.x, gen_code(1, 0, 0, 0));
                f(1, tb.x, gen_code(0, 1, 0, 0));
                f(2, tb.x - rb.x, gen_code(1, 1, 0, 0));
                f(3, (Lt - tb.y) - (Lx - rb.y), kGenStar);
                if constexpr (EXT) {
                    f(4, -lx1, gen_code(2, 0, 0, 0));
                    f(5, -lx1, gen_code(2, 0, 1, 0));
                    f(6, -lx2, gen_code(3, 0, 0, 0));
                    f(7, -lx2, gen_code(3, 0, 1, 0));
                    f(8, lt1, gen_code(0, 2, 0, 0));
                    f(9, lt1, gen_code(0, 2, 1, 0));
                    f(10, lt2, gen_code(0, 3, 0, 0));
                    f(11, lt2, gen_code(0, 3, 1, 0));
#pragma unroll
                    for (int j = 1; j <= 8; ++j) {
                        const int ka = j / 3 + 1, kb = j % 3 + 1;
                        f(11 + j, (kb == 1 ? tb.x : (kb == 2 ? lt1 : lt2)) - (ka == 1 ? rb.x : (ka == 2 ? lx1 : lx2)),
                          gen_code(ka, kb, 0, 0));
                    }
                }
            };
            if (scan) {
                int step = valid && m < exists ? m - slack : 0x7FFFFFFF;
                if (__builtin_amdgcn_ballot_w64(step < scan_lb)) {
                    int lb = big, dj = big, code = 0;
                    if (pen)
                        each_move([&](int j, int load, int c) {
                            const int over = max(Lx + load - cap, 0) + max(Lt - load - cap, 0);
                            const int v = d[j] < exists ? d[j] + wL * over : big;
                            if (v < lb) {
                                lb = v;
                                dj = d[j];
                                code = c;
                            }
                        });
                    else
                        each_move([&](int j, int load, int c) {
                            const int v = ((cap - Lx - load) | (cap - Lt + load)) >= 0 ? d[j] : big;
                            if (v < lb) {
                                lb = v;
                                code = c;
                            }
                        });
                    if (!pen) dj = lb;
                    lb -= slack;
                    step = valid && dj < exists ? lb : 0x7FFFFFFF;
                    if (step < scan_lb) {
                        scan_lb = lb;
                        scan_d = dj;
                        scan_mv = (cb + lane) | ((x - s0) << kGenTBits) | (code << (kGenTBits + 8));
                    }
                }
#pragma unroll
                for (int o = 32; o >= 1; o >>= 1) step = min(step, __shfl_xor(step, o));
                if (lane == 0 && idx - first < kGenSteps) q.step_min[idx - first] = step;
            } else if (__builtin_amdgcn_ballot_w64(valid && m < exists && m - slack <= thr)) {
                const int had = cnt;
                each_move([&](int j, int load, int code) {
                    if (j < m0) return;
                    const int over = max(Lx + load - cap, 0) + max(Lt - load - cap, 0);
                    const int lb = pen ? d[j] - slack + wL * over : (over ? big : d[j]);
                    const bool p = valid && d[j] < exists && lb <= thr;
                    const unsigned long long mask = __builtin_amdgcn_ballot_w64(p);
                    if (!mask) return;
                    if (cnt > kGenQueue - 64) {
                        next = min(next, j);
                        return;
                    }
                    const int at = cnt + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
                    if (p) {
                        q.move[at] = (cb + lane) | ((x - s0) << kGenTBits) | (code << (kGenTBits + 8));
                        q.bound[at] = lb;
                        q.delta[at] = d[j];
                    }
                    cnt += __builtin_popcountll(mask);
                });
                pushed += cnt - had;
            }
            if (next == 0x7FFFFFFF) {  // on to the next row, or the next chunk
                m0 = 0;
                ++idx;
                constexpr int many = EXT ? kGenDenseExt : kGenDense;
                queued += pushed;
                if (queued >= many && 4 * pushed >= many) end = idx;  // gen_dense takes the rest
                pushed = 0;
                ra = na;
                rb = nb;
                rg = ng;
                if (++x == s1) {
                    x = s0;
                    cb += 64;
                    fresh = true;
                    fresh_cols = true;
                } else {
#pragma unroll
                    for (int a = 0; a <= A; ++a)
#pragma unroll
                        for (int b = 0; b < A + 2; ++b)
                            if (EXT || b == 1) w[a][b] = w[a + 1][b];
                    if (!EXT) {
                        w[1][0] = dist(x, nd[0]);
                        w[1][2] = dist(x, nd[2]);
                    }
                }
            } else {
                m0 = next;
            }
        }
        if (fin && scan) {  // the best of every eight lanes become the queue; then once more over the steps
            int g = scan_d < exists ? scan_lb : 0x7FFFFFFF;
#pragma unroll
            for (int o = 1; o <= 4; o <<= 1) g = min(g, __shfl_xor(g, o));
            const unsigned long long eq = __builtin_amdgcn_ballot_w64(scan_d < exists && scan_lb == g);
            const bool first = (eq >> lane & 1) && !(eq >> (lane & ~7) & ((1ull << (lane & 7)) - 1));
            const unsigned long long mask = __builtin_amdgcn_ballot_w64(first);
            const int at = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
            if (first) {
                q.move[at] = scan_mv;
                q.bound[at] = scan_lb;
                q.delta[at] = scan_d;
            }
            cnt = __builtin_popcountll(mask);
        }
        if (cnt >= 64 || (fin && cnt > 0)) {  // evaluate the last (up to) 64 queued moves
            const int take = min(cnt, 64), e = cnt - take + lane;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the queue is this wavefront's own
            __builtin_amdgcn_wave_barrier();
            if (lane < take && q.bound[e] <= threshold()) {
                const int mv = q.move[e];
                const int xx = s0 + ((mv >> kGenTBits) & 255), tt = mv & ((1 << kGenTBits) - 1);
                const int code = (mv >> (kGenTBits + 8)) & 63;
                if (multi) {  // the best improving move of each pair of routes
                    int b1 = kAdmissibleBound;
                    uint32_t i1 = 0xFFFFFFFFu;
                    gen_eval_move<TW, PD>(S, xx, tt, code, q.delta[e], dd, df, b1, i1);
                    if (b1 < 0 && i1 != 0xFFFFFFFFu)
                        atomicMin(S.pairkey + (size_t)gld(S.a4 + xx).y * S.R + gld(S.a4 + tt).y, pack_key(b1, i1));
                    if (i1 != 0xFFFFFFFFu) consider(b1, i1, bd, bid);
                } else {
                    gen_eval_move<TW, PD>(S, xx, tt, code, q.delta[e], dd, df, bd, bid);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            cnt -= take;
            if (!dd) {  // publish what was found
                int wmin = bd;
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) wmin = min(wmin, __shfl_xor(wmin, off));
                if (lane == 0) atomicMin(thr_sh, wmin);
            }
        }
        if (fin && cnt == 0) {
            if (!scan) break;
            scan = false;
            if (first == end) break;
            idx = first;
            x = s0 + first % nr;
            cb = s0 + 1 + first / nr * 64;
            fresh = fresh_cols = true;
        }
    }
    // (out of line where the registers of the loop above are better for it: with
    // pickups a step 32.9 us so and 34.7 in line, with windows alone 57 and 60
    // the other way round)
    auto rest = [&]() {
        gen_dense<TW, PD, EXT, W16>(S, s0, s1, first, end, last, op_mask, dd, df, rows, thr_sh, q.step_min, bd, bid);
    };
    if constexpr (TW && !PD) {
        if (end < last) rest();
    } else {
        if (__builtin_expect(end < last, 0)) rest();
    }
    block_argmin_commit(bd, bid, S.best_key, red);
}

// Views of a route on the general path: staged (gen_arrays), and direct.  A
// distance is looked up by two positions, each with its key: on the direct
// view its node, which the walks read a step ahead (one of the two reads a
// distance waits for), on the staged one nothing.  The walks look up the row
// of a position that stays the same for the lane: on the direct view its 4 KB
// stay in the cache, where the other way round every step reads new rows (one
// route of 1000 customers 0.68 ms a step, 0.56).
template <bool TW, bool PD>
struct GenLds {
    static constexpr bool direct = false;
    const int *b;
    int P;
    __device__ int node(int p) const { return b[p]; }
    __device__ int edge(int p) const { return b[P + p]; }
    __device__ Ld load(int p) const { return Ld{b[2 * P + p], b[3 * P + p], max(b[2 * P + p], b[3 * P + p])}; }
    __device__ Tw at(int p) const { return tw_node(b[4 * P + p], b[5 * P + p], b[6 * P + p]); }
    __device__ Tw sum(int o, int p) const { return Tw{b[o * P + p], b[(o + 1) * P + p], b[(o + 2) * P + p], b[(o + 3) * P + p]}; }
    __device__ Ld lsum(int o, int p) const { return Ld{b[o * P + p], b[(o + 1) * P + p], b[(o + 2) * P + p]}; }
    __device__ Tw pre(int p) const { return sum(7, p); }          // prefix ending at p
    __device__ Tw post(int p) const { return sum(11, p + 1); }    // suffix after p
    __device__ Ld lpre(int p) const { return lsum(TW ? 15 : 7, p); }
    __device__ Ld lpost(int p) const { return lsum(TW ? 18 : 10, p + 1); }
    __device__ int key(int) const { return 0; }
    __device__ int node(int p, int) const { return b[p]; }
    __device__ int dd(int p, int, int q, int) const { return b[gen_arrays<TW, PD>() * P + p * P + q]; }
};

struct GenGlobal {
    static constexpr bool direct = true;
    const SolDev &S;
    int off, L;
    __device__ int node(int p) const { return p <= L ? nodeof(gld(S.a4 + off + p).x) : 0; }
    __device__ int edge(int p) const { return gld(S.a4 + off + p).z; }
    __device__ Ld load(int p) const { return ld_node_at(S, off + p); }
    __device__ Tw at(int p) const { return tw_node_at(S, off + p); }
    __device__ Tw pre(int p) const { return tw_of(gld(S.pf4 + off + p)); }
    __device__ Tw post(int p) const { return p >= L ? tw_depot(S) : tw_of(gld(S.pb4 + off + p + 1)); }
    __device__ Ld lpre(int p) const { return ld_of(gld(S.pl4 + off + p)); }
    __device__ Ld lpost(int p) const { return p >= L ? Ld{0, 0, 0} : ld_of(gld(S.ql4 + off + p + 1)); }
    __device__ int key(int p) const { return node(p); }
    __device__ int node(int, int k) const { return k; }
    __device__ int dd(int, int kp, int, int kq) const { return gld(S.D + (size_t)kp * S.np1 + kq); }
};

// Intra-route moves of route r (slots off .., L customers, view V) whose
// first position is i: walk 0 the 2-opt walk, 1..3 or-opt of k = walk nodes
// moved forward, 4..6 k = walk - 3 moved backward, 7 the same-route swap walk.
// The middle summaries grow one node per step; a move is concatenated only
// when its delta, less what the route could shed in penalties, can reach the
// lane's best or the workgroup's (thr_sh; null: the lane's alone).
template <bool TW, bool PD, class RV>
__device__ __forceinline__ void gen_moves(const SolDev &S, const RV &V, int r, int off, int L, int i, uint32_t op_mask,
                                          int walk, int32_t *dd, uint8_t *df, int *thr_sh, int &bd, uint32_t &bid) {
    const int n = S.n, cap = S.cap;
    const uint32_t uQ = (uint32_t)S.Q;
    const bool opSwap = (op_mask & 2) && walk == 7, op2o = (op_mask & 8) && walk == 0, opOr = op_mask & 16;
    auto ref = [&](int p) { return p == 0 ? (uint32_t)(n + r) : (uint32_t)(V.node(p) - 1); };
    auto Npos = [&](int p) { return TW ? V.at(p) : Tw{}; };
    auto Fpos = [&](int p) { return TW ? V.pre(p) : Tw{}; };
    auto Bafter = [&](int p) { return TW ? V.post(p) : Tw{}; };
    auto LNpos = [&](int p) { return PD ? V.load(p) : Ld{}; };
    auto LFpos = [&](int p) { return PD ? V.lpre(p) : Ld{}; };
    auto LBafter = [&](int p) { return PD ? V.lpost(p) : Ld{}; };
    // on the direct view the part that closes a new route is read beside the
    // step's distances, not after the test (`at` does it, `use` reads it back)
    Tw endTw{};
    Ld endLd{};
    auto at = [&](auto f, auto lf, int p) {
        if constexpr (RV::direct) {
            endTw = f(p);
            endLd = lf(p);
        }
    };
    auto use = [&](auto f, int p) {
        if constexpr (RV::direct) return endTw;
        else return f(p);
    };
    auto luse = [&](auto f, int p) {
        if constexpr (RV::direct) return endLd;
        else return f(p);
    };
    const int4 g = gld(S.g4 + off);
    const int lvR = max(g.z - cap, 0), tvR = g.w;
    const int slack = S.pen ? S.wL * lvR + S.wT * tvR : 0;
    const bool hopeless = !S.pen && !PD && lvR > 0;  // an intra-route move keeps the load
    int thr = bd;
    auto can = [&](int dD) { return dd || (!hopeless && dD - slack <= thr); };
    auto refresh = [&]() {
        thr = bd;
        if (thr_sh) thr = min(bd, __hip_atomic_load(thr_sh, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
    };
    // new route: time warp tvNew, load excess lvNew
    auto rec = [&](int dD, int tvNew, int lvNew, uint32_t id) {
        const int was = bd;
        gen_record(S, dD, lvNew - lvR, tvNew - tvR, lvNew == 0, tvNew == 0, id, dd, df, bd, bid);
        if (thr_sh && bd < was) atomicMin(thr_sh, bd);
    };
    auto excess = [&](const Ld &x) { return PD ? max(x.lm - cap, 0) : lvR; };
    const int eP = V.edge(i - 1), eI = V.edge(i);
    const int kP = V.key(i - 1), kI = V.key(i);
    const Tw Fi1 = Fpos(i - 1);
    const Ld LFi1 = LFpos(i - 1);
    if (walk == 0 || walk == 7) {  // ---- 2OPT(i, j) or SWAP(i, j), j > i
        if (!op2o && !opSwap) return;
        Tw rev = Npos(i), mid{};
        Ld lrev = LNpos(i), lmid{};
        const int kI1 = V.key(i + 1);
        int ejm = eI, kjm = kI, kj = kI1, kj1 = V.key(min(i + 2, L + 1));
#pragma unroll 1
        for (int j = i + 1; j <= L; ++j) {
            const int ej = V.edge(j), kn = V.key(min(j + 2, L + 1));
            at(Bafter, LBafter, j);
            refresh();
            if (TW && op2o) rev = tw_cat(Npos(j), ejm, rev);
            if (PD && op2o) lrev = ld_cat(LNpos(j), lrev);
            const int d1 = V.dd(i - 1, kP, j, kj), d2 = V.dd(i, kI, j + 1, kj1);
            const int dO = d1 + d2 - eP - ej;
            int dA = 0, dB = 0, dS = dO;
            if (j > i + 1) {
                dA = V.dd(i + 1, kI1, j, kj);
                dB = V.dd(i, kI, j - 1, kjm);
                dS = d1 + dA + dB + d2 - eP - eI - ejm - ej;
            }
            const uint32_t refI = V.node(i, kI) - 1, refJ = V.node(j, kj) - 1;
            const uint32_t lo = min(refI, refJ), hi = max(refI, refJ);
            if (op2o && can(dO)) {
                const int tv = TW ? tw_cat(tw_cat(Fi1, d1, rev), d2, use(Bafter, j)).v : 0;
                rec(dO, tv, excess(ld_cat(ld_cat(LFi1, lrev), luse(LBafter, j))), (12u * uQ + lo) * uQ + hi);
            }
            if (opSwap && can(dS)) {
                Tw f = TW ? tw_cat(Fi1, d1, Npos(j)) : Tw{};
                Ld lf = PD ? ld_cat(LFi1, LNpos(j)) : Ld{};
                if (j > i + 1) {
                    if (TW) f = tw_cat(f, dA, mid);
                    if (PD) lf = ld_cat(lf, lmid);
                }
                const int tv = TW ? tw_cat(tw_cat(f, j > i + 1 ? dB : ejm, Npos(i)), d2, use(Bafter, j)).v : 0;
                rec(dS, tv, excess(ld_cat(ld_cat(lf, LNpos(i)), luse(LBafter, j))), (5u * uQ + lo) * uQ + hi);
            }
            if (TW && opSwap) mid = (j == i + 1) ? Npos(j) : tw_cat(mid, ejm, Npos(j));  // c_{i+1} .. c_j
            if (PD && opSwap) lmid = (j == i + 1) ? LNpos(j) : ld_cat(lmid, LNpos(j));
            ejm = ej;
            kjm = kj;
            kj = kj1;
            kj1 = kn;
        }
        return;
    }
    // ---- OR-OPT: segment c_i .. c_{i+k-1} moved right after c_j
    const int k = walk <= 3 ? walk : walk - 3;
    if (!opOr || i + k - 1 > L) return;
    const int gi = i + k - 1, wi = i + k;
    const int kG = V.key(gi), kW = V.key(wi);
    const int dPW = V.dd(i - 1, kP, wi, kW), base = dPW - eP - V.edge(gi);
    Tw sig{};
    Ld lsig{};
    if (TW) sig = Npos(i);
    if (PD) lsig = LNpos(i);
#pragma unroll 1
    for (int u = 1; u < k; ++u) {
        if (TW) sig = tw_cat(sig, V.edge(i + u - 1), Npos(i + u));
        if (PD) lsig = ld_cat(lsig, LNpos(i + u));
    }
    Tw mid{};
    Ld lmid{};
    if (walk <= 3) {
        int kj = kW, kj1 = V.key(min(wi + 1, L + 1));
#pragma unroll 1
        for (int j = wi; j <= L; ++j) {  // forward: middle c_{i+k} .. c_j
            const int kn = V.key(min(j + 2, L + 1));
            at(Bafter, LBafter, j);
            refresh();
            if (TW) mid = (j == wi) ? Npos(j) : tw_cat(mid, V.edge(j - 1), Npos(j));
            if (PD) lmid = (j == wi) ? LNpos(j) : ld_cat(lmid, LNpos(j));
            const int dVF = V.dd(i, kI, j, kj), dGV = V.dd(gi, kG, j + 1, kj1), dO = base + dVF + dGV - V.edge(j);
            if (can(dO)) {
                const int tv = TW ? tw_cat(tw_cat(tw_cat(Fi1, dPW, mid), dVF, sig), dGV, use(Bafter, j)).v : 0;
                rec(dO, tv, excess(ld_cat(ld_cat(ld_cat(LFi1, lmid), lsig), luse(LBafter, j))),
                    ((16u + k) * uQ + ref(i)) * uQ + ref(j));
            }
            kj = kj1;
            kj1 = kn;
        }
        return;
    }
    int kj = V.key(max(i - 2, 0)), kj1 = kP;
#pragma unroll 1
    for (int j = i - 2; j >= 0; --j) {  // backward: middle c_{j+1} .. c_{i-1}
        const int kn = V.key(max(j - 1, 0));
        at(Fpos, LFpos, j);
        refresh();
        if (TW) mid = (j == i - 2) ? Npos(i - 1) : tw_cat(Npos(j + 1), V.edge(j + 1), mid);
        if (PD) lmid = (j == i - 2) ? LNpos(i - 1) : ld_cat(LNpos(j + 1), lmid);
        const int dVF = V.dd(i, kI, j, kj), dGV = V.dd(gi, kG, j + 1, kj1), dO = base + dVF + dGV - V.edge(j);
        if (can(dO)) {
            const int tv = TW ? tw_cat(tw_cat(tw_cat(use(Fpos, j), dVF, sig), dGV, mid), dPW, Bafter(gi)).v : 0;
            rec(dO, tv, excess(ld_cat(ld_cat(ld_cat(luse(LFpos, j), lsig), lmid), LBafter(gi))),
                ((16u + k) * uQ + ref(i)) * uQ + ref(j));
        }
        kj1 = kj;
        kj = kn;
    }
}

constexpr int kGenRegionBytes = 16384;  // LDS of a staged group on the general path

// Whether a group's routes share one staged region, lane = first position.
template <bool TW, bool PD>
__device__ __forceinline__ bool gen_group_fits(int sumL, int words) {
    return sumL <= 64 && words <= kGenRegionBytes / 4;
}

// LDS words of a staged route of P positions.
template <bool TW, bool PD>
__device__ __forceinline__ int gen_words(int P) { return gen_arrays<TW, PD>() * P + P * P; }

// Fewest customers of a solution that can have routes walked by slots: one
// route too long for the region (21 arrays), or more than 64 in a group.
constexpr int kGenSlotsFrom = 50;
static_assert((7 + 8 + 6) * (kGenSlotsFrom + 1) + (kGenSlotsFrom + 1) * (kGenSlotsFrom + 1) <= kGenRegionBytes / 4,
              "a route of kGenSlotsFrom - 1 customers is staged");

// In a group that does not fit: whether its routes are walked by slots
// (gen_slot_block) and not staged one after another.  Two chains of staged
// steps take about as long as one of steps that gather from memory; more
// (short routes beside empty ones, whose number sets the groups) longer.
constexpr int kGenInTurn = 2;

// The moves of one wavefront's walk of route r (slots off .., L customers,
// view V) whose first position is i, i + step, ..; for a multi-move step also
// the route's best improving move.
template <bool TW, bool PD, class RV>
__device__ __forceinline__ void gen_walk(const SolDev &S, const RV &V, int r, int off, int L, int i, int step,
                                         uint32_t op_mask, int walk, int32_t *dd, uint8_t *df, int *thr_sh, int &bd,
                                         uint32_t &bid) {
    const bool multi = op_mask & kMulti;
    int b1 = multi ? initial_bound(op_mask) : bd;
    uint32_t i1 = multi ? 0xFFFFFFFFu : bid;
#pragma unroll 1
    for (; i <= L; i += step) gen_moves<TW, PD>(S, V, r, off, L, i, op_mask, walk, dd, df, thr_sh, b1, i1);
    if (multi) {
        if (b1 < 0 && i1 != 0xFFFFFFFFu) atomicMin(S.pairkey + (size_t)r * S.R + r, pack_key(b1, i1));
        if (i1 != 0xFFFFFFFFu) consider(b1, i1, bd, bid);
    } else {
        bd = b1;
        bid = i1;
    }
}

// One workgroup evaluates the intra-route moves of the routes [r0, r1) on the
// general path, wavefront w walk w (as intra_block).  Routes that are not
// staged are left to gen_slot_block.
template <bool TW, bool PD>
__device__ __forceinline__ void gen_intra_block(const SolDev &S, int r0, int r1, uint32_t op_mask,
                                                int32_t *__restrict__ dd, uint8_t *__restrict__ df, int *region, int *thr_sh) {
    const int lane = threadIdx.x & 63;
    const int walk = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int bd = initial_bound(op_mask);
    if (threadIdx.x == 0) *thr_sh = bd;
    if (dd || (op_mask & kMulti)) thr_sh = nullptr;  // every move, or every route's best, is wanted
    __syncthreads();
    uint32_t bid = 0xFFFFFFFFu;
    GroupStage g;
    const int G = r1 - r0;
    constexpr int NA = gen_arrays<TW, PD>();
    group_layout<NA>(S, r0, G, g);
    if (gen_group_fits<TW, PD>(g.sumL, g.words)) {
        int myk = -1, myi = 0, myP = 0, myAt = 0, myOff = 0, cum = 0;
#pragma unroll
        for (int k = 0; k < kIntraMaxGroup; ++k) {
            const int L = g.P[k] - 2;
            if (k < G && myk < 0 && lane < cum + L) {
                myk = k;
                myi = lane - cum + 1;
                myP = g.P[k];
                myAt = g.at[k];
                myOff = g.offs[k];
            }
            cum += k < G ? L : 0;
        }
        stage_group<TW, true, PD>(S, g, region);
        const GenLds<TW, PD> V{region + myAt, myP};
        if (myk >= 0)
            gen_walk<TW, PD>(S, V, r0 + myk, myOff, myP - 2, myi, 1 << 30, op_mask, walk, dd, df, thr_sh, bd, bid);
    } else {
        int staged = 0;
#pragma unroll
        for (int k = 0; k < kIntraMaxGroup; ++k)
            staged += g.P[k] > 2 && gen_words<TW, PD>(g.P[k]) <= kGenRegionBytes / 4;
        if (staged > kGenInTurn) return;  // uniform
        for (int k = 0; k < G; ++k) {
            const int r = r0 + k;
            group_layout<NA>(S, r, 1, g);
            if (g.sumL == 0 || g.words > kGenRegionBytes / 4) continue;
            __syncthreads();  // the previous route is done with the region
            stage_group<TW, true, PD>(S, g, region);
            const GenLds<TW, PD> V{region, g.P[0]};
            gen_walk<TW, PD>(S, V, r, g.offs[0], g.P[0] - 2, lane + 1, 64, op_mask, walk, dd, df, thr_sh, bd, bid);
        }
    }
    wave_argmin_commit(bd, bid, S.best_key);
}

// The routes gen_intra_block leaves (too long for its region, or too many to
// a group), by slots: one workgroup takes the first positions in the slots
// [s0, s0 + width), lane = slot, wavefront = walk, all data from memory, so a
// route of any length is one chain of its length spread over the chip: a
// penalised step with one route of 1000 customers (CVRP) 0.56 ms, 7.2 ms with
// all of the route's first positions in turn on one workgroup.  32 slots a
// workgroup: with 64 the gathers of eight wavefronts kept one compute unit's
// address path busy (0.78 ms when 32 took 0.68), 16 gained little more (0.62).  With no such route
// the workgroup ends after two reads.
template <bool TW, bool PD>
__device__ __forceinline__ void gen_slot_block(const SolDev &S, int s0, int width, int G, uint32_t op_mask,
                                               int32_t *__restrict__ dd, uint8_t *__restrict__ df, int *thr_sh) {
    const int s = s0 + (threadIdx.x & 63);
    const int4 a = gld(S.a4 + min(s, S.Q));
    const int r = min(a.y, S.R - 1), r0 = r / G * G;  // (slot Q's route is R)
    int off = 0, L = 0, sumL = 0, words = 0, staged = 0;
    int o[kIntraMaxGroup + 1];
#pragma unroll
    for (int k = 0; k <= kIntraMaxGroup; ++k) o[k] = gld(S.roff + min(r0 + min(k, G), S.R));
#pragma unroll
    for (int k = 0; k < kIntraMaxGroup; ++k) {
        const int P = o[k + 1] - o[k] + 1;  // 1 beyond the group
        const int w = P > 1 ? gen_words<TW, PD>(P) : 0;
        if (r0 + k == r) {
            off = o[k];
            L = P - 2;
        }
        sumL += max(P - 2, 0);
        words += w;
        staged += P > 2 && w <= kGenRegionBytes / 4;
    }
    const bool mine = s < min(s0 + width, S.Q) && (flagsof(a.x) & kFlagCustomer) &&
                      (gen_words<TW, PD>(L + 2) > kGenRegionBytes / 4 ||
                       (!gen_group_fits<TW, PD>(sumL, words) && staged > kGenInTurn));
    if (!__builtin_amdgcn_ballot_w64(mine)) return;  // the same slots in every wavefront
    const int walk = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int bd = initial_bound(op_mask);
    if (threadIdx.x == 0) *thr_sh = bd;
    if (dd || (op_mask & kMulti)) thr_sh = nullptr;  // as gen_intra_block
    __syncthreads();
    uint32_t bid = 0xFFFFFFFFu;
    const GenGlobal V{S, off, L};
    if (mine) gen_walk<TW, PD>(S, V, r, off, L, s - off, 1 << 30, op_mask, walk, dd, df, thr_sh, bd, bid);
    wave_argmin_commit(bd, bid, S.best_key);
}

// First row slot of strip k of n (k = n gives Q): rows grow as (1 - k/n)^(-1/4),
// between strips of equal work (whose last ones had so many rows that they
// took several rounds of staging and ended last) and of equal rows.
__device__ __forceinline__ int strip_begin(int Q, int k, int n) {
    if (k >= n) return Q;
    const float r = sqrtf(1.0f - (float)k / (float)n);
    return Q - min(Q, (int)ceilf((float)Q * r * sqrtf(r)));
}

// One evaluation on the general path (as k_eval_solution): workgroups below
// nslot take 64 slots each for the routes that are not staged, the next nintra
// the intra-route groups of G routes, the others one strip of row slots each,
// at most `rows` of them staged at a time.
template <bool TW, bool PD, bool EXT, bool W16>
__global__ __launch_bounds__(kInterThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_eval_general(
    const SolDev S, int nslot, int width, int nintra, int G, int rows, uint32_t op_mask, int32_t *__restrict__ dd,
    uint8_t *__restrict__ df) {
    extern __shared__ int4 smem4[];
    __shared__ unsigned long long red[kInterWaves];
    __shared__ int thr_sh;
    __shared__ GenQueue queues[kInterWaves];
    if (skip_solution(S, op_mask)) return;  // uniform for the grid
    const int item = (int)blockIdx.x - nslot;
    if (item < 0) {
        gen_slot_block<TW, PD>(S, blockIdx.x * width, width, G, op_mask, dd, df, &thr_sh);
        return;
    }
    if (item < nintra) {
        const int r0 = item * G;
        gen_intra_block<TW, PD>(S, r0, min(S.R, r0 + G), op_mask, dd, df, (int *)smem4, &thr_sh);
        return;
    }
    const int k = item - nintra, n = (int)gridDim.x - nslot - nintra;
    const int s0 = __builtin_amdgcn_readfirstlane(strip_begin(S.Q, k, n));
    const int s1 = __builtin_amdgcn_readfirstlane(strip_begin(S.Q, k + 1, n));
    for (int x = s0; x < s1; x += rows)
        gen_strip<TW, PD, EXT, W16>(S, x, min(s1, x + rows), op_mask, dd, df, smem4, red, &thr_sh, queues);
}

// Batched form: persistent launches evaluate every solution of the batch.
// PH bit 1: intra-route groups (one wavefront per group of routes); PH bit 0:
// inter-route items (whole workgroup per item, largest first).  PH = 3 runs
// both phases in one launch, the latency-bound intra-route walks first so
// that they overlap other workgroups' inter-route work and the small
// inter-route items fill the tail; PH = 1 and PH = 2 are the two halves as
// separate launches.
// Solutions of both problem types and both distance widths share a launch;
// each item takes the path of its own solution.  Workgroup b is dispatched
// to XCD x = b mod nx and works on the items of the solutions placed there:
// its wavefronts take the intra-route groups j * 8 + wave, then every
// (G' * 8)-th after it, of the XCD's group list (j = b / nx, G' =
// gridDim.x / nx); then the workgroup pulls the XCD's inter-route items
// items[woff[x] ..  woff[x + 1]) (largest first) from a queue, counter
// qctr[2x] (items taken), so that whichever workgroup is free takes the
// next one.  Each workgroup's next pull is issued while it evaluates its
// current item.  A workgroup that finds the queue empty counts itself in
// qctr[2x + 1]; the last of the XCD's workgroups to do so puts both
// counters back to zero, ready for the next launch.
template <int PH>
__global__ __launch_bounds__(kInterThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_eval_batch(
    const SolDev *__restrict__ sols, const InterItem *__restrict__ items, const int *__restrict__ woff,
    uint32_t *__restrict__ qctr, const IntraItem *__restrict__ intra, const int *__restrict__ ixoff, int nx,
    uint32_t op_mask) {
    extern __shared__ int4 smem4[];
    __shared__ int thr_sh;
    const int wave = threadIdx.x >> 6;
    const int x = blockIdx.x % nx, j = blockIdx.x / nx, step = gridDim.x / nx;
    if ((PH & 2) && (op_mask & (2 | 8 | 16))) {
        int *region = (int *)smem4 + wave * (kIntraRegionBytes / 4);
        const int end = ixoff[x + 1];
        for (int it = ixoff[x] + j * kInterWaves + wave; it < end; it += step * kInterWaves) {
            const IntraItem item = intra[it];
            const SolDev &S = sols[item.sol];
            if (skip_solution(S, op_mask)) continue;
            if (S.has_tw)
                intra_group_flat<true>(S, item, op_mask, region);
            else
                intra_group_flat<false>(S, item, op_mask, region);
        }
    }
    __syncthreads();  // the intra-route regions and the inter-route rows share LDS
    if ((PH & 1) && (op_mask & 7)) {
        __shared__ int q_sh[2];  // pulled item index, alternate slots by iteration
        const int first = woff[x], cnt = woff[x + 1] - first;
        uint32_t *taken = qctr + 2 * x, *finished = taken + 1;
        if (threadIdx.x == 0) q_sh[0] = (int)atomicAdd(taken, 1u);
        __syncthreads();
        for (int round = 0;; ++round) {
            const int k = q_sh[round & 1];
            if (k >= cnt) break;  // the same for the whole workgroup
            int next = 0;
            if (threadIdx.x == 0) next = (int)atomicAdd(taken, 1u);  // lands while this item is evaluated
            const InterItem item = items[first + k];
            const SolDev &S = sols[item.sol];
            if (skip_solution(S, op_mask)) {
                if (threadIdx.x == 0) q_sh[(round + 1) & 1] = next;
                __syncthreads();
                continue;
            }
            constexpr bool CNT = (PH & 4) != 0;
            if (S.has_tw) {
                if (S.D16)
                    inter_item<true, false, true, CNT, true>(S, item, op_mask, nullptr, nullptr, smem4, nullptr, &thr_sh);
                else
                    inter_item<true, false, false, CNT, true>(S, item, op_mask, nullptr, nullptr, smem4, nullptr, &thr_sh);
            } else {
                if (S.D16)
                    inter_item<false, false, true, CNT, true>(S, item, op_mask, nullptr, nullptr, smem4, nullptr, &thr_sh);
                else
                    inter_item<false, false, false, CNT, true>(S, item, op_mask, nullptr, nullptr, smem4, nullptr, &thr_sh);
            }
            // slot (round + 1) & 1 was last read in the previous round, before
            // that round's closing barrier
            if (threadIdx.x == 0) q_sh[(round + 1) & 1] = next;
            __syncthreads();
        }
        if (threadIdx.x == 0 && atomicAdd(finished, 1u) == gridDim.x / nx - 1) {
            // every workgroup of the XCD has made its last pull
            atomicExch(taken, 0u);
            atomicExch(finished, 0u);
        }
    }
}

// ------------------------------------------------- finalize / apply / LS ---

enum { kModeRecord = 0, kModeLS = 1, kModeApplyRec = 2 };

struct MoveInfo {
    int op, k, a, b, ra, rb, pa, pb, La, Lb, nLa, nLb, valid, delta;
    uint32_t id;
};

__device__ __forceinline__ int old_node(const SolDev &S, int r, int p) {
    return p == 0 ? 0 : nodeof(S.a4[S.roff[r] + p].x);
}

// Old position whose node stands at new position p >= 1 of a touched route
// (Section 4.1 operators): route ra, or rb when isB.  The old position is in
// rb when fromB is set, else in ra.
__device__ __forceinline__ int new_src(const MoveInfo &m, bool isB, int p, bool &fromB) {
    fromB = isB;
    switch (m.op) {
    case 0:
        if (!isB) return p < m.pa ? p : p + 1;
        if (p <= m.pb) return p;
        if (p > m.pb + 1) return p - 1;
        fromB = false;
        return m.pa;
    case 1:
        if (m.ra == m.rb) return p == m.pa ? m.pb : (p == m.pb ? m.pa : p);
        if (p != (isB ? m.pb : m.pa)) return p;
        fromB = !isB;
        return isB ? m.pa : m.pb;
    case 2:
        if (!isB) {
            if (p <= m.pa) return p;
            fromB = true;
            return m.pb + p - m.pa;
        }
        if (p <= m.pb) return p;
        fromB = false;
        return m.pa + p - m.pb;
    case 3: {
        const int i = min(m.pa, m.pb), j = max(m.pa, m.pb);
        return (p >= i && p <= j) ? i + j - p : p;
    }
    case 5:
    case 6: {  // the k-segment at (ra, pa) moves right after position pb of rb, kept or reversed
        const int k = m.k;
        if (!isB) return p < m.pa ? p : p + k;
        if (p <= m.pb) return p;
        if (p > m.pb + k) return p - k;
        const int q = p - m.pb - 1;
        fromB = false;
        return m.pa + (m.op == 5 ? q : k - 1 - q);
    }
    case 7:
    case 8:
    case 9: {  // segments (ra, pa, ka) and (rb, pb, kb) exchange places
        const int ka = m.op - 6, kb = m.k;
        if (!isB) {
            if (p < m.pa) return p;
            if (p >= m.pa + kb) return p - kb + ka;
            fromB = true;
            return m.pb + p - m.pa;
        }
        if (p < m.pb) return p;
        if (p >= m.pb + ka) return p - ka + kb;
        fromB = false;
        return m.pa + p - m.pb;
    }
    default: {
        const int i = m.pa, j = m.pb, k = m.k;
        if (j > i) {  // forward
            if (p < i || p > j) return p;
            return p <= j - k ? p + k : i + p - (j - k + 1);
        }
        if (p <= j || p >= i + k) return p;
        return p <= j + k ? i + p - j - 1 : p - k;
    }
    }
}

// Node at new position p of a touched route r.
__device__ __forceinline__ int new_node(const SolDev &S, const MoveInfo &m, int r, int p) {
    if (p == 0) return 0;
    bool fromB;
    const int q = new_src(m, r != m.ra, p, fromB);
    return old_node(S, fromB ? m.rb : m.ra, q);
}

// Operator, segment length and refs of a move id.
__device__ __forceinline__ void decode_id(const SolDev &S, uint32_t id, MoveInfo &m) {
    const uint32_t Q = (uint32_t)S.Q, qq = Q * Q;
    const uint32_t opk = id / qq, rem = id - opk * qq;
    m.id = id;
    m.op = (int)(opk >> 2);
    m.k = (int)(opk & 3);
    m.a = (int)(rem / Q);
    m.b = (int)(rem - (uint32_t)m.a * Q);
}

// With the refs' routes, positions and route lengths known: whether the id
// is a move of N(S), and the new lengths of the touched routes.
__device__ __forceinline__ void check_move(int n, MoveInfo &m) {
    const bool aC = m.a < n, bC = m.b < n;
    bool ok = false;
    m.nLa = m.La;
    m.nLb = m.Lb;
    switch (m.op) {
    case 0:
        ok = m.k == 1 && aC && m.ra != m.rb;
        m.nLa = m.La - 1;
        m.nLb = m.Lb + 1;
        break;
    case 1: ok = m.k == 1 && m.a < m.b && bC; break;
    case 2:
        ok = m.k == 0 && m.a < m.b && m.ra != m.rb;
        m.nLa = m.pa + m.Lb - m.pb;
        m.nLb = m.pb + m.La - m.pa;
        break;
    case 3: ok = m.k == 0 && m.a < m.b && bC && m.ra == m.rb; break;
    case 4:
        ok = m.k >= 1 && m.k <= 3 && aC && m.ra == m.rb && m.pa + m.k - 1 <= m.La &&
             !(m.pb >= m.pa - 1 && m.pb <= m.pa + m.k - 1);
        break;
    case 5:
    case 6:
        ok = m.k >= 2 && m.k <= 3 && aC && m.ra != m.rb && m.pa + m.k - 1 <= m.La;
        m.nLa = m.La - m.k;
        m.nLb = m.Lb + m.k;
        break;
    case 7:
    case 8:
    case 9: {  // cross-exchange of (a, op - 6) and (b, k)
        const int ka = m.op - 6, kb = m.k;
        ok = kb >= 1 && kb <= 3 && m.a < m.b && bC && m.ra != m.rb && m.pa + ka - 1 <= m.La &&
             m.pb + kb - 1 <= m.Lb && !(ka == 1 && kb == 1);
        m.nLa = m.La - ka + kb;
        m.nLb = m.Lb - kb + ka;
        break;
    }
    default: break;  // beyond the ten operators
    }
    m.valid = ok;
}

__device__ __forceinline__ void decode_move(const SolDev &S, uint32_t id, MoveInfo &m) {
    decode_id(S, id, m);
    const int sa = S.ref2slot[m.a], sb = S.ref2slot[m.b];
    m.ra = S.a4[sa].y;
    m.rb = S.a4[sb].y;
    m.pa = sa - S.roff[m.ra];
    m.pb = sb - S.roff[m.rb];
    m.La = S.roff[m.ra + 1] - S.roff[m.ra] - 1;
    m.Lb = S.roff[m.rb + 1] - S.roff[m.rb] - 1;
    check_move(S.n, m);
}

__device__ __forceinline__ void acc_add(const SolDev &S, int k, long long v) {
    if (v) atomicAdd((unsigned long long *)(S.acc + k), (unsigned long long)v);
}

// |N(S)| per operator after move m (one thread): the touched routes' terms
// change.  `acc` holds the accumulators as they were before.
__device__ __forceinline__ void count_move(const SolDev &S, const MoveInfo &m, const long long *acc) {
    if (m.ra == m.rb) return;
    const long long Q = S.Q;
    const RouteCounts a0 = route_counts(m.La, Q), a1 = route_counts(m.nLa, Q), b0 = route_counts(m.Lb, Q),
                      b1 = route_counts(m.nLb, Q);
    S.acc[kAccCnt0 + 0] = acc[kAccCnt0 + 0] + (a1.rel - a0.rel) + (b1.rel - b0.rel);
    S.acc[kAccCnt0 + 2] = acc[kAccCnt0 + 2] - ((a1.star2 - a0.star2) + (b1.star2 - b0.star2)) / 2;
    S.acc[kAccCnt0 + 3] = acc[kAccCnt0 + 3] + (a1.two - a0.two) + (b1.two - b0.two);
    S.acc[kAccCnt0 + 4] = acc[kAccCnt0 + 4] + (a1.oropt - a0.oropt) + (b1.oropt - b0.oropt);
    S.acc[kAccExtSeg] = acc[kAccExtSeg] + (a1.seg - a0.seg) + (b1.seg - b0.seg);
    S.acc[kAccExtK] = acc[kAccExtK] + (a1.k - a0.k) + (b1.k - b0.k);
    S.acc[kAccExtK2] = acc[kAccExtK2] + (a1.k2 - a0.k2) + (b1.k2 - b0.k2);
}

// Apply m (valid).  All threads of the block participate.  Every slot
// attribute is route-local, so only the touched routes are rebuilt; the
// routes strictly between two touched routes of different lengths move as a
// block by the first one's length change (a plain copy of their records).
// The cost and the violations change by the touched routes' difference
// (summing every route again took two rounds of the workgroup's threads and,
// after each rebuilt route, eight 64-bit reductions); |N(S)| is the caller's.
__device__ __forceinline__ void apply_move_block(const SolDev &S, const MoveInfo &m, ApplyShared &sh) {
    const int R = S.R, T = blockDim.x, tid = threadIdx.x;
    const bool inter = m.ra != m.rb;
    const int dA = m.nLa - m.La, dB = inter ? m.nLb - m.Lb : 0;
    auto shift = [&](int r) { return (r > m.ra ? dA : 0) + (inter && r > m.rb ? dB : 0); };
    const bool gen = S.pen || S.pd || S.gen;
    long long cost = 0, excess = 0, warps = 0;  // thread 0: less what the touched routes came to
    if (tid == 0) {
        cost -= gld(S.rdist + m.ra) + (inter ? gld(S.rdist + m.rb) : 0);
        if (gen) {
            excess -= route_excess(S, m.ra) + (inter ? route_excess(S, m.rb) : 0);
            warps -= route_warp(S, m.ra) + (inter ? route_warp(S, m.rb) : 0);
        }
    }
    // 1. new offsets, and the touched routes' nodes (read from the old layout)
    for (int r = tid; r <= R; r += T) S.roff_alt[r] = S.roff[r] + shift(r);
    const int baseA = S.roff[m.ra] + shift(m.ra);
    for (int p = tid; p <= m.nLa; p += T) S.nr_alt[baseA + p] = make_int2(new_node(S, m, m.ra, p), m.ra);
    int baseB = 0;
    if (inter) {
        baseB = S.roff[m.rb] + shift(m.rb);
        for (int p = tid; p <= m.nLb; p += T) S.nr_alt[baseB + p] = make_int2(new_node(S, m, m.rb, p), m.rb);
    }
    __threadfence_block();
    __syncthreads();
    // 2. routes strictly between the touched ones move by d; rounds of T
    //    slots, each read completely before it is written, taken in the
    //    direction of the move so no round overwrites a later one's source
    if (inter) {
        const int r1 = min(m.ra, m.rb), r2 = max(m.ra, m.rb);
        const int d = r1 == m.ra ? dA : dB;
        const int lo = S.roff[r1 + 1], hi = S.roff[r2];  // old slots of the routes between
        if (d != 0 && hi > lo) {
            const int rounds = (hi - lo + T - 1) / T;
            for (int k = 0; k < rounds; ++k) {
                const int rk = d < 0 ? k : rounds - 1 - k;
                const int src = lo + rk * T + tid;
                const bool on = src < hi;
                int4 a = make_int4(0, 0, 0, 0), b = a, t = a, w = a, pf = a, pb = a, pl = a, ql = a, g = a;
                int pd = 0;
                if (on) {
                    a = S.a4[src];
                    b = S.b4[src];
                    t = S.t4[src];
                    w = S.w4[src];
                    pd = S.pdist[src];
                    if (gen) {
                        pf = S.pf4[src];
                        pb = S.pb4[src];
                        pl = S.pl4[src];
                        ql = S.ql4[src];
                        g = S.g4[src];
                    }
                }
                __syncthreads();
                if (on) {
                    const int dst = src + d;
                    S.a4[dst] = a;
                    S.b4[dst] = b;
                    S.t4[dst] = t;
                    S.w4[dst] = w;
                    S.pdist[dst] = pd;
                    if (gen) {
                        S.pf4[dst] = pf;
                        S.pb4[dst] = pb;
                        S.pl4[dst] = pl;
                        S.ql4[dst] = ql;
                        S.g4[dst] = g;
                    }
                    const int node = nodeof(a.x);
                    S.ref2slot[(flagsof(a.x) & kFlagCustomer) ? node - 1 : S.n + a.y] = dst;
                }
                __threadfence_block();
                __syncthreads();
            }
        }
    }
    for (int r = tid; r <= R; r += T) S.roff[r] = S.roff_alt[r];
    __threadfence_block();
    __syncthreads();
    // 3. rebuild the touched routes in place
    rebuild_range<1>(S, S.nr_alt, S.roff_alt, baseA, baseA + m.nLa + 1, sh);
    if (inter) rebuild_range<1>(S, S.nr_alt, S.roff_alt, baseB, baseB + m.nLb + 1, sh);
    if (tid == 0) cost += gld(S.rdist + m.ra) + (inter ? gld(S.rdist + m.rb) : 0);
    if (gen) {  // summaries of the touched routes
        __shared__ GenRoute g[2];
        const int wave = threadIdx.x >> 6;
        if (wave == 0) gen_route_sums(S, m.ra, g[0]);
        if (wave == 1 && inter) gen_route_sums(S, m.rb, g[1]);
        __threadfence_block();
        __syncthreads();
        if (m.nLa >= 64) gen_slots(S, g, m.ra, baseA, baseA + m.nLa + 1);
        if (inter && m.nLb >= 64) gen_slots(S, g + 1, m.rb, baseB, baseB + m.nLb + 1);
        for (int k = 0; k < (inter ? 2 : 1); ++k) {
            excess += max(g[k].peak - S.cap, 0);
            warps += g[k].warp;
        }
    }
    if (tid == 0) {
        acc_add(S, kAccCost, cost);
        if (gen) {
            acc_add(S, kAccLoadExcess, excess);
            acc_add(S, kAccTimeWarp, warps);
        }
    }
}

// Local-search accounting of one evaluation (one thread): |N(S)| of the
// enabled operators (granular: the inter-route moves as counted) into
// acc[kAccMoves], and with kCountFull the slot pairs the
// screens visited.  `acc` holds the accumulators as they were before the
// step's move.
__device__ __forceinline__ void ls_count_moves(const SolDev &S, uint32_t op_mask, const long long *acc) {
    long long m = 0;
    if (op_mask & 32u) m += acc[kAccExtSeg];
    if (op_mask & 64u) m += acc[kAccExtSeg];
    if (op_mask & 128u)  // ordered pairs of customers of different routes: k(x) k(t) exchanges less the swap
        m += (acc[kAccExtK] * acc[kAccExtK] - (long long)S.n * S.n - acc[kAccExtK2]) / 2;
    if (op_mask & kGranular) {  // inter-route moves as counted; intra-route ones complete
        m = acc[kAccGranInter];
        if (op_mask & 2) m += acc[kAccCnt0 + 3];  // same-route swaps: L(L-1)/2 per route, as 2-opt
        if (op_mask & 8) m += acc[kAccCnt0 + 3];
        if (op_mask & 16) m += acc[kAccCnt0 + 4];
    } else {
        for (int op = 0; op < 5; ++op)
            if (op_mask >> op & 1) m += acc[kAccCnt0 + op];
    }
    S.acc[kAccMoves] = acc[kAccMoves] + m;
    if ((op_mask & kCountFull) && (op_mask & 7))
        S.acc[kAccScreenPairs] = acc[kAccScreenPairs] + acc[kAccCnt0 + 2];  // = slot pairs of different routes
}

// Moves the records of the slots [lo, hi) by d (routes strictly between the
// two touched ones).  Rounds of U slots per thread taken in the direction of
// the move, each read completely before it is written; between the first
// round's loads and its stores the caller's `between` runs (its loads
// overlap them).  Every thread of the block calls it; contains at least one
// barrier after `between`.
template <bool GEN, int U, class F>
__device__ __forceinline__ void shift_slots(const SolDev &S, int lo, int hi, int d, F between) {
    const int T = blockDim.x, tid = threadIdx.x;
    const int per = T * U, rounds = max(1, (hi - lo + per - 1) / per);
    for (int k = 0; k < rounds; ++k) {
        const int first = lo + (d < 0 ? k : rounds - 1 - k) * per + tid;
        int4 a[U], b[U], t[U], w[U], pf[U], pb[U], pl[U], ql[U], g[U];
        int pd[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int src = first + u * T;
            if (src < hi) {
                a[u] = gld(S.a4 + src);
                b[u] = gld(S.b4 + src);
                t[u] = gld(S.t4 + src);
                w[u] = gld(S.w4 + src);
                pd[u] = gld(S.pdist + src);
                if (GEN) {
                    pf[u] = gld(S.pf4 + src);
                    pb[u] = gld(S.pb4 + src);
                    pl[u] = gld(S.pl4 + src);
                    ql[u] = gld(S.ql4 + src);
                    g[u] = gld(S.g4 + src);
                }
            }
        }
        if (k == 0) between();
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int src = first + u * T, dst = src + d;
            if (src < hi) {
                gst(S.a4 + dst, a[u]);
                gst(S.b4 + dst, b[u]);
                gst(S.t4 + dst, t[u]);
                gst(S.w4 + dst, w[u]);
                gst(S.pdist + dst, pd[u]);
                if (GEN) {
                    gst(S.pf4 + dst, pf[u]);
                    gst(S.pb4 + dst, pb[u]);
                    gst(S.pl4 + dst, pl[u]);
                    gst(S.ql4 + dst, ql[u]);
                    gst(S.g4 + dst, g[u]);
                }
                gst(S.ref2slot + ((flagsof(a[u].x) & kFlagCustomer) ? nodeof(a[u].x) - 1 : S.n + a[u].y), dst);
            }
        }
    }
    if (rounds > 1) __syncthreads();  // the last round's sources may be the caller's destinations
}

// One block per solution.  kModeRecord: publish the best move (status 1 if
// none) and reset the key.  kModeLS: also apply it when its delta is negative
// and the step cap allows, else mark the solution converged.  kModeApplyRec:
// apply the move record the host wrote into S.rec.  host_out (nullable,
// single solution): pinned host memory that receives the move record and
// state[0..3] straight from the kernel (12 ints), so that no copy follows.
//
// The step is bound by the length of its chain of dependent memory reads
// (one workgroup, a few KB), so it has as few links as the data allow: key,
// state, accumulators and route offsets at once; the refs' slots; then the
// touched routes' nodes together with the records that move; then the
// distances.  The routes are found by comparing every route's slot range
// (one route per thread) with the two slots instead of following slot ->
// route -> offsets; the new routes are rebuilt in the registers of one
// wavefront each, the general path's summaries by further wavefronts at the
// same time; cost and |N(S)| change by the touched routes' difference.
// Measured per launch against a form that passed offsets, nodes and totals
// through memory with nine barriers and built the summaries in one thread per
// route: n = 1000 6.2 against 10.5 us, with time-warp summaries 6.9 against
// 17.8 us, with load summaries too (n = 603) 6.7 against 22.6 us, the 256
// solutions of 100..2000 customers 11.0 against 17.3 us.
//
// Every touched route must fit a wavefront (fewer than 64 customers, before
// and after); longer ones go through apply_move_block.
__device__ __forceinline__ void finalize_block(const SolDev &S, int mode, uint32_t op_mask, int32_t *host_out) {
    __shared__ ApplyShared sh;
    __shared__ int4 route_sh[2];  // {route, first slot, first slot of the next route, 0} of the two refs
    const int tid = threadIdx.x, T = blockDim.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool book = tid == T - 64;  // the thread that keeps the record, the state and the counters
    const int R = S.R, Q = S.Q;
    int done = S.state[kStDone];
    const int steps = S.state[kStSteps], max_steps = S.state[kStMaxSteps], version = S.state[kStVersion];
    const unsigned long long key = *S.best_key;
    long long acc[kAccCount];
    if (book)
        for (int q = 0; q < kAccCount; ++q) acc[q] = S.acc[q];
    int r_lo = 0, r_hi = 0;  // slot range of route tid
    if (mode != kModeRecord && tid < R) {
        r_lo = gld(S.roff + tid);
        r_hi = gld(S.roff + tid + 1);
    }
    MoveInfo m;
    m.valid = 0;
    m.delta = 0;
    bool skip = false;
    if (mode == kModeApplyRec) {
        m.delta = S.rec[4];
        decode_id(S, (uint32_t)S.rec[6], m);
    } else {
        skip = mode == kModeLS && done;
        if (!skip && key != ~0ull) {
            m.delta = (int)((uint32_t)(key >> 32) ^ 0x80000000u);
            decode_id(S, (uint32_t)(key & 0xFFFFFFFFu), m);
        }
    }
    const bool found = !skip && (mode == kModeApplyRec || key != ~0ull);
    // the move's routes, unless it is only recorded
    bool want = found && (mode == kModeApplyRec || (mode == kModeLS && m.delta < 0 && steps < max_steps));
    if (want) {
        const int sa = gld(S.ref2slot + m.a), sb = gld(S.ref2slot + m.b);
        for (int r = tid; r < R; r += T) {
            if (r != tid) {
                r_lo = gld(S.roff + r);
                r_hi = gld(S.roff + r + 1);
            }
            if (sa >= r_lo && sa < r_hi) route_sh[0] = make_int4(r, r_lo, r_hi, 0);
            if (sb >= r_lo && sb < r_hi) route_sh[1] = make_int4(r, r_lo, r_hi, 0);
        }
        __syncthreads();
        m.ra = __builtin_amdgcn_readfirstlane(route_sh[0].x);
        m.rb = __builtin_amdgcn_readfirstlane(route_sh[1].x);
        m.pa = __builtin_amdgcn_readfirstlane(sa - route_sh[0].y);
        m.pb = __builtin_amdgcn_readfirstlane(sb - route_sh[1].y);
        m.La = __builtin_amdgcn_readfirstlane(route_sh[0].z - route_sh[0].y - 1);
        m.Lb = __builtin_amdgcn_readfirstlane(route_sh[1].z - route_sh[1].y - 1);
        check_move(S.n, m);
        want = m.valid;
    } else {
        __syncthreads();  // everything above has been read
    }
    if (book && !skip) {
        if (mode == kModeApplyRec) {
            S.state[kStStatus] = m.valid ? 0 : -1;
        } else {
            *S.best_key = ~0ull;
            if (mode == kModeLS) ls_count_moves(S, op_mask, acc);
            S.acc[kAccGranInter] = 0;
            int rec[8] = {0, 0, 0, 0, 0, 0, 0, version};
            if (found) {
                rec[0] = m.op;
                rec[1] = m.k;
                rec[2] = m.a;
                rec[3] = m.b;
                rec[4] = m.delta;
                rec[5] = 3;
                rec[6] = (int)m.id;
            }
            for (int q = 0; q < 8; ++q) S.rec[q] = rec[q];
            S.state[kStStatus] = found ? 0 : 1;
            if (mode == kModeLS && !want) S.state[kStDone] = done = 1;
            if (host_out) {  // the record and state[0..3], straight into pinned host memory
                for (int q = 0; q < 8; ++q) host_out[q] = rec[q];
                host_out[8 + kStDone] = done;
                host_out[8 + kStSteps] = steps;
                host_out[8 + kStStatus] = found ? 0 : 1;
                host_out[8 + kStVersion] = version;
                // then the word the host waits for: everything this thread
                // wrote, here and in the workspace, is visible before it, and
                // in record mode nothing is written after it
                __threadfence_system();
                __hip_atomic_store(host_out + kHostDone, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            }
        }
    }
    if (!want) return;
    const bool inter = m.ra != m.rb;
    if (book) {
        S.state[kStVersion] = version + 1;
        S.state[kStSteps] = steps + 1;
        if (mode == kModeLS && steps + 1 >= max_steps) S.state[kStDone] = 1;
        count_move(S, m, acc);
    }
    if (max(max(m.La, m.Lb), max(m.nLa, m.nLb)) >= 64) {
        __syncthreads();
        apply_move_block(S, m, sh);
        return;
    }
    const bool gen = S.pen || S.pd || S.gen;
    const int offA = route_sh[0].y, offB = route_sh[1].y;
    const int dA = m.nLa - m.La, dB = inter ? m.nLb - m.Lb : 0;
    const int r1 = min(m.ra, m.rb), r2 = max(m.ra, m.rb);
    const int d = r1 == m.ra ? dA : dB;  // shift of the routes between and of the later one's start
    const bool moves = inter && d != 0;
    const int lo = r1 == m.ra ? route_sh[0].z : route_sh[1].z, hi = r1 == m.ra ? offB : offA;
    const int baseA = offA + (moves && m.ra == r2 ? d : 0), baseB = offB + (moves && m.rb == r2 ? d : 0);
    // wavefronts 0 / 1: the attributes of route ra / rb; 2 / 3 and 4 / 5 on
    // the general path: their time-warp and load summaries
    const bool isB = wave & 1;
    const int role = wave >> 1;
    const bool works = (!isB || inter) && (role == 0 || (role == 1 && gen && S.has_tw) || (role == 2 && S.pd));
    const int L = isB ? m.nLb : m.nLa, base = isB ? baseB : baseA, r = isB ? m.rb : m.ra, off = isB ? offB : offA;
    SlotAttr x;  // role 0: the slot's attributes; roles 1 and 2: prefix summary in x.a, suffix summary in x.b
    int2 rem = make_int2(0, 0);
    int old = 0, old_load = 0;
    auto route = [&]() {
        if (!works) return;
        const int na = lane <= m.La ? nodeof(gld(S.a4 + offA + lane).x) : 0;
        const int nb = inter && lane <= m.Lb ? nodeof(gld(S.a4 + offB + lane).x) : 0;
        if (role == 0) {
            old = gld(S.rdist + r);
            old_load = gld(S.b4 + off).z;
        } else {
            old = role == 1 ? gld(S.pb4 + off).w : gld(S.ql4 + off).z;
        }
        bool fromB;
        const int q = new_src(m, isB, max(lane, 1), fromB);
        const int qa = __shfl(na, q & 63), qb = __shfl(nb, q & 63);
        const int node = lane == 0 || lane > L ? 0 : (fromB && inter ? qb : qa);
        if (role == 0) {
            x = route_attr(S, node, r, L);
            if (gen) rem = segment_removal(S, node, x.a.z, L);
        } else if (role == 1) {
            Tw f, b;
            tw_route_wave(S, node, L, f, b);
            x.a = tw_pack(f);
            x.b = tw_pack(b);
        } else {
            Ld f, b;
            ld_route_wave(S, node, L, f, b);
            x.a = ld_pack(f);
            x.b = ld_pack(b);
        }
    };
    if (gen)
        shift_slots<true, 1>(S, lo, moves ? hi : lo, d, route);
    else
        shift_slots<false, 2>(S, lo, moves ? hi : lo, d, route);
    if (works) {
        if (role == 0) {
            store_attr(S, x, r, base, L);
            if (gen && lane <= L) {  // the other wavefronts add what they know
                int *g = (int *)(S.g4 + base + lane);
                gst((int2 *)g, rem);
                if (!S.pd) gst(g + 2, x.b.z);
                if (!S.has_tw) gst(g + 3, 0);
            }
            if (lane == L) acc_add(S, kAccCost, (long long)x.rdist - old);
            if (lane == 0 && gen && !S.pd)
                acc_add(S, kAccLoadExcess, (long long)max(x.b.z - S.cap, 0) - max(old_load - S.cap, 0));
        } else if (role == 1) {
            if (lane <= L) {
                gst(S.pf4 + base + lane, x.a);
                gst(S.pb4 + base + lane, x.b);
                gst((int *)(S.g4 + base + lane) + 3, __shfl(x.b.w, 0));
            }
            if (lane == 0) acc_add(S, kAccTimeWarp, (long long)x.b.w - old);
        } else {
            if (lane <= L) {
                gst(S.pl4 + base + lane, x.a);
                gst(S.ql4 + base + lane, x.b);
                gst((int *)(S.g4 + base + lane) + 2, __shfl(x.b.z, 0));
            }
            if (lane == 0) acc_add(S, kAccLoadExcess, (long long)max(x.b.z - S.cap, 0) - max(old - S.cap, 0));
        }
    }
    if (moves)
        for (int q = tid; q < R; q += T)
            if (q > r1 && q <= r2) gst(S.roff + q, gld(S.roff + q) + d);
}

// `steps` (nullable): a batch's step counter, advanced once per launch.
// Empty slots of a slot batch (Q = 0) are skipped.
__global__ __launch_bounds__(kApplyThreads) void k_finalize(const SolDev *__restrict__ sols, int mode,
                                                            uint32_t op_mask, int *__restrict__ steps) {
    if (steps && blockIdx.x == 0 && threadIdx.x == 0) *steps += 1;
    if (sols[blockIdx.x].Q == 0) return;
    finalize_block(sols[blockIdx.x], mode, op_mask, nullptr);
}

// The same for one solution, its descriptor by value (see k_eval_solution).
__global__ __launch_bounds__(kApplyThreads) void k_finalize_one(const SolDev S, int mode, uint32_t op_mask,
                                                                int32_t *__restrict__ host_out) {
    finalize_block(S, mode, op_mask, host_out);
}

// ------------------------------------------------------------ multi-move --
// Several independent moves per step (Section 7, after Dynasearch): the
// candidates are the per-route-pair bests of the last evaluation
// (S.pairkey); taken in (delta, id) order, a candidate is selected when
// neither of its routes is used by an earlier selection.  Moves on disjoint
// routes keep their deltas and feasibility when applied one after another.
// The greedy set is found in rounds of locally dominant candidates: a
// candidate whose key is the smallest among the candidates at each of its
// (free) routes is taken by the sequential greedy too (no smaller key can
// take one of its routes first), and the candidates dominant in one round
// share no route; repeating on the routes still free gives the greedy set in
// a few rounds (sorting the candidates and going down them in one thread took
// most of a launch of 170 us at n = 1000, against 37 us, and 11 us for the
// layout's build).  Up to kMultiCands candidates are kept in LDS for
// the rounds, more are read from the table each time.  Requires
// R <= kMultiMaxR.
constexpr int kMultiCands = 2048;
constexpr int kMultiMaxR = 4096;

__device__ __forceinline__ bool key_improving(unsigned long long k) { return k < 0x8000000000000000ull; }

struct MultiShared {
    unsigned long long best[kMultiMaxR];   // per route: least key of its candidates
    unsigned long long key[kMultiCands];   // candidates
    int pair[kMultiCands];                 // their routes, r1 << 16 | r2
};
// the selected moves decoded, and per route the selected move touching it
constexpr int kMultiMoves = (int)((sizeof(MultiShared) - 4 * kMultiMaxR) / sizeof(MoveInfo));
struct MultiApply {
    int mov_of[kMultiMaxR];
    MoveInfo mv[kMultiMoves];
};
static_assert(sizeof(MultiApply) <= sizeof(MultiShared), "multi-move LDS");

// kModeRecord: selection only, written to S.msel in (delta, id) order.
// kModeLS: also put the new layout of the routes into roff_alt and nr_alt for
// k_build_routes (kStBuild), count the step, and mark the solution converged
// when nothing is selected or the step cap is reached.  Clears S.pairkey.
__global__ __launch_bounds__(kApplyThreads) void k_multi_step(const SolDev S, int mode, uint32_t op_mask) {
    __shared__ ApplyShared sh;
    __shared__ MoveInfo mi;
    __shared__ MultiShared ms;
    __shared__ unsigned char used[kMultiMaxR];
    __shared__ int cnt_sh, nsel_sh, long_sh;
    __shared__ unsigned long long first_sh;
    const int tid = threadIdx.x, T = blockDim.x, R = S.R, lane = tid & 63, wave = tid >> 6;
    const size_t RR = (size_t)R * R;
    if (mode == kModeLS && S.state[kStDone]) return;
    if (tid == 0) {
        cnt_sh = nsel_sh = long_sh = 0;
        first_sh = ~0ull;
        if (mode == kModeLS) ls_count_moves(S, op_mask, S.acc);
        S.acc[kAccGranInter] = 0;
        *S.best_key = ~0ull;
    }
    for (int r = tid; r < R; r += T) used[r] = 0;
    __syncthreads();
    // 1. compact the improving candidates (one LDS atomic per wavefront), and
    // clear the table for the next evaluation when they all fit
    for (size_t q0 = 0; q0 < RR; q0 += T) {
        const size_t q = q0 + tid;
        const unsigned long long k = q < RR ? S.pairkey[q] : ~0ull;
        const bool on = key_improving(k);
        const unsigned long long mask = __builtin_amdgcn_ballot_w64(on);
        if (!mask) continue;
        int at = 0;
        if (lane == 0) at = atomicAdd(&cnt_sh, __builtin_popcountll(mask));
        at = __builtin_amdgcn_readfirstlane(at) +
             __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
        if (on && at < kMultiCands) {
            const int r1 = (int)((uint32_t)q / (uint32_t)R);
            ms.key[at] = k;
            ms.pair[at] = (r1 << 16) | ((int)q - r1 * R);
        }
    }
    __syncthreads();
    const bool in_lds = cnt_sh <= kMultiCands;
    const size_t count = in_lds ? (size_t)cnt_sh : RR;
    if (in_lds)
        for (size_t q = tid; q < RR; q += T) S.pairkey[q] = ~0ull;
    // 2. rounds of locally dominant candidates
    int32_t *sel = S.msel + 1;  // (id, delta) per selected move
    auto candidate = [&](size_t q, unsigned long long &k, int &r1, int &r2) {
        if (in_lds) {
            k = ms.key[q];
            r1 = ms.pair[q] >> 16;
            r2 = ms.pair[q] & 0xFFFF;
        } else {
            k = S.pairkey[q];
            if (!key_improving(k)) return false;
            r1 = (int)((uint32_t)q / (uint32_t)R);
            r2 = (int)q - r1 * R;
        }
        return !used[r1] && !used[r2];
    };
    for (int before = 0;;) {
        for (int r = tid; r < R; r += T) ms.best[r] = ~0ull;
        __syncthreads();
        unsigned long long k;
        int r1, r2;
        for (size_t q = tid; q < count; q += T)
            if (candidate(q, k, r1, r2)) {
                if (k < ms.best[r1]) atomicMin(&ms.best[r1], k);
                if (k < ms.best[r2]) atomicMin(&ms.best[r2], k);
            }
        __syncthreads();
        // a dominant candidate's routes are its own in this round, so marking
        // them disturbs no other dominant one
        for (size_t q = tid; q < count; q += T)
            if (candidate(q, k, r1, r2) && ms.best[r1] == k && ms.best[r2] == k) {
                const int slot = atomicAdd(&nsel_sh, 1);  // < R: the taken candidates share no route
                sel[2 * slot] = (int32_t)(uint32_t)(k & 0xFFFFFFFFu);
                sel[2 * slot + 1] = (int)((uint32_t)(k >> 32) ^ 0x80000000u);
                used[r1] = used[r2] = 1;
                atomicMin(&first_sh, k);
            }
        __syncthreads();
        const int now = nsel_sh;
        if (now == before) break;
        before = now;
    }
    const int ns = nsel_sh;
    if (!in_lds)
        for (size_t q = tid; q < RR; q += T) S.pairkey[q] = ~0ull;
    __threadfence_block();
    __syncthreads();
    if (tid == 0) S.msel[0] = ns;
    if (mode != kModeLS) {
        // (delta, id) order: sort the selection's keys (bitonic, in LDS; ns <= R)
        unsigned long long *keys = ms.best;
        int np2 = 1;
        while (np2 < ns) np2 <<= 1;
        for (int q = tid; q < np2; q += T)
            keys[q] = q < ns ? pack_key(sel[2 * q + 1], (uint32_t)sel[2 * q]) : ~0ull;
        __syncthreads();
        for (int kk = 2; kk <= np2; kk <<= 1)
            for (int jj = kk >> 1; jj > 0; jj >>= 1) {
                for (int q = tid; q < np2; q += T) {
                    const int p2 = q ^ jj;
                    if (p2 > q) {
                        const bool up = (q & kk) == 0;
                        const unsigned long long a = keys[q], b = keys[p2];
                        if ((a > b) == up) {
                            keys[q] = b;
                            keys[p2] = a;
                        }
                    }
                }
                __syncthreads();
            }
        for (int q = tid; q < ns; q += T) {
            sel[2 * q] = (int32_t)(uint32_t)(keys[q] & 0xFFFFFFFFu);
            sel[2 * q + 1] = (int)((uint32_t)(keys[q] >> 32) ^ 0x80000000u);
        }
        return;
    }
    // 3. the new layout.  Routes are disjoint, so it is the old one with each
    // touched route replaced by its new node sequence, whatever the order of
    // the moves.  A selection too large for the LDS is applied move by move
    // instead.
    MultiApply &ma = reinterpret_cast<MultiApply &>(ms);
    const bool one_by_one = ns > kMultiMoves;
    if (ns > 0 && !one_by_one) {
        int *mov_of = ma.mov_of;
        for (int r = tid; r < R; r += T) mov_of[r] = -1;
        __syncthreads();
        for (int q = tid; q < ns; q += T) {
            MoveInfo m;
            decode_move(S, (uint32_t)sel[2 * q], m);
            m.delta = sel[2 * q + 1];
            ma.mv[q] = m;
            if (m.valid) {
                mov_of[m.ra] = q;
                mov_of[m.rb] = q;
            }
        }
        __syncthreads();
        auto newL = [&](int r) {
            const int q = mov_of[r];
            if (q < 0) return S.roff[r + 1] - S.roff[r] - 1;
            return r == ma.mv[q].ra ? ma.mv[q].nLa : ma.mv[q].nLb;
        };
        // new offsets: an exclusive scan of newL over the routes (each thread
        // a contiguous run of routes, then the threads' totals)
        const int per = (R + T - 1) / T, r0 = min(tid * per, R), r1 = min(r0 + per, R);
        int own = 0;
        for (int r = r0; r < r1; ++r) {
            const int l = newL(r);
            own += l;
            if (l >= 64) long_sh = 1;
        }
        int incl = own;
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(incl, off);
            if (lane >= off) incl += v;
        }
        if (lane == 63) sh.red[wave][0] = incl;
        __syncthreads();
        int before = incl - own;
        for (int w = 0; w < wave; ++w) before += (int)sh.red[w][0];
        for (int r = r0; r < r1; ++r) {
            S.roff_alt[r] = before;
            before += newL(r);
        }
        if (tid == 0) S.roff_alt[R] = S.n;
        __threadfence_block();
        __syncthreads();
        // customers of the new layout, one wavefront per route
        int32_t *cust = (int32_t *)S.nr_alt;
        for (int r = wave; r < R; r += T / 64) {
            const int q = mov_of[r], base = S.roff_alt[r], nl = newL(r);
            for (int p = lane; p < nl; p += 64)
                cust[base + p] = q < 0 ? old_node(S, r, p + 1) : new_node(S, ma.mv[q], r, p + 1);
        }
        // |N(S)| changes by the touched routes' terms
        long long d[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int q = tid; q < ns; q += T) {
            const MoveInfo &m = ma.mv[q];
            if (!m.valid) continue;
            d[0] += 1;
            if (m.ra == m.rb) continue;
            const RouteCounts a0 = route_counts(m.La, S.Q), a1 = route_counts(m.nLa, S.Q),
                              b0 = route_counts(m.Lb, S.Q), b1 = route_counts(m.nLb, S.Q);
            d[1] += a1.rel - a0.rel + b1.rel - b0.rel;
            d[2] -= (a1.star2 - a0.star2 + b1.star2 - b0.star2) / 2;
            d[3] += a1.two - a0.two + b1.two - b0.two;
            d[4] += a1.oropt - a0.oropt + b1.oropt - b0.oropt;
            d[5] += a1.seg - a0.seg + b1.seg - b0.seg;
            d[6] += a1.k - a0.k + b1.k - b0.k;
            d[7] += a1.k2 - a0.k2 + b1.k2 - b0.k2;
        }
        __syncthreads();
        for (int i = 0; i < 8; ++i) {
            long long v = d[i];
            for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
            if (lane == 0) sh.red[wave][i] = v;
        }
        __syncthreads();
        if (tid < 8) {
            long long v = 0;
            for (int w = 0; w < T / 64; ++w) v += sh.red[w][tid];
            const int to[8] = {-1, kAccCnt0, kAccCnt0 + 2, kAccCnt0 + 3, kAccCnt0 + 4, kAccExtSeg, kAccExtK, kAccExtK2};
            if (tid == 0) S.state[kStVersion] += (int)v;
            else S.acc[to[tid]] += v;
        }
        if (tid == 0) S.state[kStBuild] = long_sh ? 2 : 1;
    }
    if (one_by_one)
        for (int q = 0; q < ns; ++q) {
            if (tid == 0) {
                decode_move(S, (uint32_t)sel[2 * q], mi);
                mi.delta = sel[2 * q + 1];
            }
            __syncthreads();
            const MoveInfo m = mi;
            if (m.valid) apply_move_block(S, m, sh);
            __syncthreads();
            if (tid == 0 && m.valid) {
                S.state[kStVersion] += 1;
                count_move(S, m, S.acc);
            }
        }
    if (tid == 0) {
        if (ns > 0) {  // the record holds the first (best) selected move
            S.rec[4] = (int)((uint32_t)(first_sh >> 32) ^ 0x80000000u);
            S.rec[6] = (int32_t)(uint32_t)(first_sh & 0xFFFFFFFFu);
            S.state[kStSteps] += 1;
            S.acc[kAccMultiApplied] += ns;
            S.state[kStStatus] = 0;
        } else {
            S.state[kStStatus] = 1;
        }
        if (ns == 0 || S.state[kStSteps] >= S.state[kStMaxSteps]) S.state[kStDone] = 1;
    }
}

// ------------------------------------------------------ instance checks ----
// out[0] |= 1 value out of range, 2 asymmetric, 4 nonzero diagonal,
//           8 bad node data; out[1] = max distance; out[2] = max e;
// out[3] = max l; out[4] = max s; out[5] = max demand (all zero before).
//
// One pass over D: workgroup (I, J), I <= J, takes the 64 x 64 tiles (I, J)
// and (J, I), compares them across the diagonal, and writes both into the
// 16-bit copy (rows padded to `stride` with zeros; of no use when a distance
// turns out wider).  Bound by memory: 4 bytes read and 2 written per entry.
// The maxima go to one address, where atomics are taken one after the other,
// so only a larger value is sent, once per workgroup.  (Tiles of 32 read from
// both sides, an atomic per wavefront and a second pass for the copy: 308 us
// at n = 2500 against 17.)  Diagonal workgroups also check the nodes of their
// rows.
constexpr int kCheckTile = 64;

__device__ __forceinline__ void raise(int32_t *p, int v) {
    if (v > __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(p, v);
}

__global__ __launch_bounds__(256) void k_check_instance(const int32_t *__restrict__ D, int np1, int stride,
                                                        uint16_t *__restrict__ D16, const int4 *__restrict__ nd,
                                                        int has_tw, int32_t *__restrict__ out) {
    __shared__ int ta[kCheckTile][kCheckTile + 1];
    __shared__ int red[4][2];
    const int I = blockIdx.y, J = blockIdx.x;
    const int tid = threadIdx.x, x = tid & 63, wave = tid >> 6;
    if (I <= J) {  // uniform for the workgroup
        int bad = 0, mx = 0;
        auto tile = [&](int bi, int bj, bool second) {
            const int j = bj * kCheckTile + x;
            int v[kCheckTile / 4];
#pragma unroll
            for (int u = 0; u < kCheckTile / 4; ++u) {
                const int i = bi * kCheckTile + 4 * u + wave;
                v[u] = i < np1 && j < np1 ? gld(D + (size_t)i * np1 + j) : 0;
            }
#pragma unroll
            for (int u = 0; u < kCheckTile / 4; ++u) {
                const int y = 4 * u + wave, i = bi * kCheckTile + y;
                if (v[u] < 0 || v[u] >= (1 << 24)) bad |= 1;
                mx = max(mx, v[u]);
                if (!second) ta[y][x] = v[u];
                else if (v[u] != ta[x][y]) bad |= 2;
                if (i == j && v[u] != 0) bad |= 4;
                if (i < np1 && j < stride) D16[(size_t)i * stride + j] = (uint16_t)v[u];
            }
        };
        tile(I, J, false);
        __syncthreads();
        if (I != J) {
            tile(J, I, true);
        } else {
            for (int y = wave; y < kCheckTile; y += 4)
                if (ta[y][x] != ta[x][y]) bad |= 2;
            const int i = I * kCheckTile + x;
            if (wave == 0) {
                const int4 q = i < np1 ? nd[i] : make_int4(0, 0, 0, 0);
                const int lim = 1 << 26;
                bool wrong = q.x < 0 || q.x >= lim || (i == 0 && q.x != 0);
                if (has_tw)
                    wrong = wrong || q.y < 0 || q.z < q.y || q.w < 0 || q.z >= lim || q.w >= lim || (i == 0 && q.w != 0);
                if (wrong) bad |= 8;
                int m[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    for (int off = 32; off >= 1; off >>= 1) m[k] = max(m[k], __shfl_xor(m[k], off));
                    if (x == 0 && (k == 0 || has_tw)) raise(&out[k == 0 ? 5 : 1 + k], m[k]);
                }
            }
        }
        for (int off = 32; off >= 1; off >>= 1) {
            bad |= __shfl_xor(bad, off);
            mx = max(mx, __shfl_xor(mx, off));
        }
        if (x == 0) {
            red[wave][0] = bad;
            red[wave][1] = mx;
        }
        __syncthreads();
        if (tid == 0) {
            bad = red[0][0] | red[1][0] | red[2][0] | red[3][0];
            mx = max(max(red[0][1], red[1][1]), max(red[2][1], red[3][1]));
            if (bad) atomicOr(&out[0], bad);
            raise(&out[1], mx);
        }
    }
}

// Check results to pinned host memory.
__global__ void k_check_done(const int32_t *__restrict__ out, int32_t *__restrict__ host_out) {
    if (threadIdx.x < 8) host_out[threadIdx.x] = out[threadIdx.x];
}

// Pickup amounts: chk[0] |= 1 for a negative amount or a nonzero depot
// entry; chk[1] = the largest amount.
__global__ __launch_bounds__(256) void k_check_pick(const int32_t *__restrict__ pick, int np1, int32_t *chk) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= np1) return;
    const int v = pick[i];
    if (v < 0 || (i == 0 && v != 0)) atomicOr(chk, 1);
    atomicMax(chk + 1, v);
}

__global__ void k_fill_u64(unsigned long long *p, size_t count) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x)
        p[i] = ~0ull;
}

__global__ void k_zero_i32(int32_t *p, int count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0;
}

// Gather the converged flags of a batch into one array (one copy to the
// host); an empty slot reads as converged.
__global__ void k_poll_done(const SolDev *__restrict__ sols, int nsols, int32_t *out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nsols) out[i] = sols[i].Q == 0 ? 1 : sols[i].state[kStDone];
}

// Per-solution results of a batch in one array: {steps, version | converged
// << 32, moves evaluated, cost} per solution, for a single copy to the host
// (an empty slot: zeros, converged).
__global__ void k_collect(const SolDev *__restrict__ sols, int nsols, long long *out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nsols) {
        const SolDev &S = sols[i];
        if (S.Q == 0) {
            out[4 * i] = 0;
            out[4 * i + 1] = 1ll << 32;
            out[4 * i + 2] = 0;
            out[4 * i + 3] = 0;
            return;
        }
        out[4 * i] = S.state[kStSteps];
        out[4 * i + 1] = (long long)(uint32_t)S.state[kStVersion] | ((long long)(S.state[kStDone] != 0) << 32);
        out[4 * i + 2] = S.acc[kAccMoves];
        out[4 * i + 3] = S.acc[kAccCost];
    }
}

// Reset per-solution state for a new run (no memset, so it can sit in a
// captured graph).
__global__ void k_reset_state(const SolDev *__restrict__ sols, int nsols, int max_steps) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nsols || sols[i].Q == 0) return;
    reset_run(sols[i], max_steps);
}

__global__ void k_reset_one(const SolDev S, int max_steps) { reset_run(S, max_steps); }

// Measurement aid: reads `chunks` KiB from src into LDS with the 16-byte
// LDS DMA that stages 16-bit distance rows (one KiB per wavefront
// instruction) and discards them, so that a profiler's fetch counter can be
// scaled for exactly that kind of request.  Each wavefront cycles through
// four 1 KiB slots of its own and drains them every fourth instruction.
__global__ __launch_bounds__(256) void k_probe_stream(const int *__restrict__ src, long long chunks) {
    __shared__ int4 buf[4 * 4 * 64];  // 4 wavefronts x 4 slots x 1 KiB
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int k = 0;
    for (long long c = (long long)blockIdx.x * 4 + wave; c < chunks; c += (long long)gridDim.x * 4) {
        int *dst = (int *)(buf + (wave * 4 + (k & 3)) * 64);
        __builtin_amdgcn_global_load_lds((global_void_ptr)(src + c * 256 + 4 * lane), (lds_void_ptr)dst, 16, 0, 0);
        if ((++k & 3) == 0) __builtin_amdgcn_s_waitcnt(0);
    }
    __builtin_amdgcn_s_waitcnt(0);
}

// Sum of the screening counters over a batch's solutions (one thread).
__global__ void k_screen_sum(const SolDev *__restrict__ sols, int nsols, long long *out) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    long long f = 0, p = 0;
    for (int i = 0; i < nsols; ++i)
        if (sols[i].Q) {
            f += sols[i].acc[kAccFullPairs];
            p += sols[i].acc[kAccScreenPairs];
        }
    out[0] = f;
    out[1] = p;
}

}  // namespace tga
