// Device helpers shared by the plan-evaluation kernels (eval.hip: next-fit
// batching; firstfit.hip: first-fit and seed batching): wave scans, location
// arithmetic, the time-window rate, the instance of a plan row, and the route
// of one tour from its picks (section 5, Subproblem 2).
#pragma once

#include "wo_internal.h"

namespace wo {

// Tables that are not written while the kernel runs (copies and earlier kernels of
// the stream fill them), as constant memory: at a uniform address their
// values come by scalar loads into scalar registers.  (Through plain pointers
// every field of a plan's instance is a vector load and a lane read, since a
// store or a barrier might have changed it: a chain of some six trips to memory
// before a plan of a batch could start.  128 uneven instances x 256 plans 242 to
// 229 us, 4,096 paper-scale plans 74 to 72 us, in first fit 310 to 275 us.)
#define WO_CONST const __attribute__((address_space(4)))
typedef WO_CONST InstDev InstConst;
template <class T>
static __device__ __forceinline__ WO_CONST T *as_const(const T *p) { return (WO_CONST T *)(size_t)p; }

// Inclusive prefix sum over the 64 lanes of a wave (all lanes active): shifts
// by 1, 2, 4, 8 inside each row of 16 lanes, then the row totals carried by
// the row broadcasts of lanes 15 and 31.
static __device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);   // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);   // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);   // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);   // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);   // row_bcast:15
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);   // row_bcast:31
    return x;
}

// x with lane l (uniform) set to v (uniform): v_writelane
extern "C" __device__ int wo_writelane_i32(int src, int lane, int old) __asm("llvm.amdgcn.writelane.i32");
static __device__ __forceinline__ uint32_t set_lane(uint32_t x, uint32_t v, int l)
{
    return (uint32_t)wo_writelane_i32((int)v, l, (int)x);
}

// Whether this lane's bit of a uniform mask is set: the mask serves as the
// condition itself, with no shift per lane.
static __device__ __forceinline__ bool lane_in(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// A wave's LDS accesses take effect in program order: only the compiler must
// keep it between accesses of different lanes of one wave.
static __device__ __forceinline__ void lds_order() { asm volatile("" ::: "memory"); }

// Smallest value over the 64 lanes of a wave (all lanes active), the same
// shifts and broadcasts; every lane gets it.
static __device__ __forceinline__ uint32_t wave_min_u32(uint32_t v)
{
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x111, 0xF, 0xF, false));   // row_shr:1
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x112, 0xF, 0xF, false));   // row_shr:2
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x114, 0xF, 0xF, false));   // row_shr:4
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x118, 0xF, 0xF, false));   // row_shr:8
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x142, 0xA, 0xF, false));   // row_bcast:15
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x143, 0xC, 0xF, false));   // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

static __device__ __forceinline__ uint32_t mulhi24(uint32_t x, uint32_t m)
{
    return (uint32_t)(((uint64_t)(x & 0xFFFFFFu) * (uint64_t)(m & 0xFFFFFFu)) >> 32);
}

// a * b and a * b + c by the low 24 bits of a and b: full-rate instructions,
// which the compiler does not see past a value that it cannot bound.
static __device__ __forceinline__ uint32_t mul24(uint32_t a, uint32_t b)
{
    uint32_t r;
    asm("v_mul_u32_u24 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
static __device__ __forceinline__ uint32_t mad24(uint32_t a, uint32_t b, uint32_t c)
{
    uint32_t r;
    asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

static __device__ __forceinline__ float window_throughput(int64_t D, InstConst &I)
{
    // T = D / walk + t_item * items; orders * window / T: IEEE double, one
    // operation at a time (no multiply-add contraction), rounded once
#pragma clang fp contract(off)
    const double q = (double)D / I.walk;
    const double u = I.t_item * (double)I.n_lines;
    const double T = q + u;
    const double r = ((double)I.n_orders * I.window) / T;
    return (float)r;
}

// Instance of plan row p: from the per-plan table when there is one, else the
// last instance whose first row is <= p.
static __device__ __forceinline__ int instance_of(const EvalArgs &A, int64_t p)
{
    if (A.n_inst <= 1) return 0;
    if (A.plan_inst) return as_const(A.plan_inst)[p];
    int lo = 0, hi = A.n_inst - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (as_const(A.plan_begin)[mid] <= p) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Ascending sort of 32 words held in registers: Batcher's odd-even merge
// network, 191 exchanges of straight-line min and max (a bitonic one has 240).
static __device__ __forceinline__ void sort32(uint32_t (&v)[MAX_PICK_SLOTS])
{
#pragma unroll
    for (int p = 1; p < MAX_PICK_SLOTS; p <<= 1)
#pragma unroll
        for (int k = p; k > 0; k >>= 1)
#pragma unroll
            for (int i = 0; i < MAX_PICK_SLOTS; i++) {
                const int l = i + k;
                // pairs k apart from k % p on, inside one block of 2 p
                const bool pair = i >= k % p && ((i - k % p) & k) == 0 && l < MAX_PICK_SLOTS && i / (2 * p) == l / (2 * p);
                if (pair) {
                    const uint32_t a = v[i], b = v[l];
                    v[i] = min(a, b);
                    v[l] = max(a, b);
                }
            }
}

// Optimal route of one tour (the minimum route distance of section 5,
// Subproblem 2) in the manner of Ratliff and Rosenthal: a programme over the
// aisles holding picks, left to right.  A partial walk is in one of five
// classes at the two ends (front f, back b) of the last aisle decided:
//   O1: f and b of odd degree, one component;
//   F : only f in the walk (even degree);
//   B : only b in the walk (even degree);
//   E1: f and b of even degree, one component;
//   E2: f and b of even degree, two components.
// The costs leave out 2w for every step along the cross aisles, which every
// walk pays at least, so a step costs nothing in O1, F and B (one edge each way,
// or both on one side) and 2w in E1 and E2 (4w in all).  They are unsigned: a
// tour's distances are bounded at load so that every class cost stays below
// 2^30, and the unreachable value OPT_INF plus any sum of additions below 2^32.
// The programme is the larger part of the route's time (30 picks of a tour on
// one lane, a chain of dependent minima), so each form below is the shortest
// one found; the identities that shorten it are exact.
#define OPT_INF 0x40000000u
struct OptClasses { uint32_t o1, f, b, e1, e2; };

// The classes before the first aisle with picks, r steps from the depot at
// the front of aisle 0; without picks that aisle may be crossed once (O1) or
// twice (E1, and B once its front end is dropped).
static __device__ __forceinline__ OptClasses opt_start(uint32_t r, uint32_t w2, uint32_t L)
{
    return {r ? L : OPT_INF, 0u, r ? 2u * L : OPT_INF, r ? 2u * L + w2 : OPT_INF, OPT_INF};
}

// Carry the classes over r >= 1 steps to the next aisle with picks (r - 1
// aisles without picks in between; ar = 2w r, w2 = 2w).  E1 may drop an end.  In
// the aisles passed, a class may change by a crossing (cost L) or a double
// crossing (2 L); the cheapest such change is taken as early as it lowers the
// step cost and as late as it raises it.  Every double crossing is two single
// ones by way of O1, so that X = O1 + L, O1 being the new one, stands for all
// that lead to F, B and E1.  Afterwards F, B < E1.
static __device__ __forceinline__ void opt_run(OptClasses &s, uint32_t r, uint32_t ar, uint32_t w2, uint32_t L)
{
    const uint32_t Lr = r >= 2u ? L : OPT_INF;      // no aisle without picks: no change
    const uint32_t m = min(min(s.f, s.b), s.e1);
    s.o1 = min(s.o1, min(m, s.e2 + w2) + Lr);
    const uint32_t X = s.o1 + Lr;
    s.f = min(min(s.f, s.e1), X);
    s.b = min(min(s.b, s.e1), X);
    s.e1 = min(s.e1 + ar, X + w2);
    s.e2 += ar;
}

// The aisle's own edges: a crossing (L), a double crossing (2 L), in from the
// front to the last pick (cF), in from the back to the first pick (cB), or in
// from both sides leaving out the largest gap between two picks (cG; 2 L when
// the aisle has a single pick, which never beats cF or cB then).
static __device__ __forceinline__ void opt_aisle(OptClasses &s, uint32_t L, uint32_t cF, uint32_t cB, uint32_t cG)
{
    const uint32_t cBG = min(cB, cG), cFG = min(cF, cG), cmin = min(cF, cBG);
    const uint32_t m = min(min(s.f, s.b), s.e2);    // E1 is above F here
    const uint32_t o1 = s.o1;
    s.o1 = min(o1 + cmin, m + L);
    s.e2 = min(min(s.f + cBG, s.b + cFG), s.e2 + cmin);
    s.e1 = min(min(o1 + L, s.e1 + cmin), m + 2u * L);
    s.f += cF;
    s.b += cB;
}

// Walk of one tour for the return, largest-gap, combined or optimal route,
// fed the tour's picks one at a time sorted by scaled location, i.e. by
// aisle and then depth (section 5, Subproblem 2).  The first pick starts the
// walk, each further one is a step, and cost() closes it.
template <int ROUTE>
struct PickWalk {
    // the instance's values, held in vector registers: an instruction takes one
    // scalar register at most, so that copies would be made at each step
    uint32_t magic, d_s, sh, pitch_lo, pitch_hi, half;
    int32_t L, spacing;
    uint32_t ca, a_lo;                // current aisle, first aisle
    // optimal: the five classes at the current aisle, its first and last
    // depth and its largest gap (0: one pick); all three doubled
    OptClasses s;
    uint32_t ylo, yhi, gap;
    // combined: the best walks ending on the front and on the back, the last
    // aisle decided; depths as they are
    int64_t front, back;
    uint32_t done;
    // return / largest gap: previous depth in the aisle (front: 0), largest
    // gap so far in it, and the sum over closed aisles
    int32_t py, g;
    int64_t sum;

    // the depth of a scaled location in aisle a.  Locations take 24 bits, so
    // a * d_s does (d_s itself only takes a 25th in a single aisle, a = 0), but a
    // pitch may not: its index times it is two 24-bit products, each at the
    // full rate (a 32-bit one runs at a quarter of it).
    static constexpr int DOUBLED = ROUTE == WO_ROUTE_OPTIMAL;
    __device__ __forceinline__ uint32_t depth(uint32_t ls, uint32_t a) const
    {
        const uint32_t j = (ls - mul24(a, d_s)) >> sh;
        return mad24(j, pitch_lo, half) + (mul24(j, pitch_hi) << (12 + DOUBLED));
    }

    __device__ __forceinline__ PickWalk(InstConst &inst, int32_t sp, uint32_t m, uint32_t first)
        : magic(m), d_s(inst.d_s), sh(inst.shift + 1), pitch_lo(((uint32_t)inst.pitch & 0xFFFu) << DOUBLED),
          pitch_hi((uint32_t)inst.pitch >> 12), half(((uint32_t)inst.pitch / 2u) << DOUBLED), L(inst.L), spacing(sp)
    {
        asm("" : "+v"(magic), "+v"(d_s), "+v"(sh), "+v"(pitch_lo), "+v"(pitch_hi), "+v"(half), "+v"(L), "+v"(spacing));
        ca = mulhi24(first, magic);
        a_lo = ca;
        const uint32_t y = depth(first, ca);
        if (ROUTE == WO_ROUTE_OPTIMAL) {
            s = opt_start(ca, 2u * (uint32_t)spacing, (uint32_t)L);
            ylo = y;
            yhi = y;
            gap = 0;
        } else if (ROUTE == WO_ROUTE_COMBINED) {
            front = 0;
            back = (int64_t)1 << 60;      // the back is not reachable yet
            done = 0;
            ylo = y;
            yhi = y;
        } else {
            sum = 0;
            g = (int32_t)y;
            py = (int32_t)y;
        }
    }

    // Another pick; one that repeats the last (the same aisle and depth)
    // changes nothing.
    __device__ __forceinline__ void step(uint32_t ls)
    {
        uint32_t a = mulhi24(ls, magic);
        asm("" : "+v"(a));                // 32 bits: no 64-bit compare with ca
        const uint32_t yu = depth(ls, a);
        if (ROUTE == WO_ROUTE_OPTIMAL) {
            // The lanes whose aisle ca is complete.  The mask is made opaque
            // for the selects below, which the compiler would else move into
            // the other side of the branch.
            const uint64_t closes = __builtin_amdgcn_ballot_w64(a != ca);
            uint64_t sel = closes;
            asm("" : "+s"(sel));
            if (lane_in(closes)) {
                const uint32_t w = (uint32_t)spacing, r = a - ca;
                opt_aisle(s, (uint32_t)L, yhi, 2u * (uint32_t)L - ylo, 2u * (uint32_t)L - gap);
                // the spacing may pass 23 bits where the aisles are few
                opt_run(s, r, mul24(r, (w & 0x7FFFFFu) << 1) + (mul24(r, w >> 23) << 24), 2u * w, (uint32_t)L);
            }
            gap = lane_in(sel) ? 0u : max(gap, yu - yhi);
            ylo = lane_in(sel) ? yu : ylo;
            yhi = yu;
            ca = a;
        } else if (ROUTE == WO_ROUTE_COMBINED) {
            // each aisle with picks crossed or entered and left from the
            // cross aisle the picker is on, best choice by one length per
            // cross aisle
            if (a != ca) {
                const int64_t st = (int64_t)spacing * (int64_t)(ca - done);
                const int64_t f2 = min(front + 2ll * yhi, back + L), b2 = min(front + L, back + 2ll * L - 2ll * ylo);
                front = f2 + st;
                back = b2 + st;
                done = ca;
                ca = a;
                ylo = yu;
            }
            yhi = yu;
        } else {
            const int32_t y = (int32_t)yu;
            if (a != ca) {                // close aisle ca
                if (ROUTE == WO_ROUTE_RETURN) {
                    sum += py;
                } else {
                    g = max(g, L - py);
                    if (ca != a_lo) sum += L - g;
                }
                ca = a;
                py = 0;
                g = 0;
            }
            g = max(g, y - py);
            py = y;
        }
    }

    __device__ __forceinline__ int64_t cost()
    {
        if (ROUTE == WO_ROUTE_OPTIMAL) {
            opt_aisle(s, (uint32_t)L, yhi, 2u * (uint32_t)L - ylo, 2u * (uint32_t)L - gap);
            // even ends, one component; and the way along the cross aisles
            return (int64_t)(min(min(s.f, s.b), s.e1) + 2u * (uint32_t)spacing * ca);
        }
        if (ROUTE == WO_ROUTE_COMBINED) {
            // the walk ends on the front (crossing the last aisle from the back)
            const int64_t st = (int64_t)spacing * (int64_t)(ca - done);
            const int64_t f2 = min(front + 2ll * yhi, back + L), b2 = min(front + L, back + 2ll * L - 2ll * ylo);
            return min(f2, b2 + L) + st + (int64_t)spacing * (int64_t)ca;
        }
        const int64_t horiz = 2ll * spacing * ca;    // ca is the farthest aisle now
        if (ROUTE == WO_ROUTE_RETURN) return horiz + 2 * (sum + py);
        if (ca == a_lo) return horiz + 2ll * py;     // one aisle: the return route
        return horiz + 2ll * L + 2 * sum;
    }
};

// Route cost of one tour from its row of np (1 .. pick_slots) picks.  The
// slots past np repeat the first pick, which changes no route and spares
// each step a look at np.  The combined route's steps, the dearest, come in eights
// of which rows of few slots leave out the last: their entries sort to the end
// (3,732 plans of 4,000 orders at capacity 13: 261 to 204 us; at 30 185 both ways).
template <int ROUTE>
static __device__ __forceinline__ int64_t pick_route_cost(const uint32_t *picks, uint32_t np, int32_t spacing,
                                                          InstConst &I, uint32_t magic)
{
    uint32_t v[MAX_PICK_SLOTS];
    v[0] = picks[0];
    if constexpr (ROUTE != WO_ROUTE_COMBINED) {
#pragma unroll
        for (int i = 1; i < MAX_PICK_SLOTS; i++) v[i] = (uint32_t)i < np ? picks[i] : v[0];
        sort32(v);
        PickWalk<ROUTE> w(I, spacing, magic, v[0]);
#pragma unroll
        for (int i = 1; i < MAX_PICK_SLOTS; i++) w.step(v[i]);
        return w.cost();
    }
    const int slots = I.pick_slots;                      // uniform
#pragma unroll
    for (int e = 0; e < MAX_PICK_SLOTS; e += 8) {
        if (e < slots) {
#pragma unroll
            for (int i = e ? e : 1; i < e + 8; i++) v[i] = (uint32_t)i < np ? picks[i] : v[0];
        } else {
#pragma unroll
            for (int i = e; i < e + 8; i++) v[i] = 0xFFFFFFFFu;
        }
    }
    sort32(v);
    PickWalk<ROUTE> w(I, spacing, magic, v[0]);
#pragma unroll
    for (int e = 0; e < MAX_PICK_SLOTS; e += 8)
        if (e < slots)
#pragma unroll
            for (int i = e ? e : 1; i < e + 8; i++) w.step(v[i]);
    return w.cost();
}

// Route costs of the instance's orders with more lines than a pick row keeps
// (each a tour of its own, since the capacity is at most MAX_PICK_SLOTS), for
// one plan: the workgroup's NT threads stage an order's scaled locations in
// LDS (`scr`, at least 4 * I.big_np2 bytes, free for the call; zs the zone
// starts), sort them (bitonic, padded with all ones), and thread 0 walks
// them.  Returns the sum on thread 0 and 0 elsewhere; every thread must call.
template <int ROUTE, int NT>
static __device__ int64_t big_orders_cost(const EvalArgs &A, InstConst &I, const uint32_t *zs, uint32_t *scr,
                                          int32_t spacing)
{
    const int tid = threadIdx.x;
    const uint32_t *big = A.big + I.big_off;
    const uint32_t *ordoff = A.ordoff + I.ordoff_off;
    const uint32_t *ordrec = A.ordrec + I.ordrec_off;
    int64_t acc = 0;
    for (int b = 0; b < I.n_big; b++) {
        const uint32_t o = big[b];
        const uint32_t r0 = ordoff[o];
        const uint32_t m2 = min(1u << (32 - __builtin_clz(max(ordoff[o + 1] - r0, 2u) - 1u)), (uint32_t)I.big_np2);
        const uint32_t m = min(ordoff[o + 1] - r0, m2);
        __syncthreads();                 // scr is free (earlier use, previous order)
        for (uint32_t i = tid; i < m2; i += NT) {
            const uint32_t r = i < m ? ordrec[r0 + i] : 0u;
            scr[i] = i < m ? r + zs[r >> 26] : 0xFFFFFFFFu;
        }
        for (uint32_t k = 2; k <= m2; k <<= 1)
            for (uint32_t j = k >> 1; j > 0; j >>= 1) {
                __syncthreads();
                for (uint32_t i = tid; i < m2; i += NT) {
                    const uint32_t l = i ^ j;
                    if (l > i) {
                        const uint32_t x = scr[i], y = scr[l];
                        const bool up = (i & k) == 0;
                        if ((x > y) == up) {
                            scr[i] = y;
                            scr[l] = x;
                        }
                    }
                }
            }
        __syncthreads();
        if (tid == 0) {
            PickWalk<ROUTE> w(I, spacing, I.magic, scr[0]);
            // the next location in flight during a step (largest gap, orders of 500 and
            // 900 lines: 282 to 262 us)
            uint32_t next = scr[1];      // such an order has more than MAX_PICK_SLOTS
            for (uint32_t i = 1; i < m; i++) {
                const uint32_t now = next;
                next = scr[min(i + 1u, m - 1u)];
                w.step(now);
            }
            acc += w.cost();
        }
    }
    __syncthreads();                     // scr is free again
    return acc;
}

}  // namespace wo
