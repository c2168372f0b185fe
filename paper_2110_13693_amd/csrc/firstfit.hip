// First-fit order batching (see eval_ff_kernel below), for every route.
#include "eval_device.h"

namespace wo {

// value of a 64-bit lane register pair in lane l (uniform)
static __device__ __forceinline__ uint64_t lane64(uint32_t lo, uint32_t hi, int l)
{
    return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)lo, l) |
           ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)hi, l) << 32);
}

// Tours under seed batching, packed form (SEED_PACKED_ORDERS and
// SEED_PACKED_LINES above): the same rule as the general form below, with the
// search for the next order turned from a scan over every position into
// operations on bit masks.  Lane b holds a 64-bit word of positions 64 b ..
// 64 b + 63 of every mask: the positions in no tour, the bit planes of the
// orders' sizes, and the bit planes of their counts of aisles new to the tour.
// The order that joins next is found from the highest plane of the counts
// down: the fitting positions whose bit is clear, where there are any, else
// those whose bit is set; the first position left is the one.  An order that
// joins with no new aisle changes only the room.  Otherwise every order that
// visits an aisle it adds loses one new aisle: the aisle's mask of positions is
// subtracted from the planes of all positions at once.  The aisles of more
// than SEED_COLD orders (a few dozen, which most of the added aisles are: 290
// orders on average at the paper scale) keep their mask in memory, 512 bytes;
// the others keep a list, which becomes a mask in LDS.
//
// A chain of about n dependent steps per plan, bound by their latency and
// issue: the plans in flight set the rate, so LDS holds little (2.4 KB for
// 400 aisles; the registers allow 16 plans per CU) and the lists, read once per added aisle, come
// from L2, the last-level cache and memory (some 70 KB of a plan's 131 KB slice are in
// use: 4,096 plans pass 256 MB).  4,096 plans of 4,000 orders: 4.66 ms,
// against 70.6 ms for the general form, which reads every position per step
// and fits four plans per CU.  With the counts as bytes in LDS, decremented by
// atomics over the lists: 8.5 ms; with every list kept as a list: 6.6 ms; with
// a store to memory per join: 5.1 ms.
static __device__ int seed_tours_packed(const EvalArgs &A, InstConst &I, const uint16_t *seq, const uint8_t *cnt,
                                        const uint32_t *zs, uint16_t *tour_of, unsigned char *smem)
{
    const int lane = threadIdx.x;
    const int n = I.n_orders, NA = I.n_aisles;
    const uint32_t Q = (uint32_t)I.capacity;
    const SeedPackedLayout L = seed_packed_layout(NA);
    uint32_t *mask = (uint32_t *)(smem + L.mask);      // a mask of positions, zero between uses
    uint32_t *aend = (uint32_t *)(smem + L.aend);      // end of each aisle's list of positions; bits 16 and up: 1 + its mask
    uint32_t *tbits = (uint32_t *)(smem + L.tbits);    // the tour's aisle set
    unsigned char *scr = A.seed_scr + (int64_t)blockIdx.x * A.seed_stride;
    uint16_t *fwd = (uint16_t *)scr;                   // a position's first SEED_FWD aisles
    uint16_t *apos = (uint16_t *)(scr + A.seed_apos);  // positions by aisle
    uint2 *hot = (uint2 *)(scr + A.seed_hot);          // masks of the longest lists
    uint32_t *joins = A.ff_queue + (int64_t)blockIdx.x * A.ff_stride;   // every join: position | tour << 16
    const uint32_t *oo = A.ordoff + I.ordoff_off;
    const uint32_t *orr = A.ordrec + I.ordrec_off;
    const uint32_t magic = I.magic;
    const int n_blk = (n + 63) / 64;
    const uint32_t n_lines = (uint32_t)I.n_lines;

    auto aisle_of = [&](uint32_t rec) { return mulhi24(rec + zs[rec >> 26], magic); };
    // the distinct aisles of the order at position q: the first 8 lines in
    // registers, the rest (rare) one at a time
    auto for_aisles = [&](int q, auto f) {
        const uint32_t o = min((uint32_t)seq[q], (uint32_t)(n - 1));
        const uint32_t l0 = oo[o], len = oo[o + 1] - l0;
        uint32_t a[8];
#pragma unroll
        for (int i = 0; i < 8; i++) a[i] = orr[min(l0 + (uint32_t)i, n_lines - 1u)];
#pragma unroll
        for (int i = 0; i < 8; i++) a[i] = (uint32_t)i < len ? aisle_of(a[i]) : 0xFFFFFFFFu;
#pragma unroll
        for (int i = 0; i < 8; i++) {
            bool dup = (uint32_t)i >= len;
#pragma unroll
            for (int j = 0; j < i; j++) dup = dup || a[j] == a[i];
            if (!dup) f(a[i]);
        }
        for (uint32_t i = 8; i < len; i++) {
            const uint32_t x = aisle_of(orr[l0 + i]);
            bool dup = false;
            for (uint32_t j = 0; j < i; j++) dup = dup || aisle_of(orr[l0 + j]) == x;
            if (!dup) f(x);
        }
    };

    // ---- the tables -----------------------------------------------------
    for (int a = lane; a < NA; a += 64) aend[a] = 0u;
    for (int i = lane; i < 128; i += 64) mask[i] = 0u;
    __syncthreads();
    uint32_t free_lo = 0, free_hi = 0;                         // positions in no tour
    uint32_t k_lo[4] = {0, 0, 0, 0}, k_hi[4] = {0, 0, 0, 0};   // bit planes of the orders' aisle counts
    uint32_t s_lo[4] = {0, 0, 0, 0}, s_hi[4] = {0, 0, 0, 0};   // bit planes of the sizes
    uint32_t smax = 1;
    for (int b = 0; b < n_blk; b++) {
        const int q = 64 * b + lane;
        uint32_t k = 0, sz = 0;
        uint32_t fa[SEED_FWD] = {0xFFFFu, 0xFFFFu, 0xFFFFu, 0xFFFFu};
        if (q < n) {
            for_aisles(q, [&](uint32_t a) {
#pragma unroll
                for (int i = 0; i < SEED_FWD; i++)
                    if (k == (uint32_t)i) fa[i] = a;
                k++;
                atomicAdd(&aend[a], 1u);
            });
            if (k > (uint32_t)SEED_FWD) fa[SEED_FWD - 1] = 0xFFFEu;   // more aisles than the record holds
            sz = cnt[min((uint32_t)seq[q], (uint32_t)(n - 1))];
            *(uint2 *)(fwd + SEED_FWD * q) = make_uint2(fa[0] | (fa[1] << 16), fa[2] | (fa[3] << 16));
        }
        smax = max(smax, sz);
        auto put = [&](uint64_t m, uint32_t &lo, uint32_t &hi) {
            lo = set_lane(lo, (uint32_t)m, b);
            hi = set_lane(hi, (uint32_t)(m >> 32), b);
        };
        put(__ballot(q < n), free_lo, free_hi);
#pragma unroll
        for (int i = 0; i < 4; i++) {
            put(__ballot((k >> i) & 1u), k_lo[i], k_hi[i]);
            put(__ballot((sz >> i) & 1u), s_lo[i], s_hi[i]);
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) smax = max(smax, (uint32_t)__shfl_xor((int)smax, d, 64));
    smax = (uint32_t)__builtin_amdgcn_readfirstlane((int)smax);
    __syncthreads();
    {
        uint32_t carry = 0;                              // starts of the lists (exclusive scan)
        for (int a0 = 0; a0 < NA; a0 += 64) {
            const int a = a0 + lane;
            const uint32_t c = a < NA ? aend[a] : 0u;
            const uint32_t inc = wave_incl_scan(c) + carry;
            if (a < NA) aend[a] = inc - c;
            carry = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        }
    }
    __syncthreads();
    for (int q = lane; q < n; q += 64)                   // each start advances to its list's end
        for_aisles(q, [&](uint32_t a) {
            const uint32_t e = atomicAdd(&aend[a], 1u);
            if (e < n_lines) apos[e] = (uint16_t)q;      // (a malformed sequence could hold more)
        });
    __syncthreads();                                     // the lists are in memory
    // the long lists as masks of positions: the aisle's end then names its mask
    {
        uint32_t n_hot = 0;
        for (int a0 = 0; a0 < NA; a0 += 64) {
            const int a = a0 + lane;
            const uint32_t e1 = a < NA ? min(aend[a], n_lines) : 0u;
            const uint32_t e0 = a < NA && a > 0 ? min(aend[a - 1] & 0xFFFFu, n_lines) : 0u;
            const uint64_t want = __ballot(a < NA && e1 > e0 + SEED_COLD);
            const uint32_t idx = n_hot + __builtin_amdgcn_mbcnt_hi((uint32_t)(want >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)want, 0u));
            lds_order();
            if (a < NA) aend[a] = e1 | (lane_in(want) ? (idx + 1u) << 16 : 0u);
            lds_order();
            for (uint64_t m = want; m; m &= m - 1ull) {
                const int j = (int)__builtin_ctzll(m);
                const uint32_t s0 = (uint32_t)__builtin_amdgcn_readlane((int)e0, j);
                const uint32_t s1 = (uint32_t)__builtin_amdgcn_readlane((int)e1, j);
                for (uint32_t e = s0 + (uint32_t)lane; e < s1; e += 64) {
                    const uint32_t r = min((uint32_t)apos[e], (uint32_t)(n - 1));
                    atomicOr(&mask[r >> 5], 1u << (r & 31u));
                }
                lds_order();
                hot[64u * n_hot + (uint32_t)lane] = ((const uint2 *)mask)[lane];
                ((uint2 *)mask)[lane] = make_uint2(0u, 0u);
                lds_order();
                n_hot++;
            }
        }
    }
    __syncthreads();

    // ---- tour by tour ------------------------------------------------------
    // the joins, (position, tour) each, collect in a register and go to
    // memory 64 at a time: a store per join would have every step wait for it
    int T = 0, n_join = 0;                               // uniform
    uint32_t joined = 0;
    for (;;) {
        const uint64_t any = __ballot((free_lo | free_hi) != 0u);
        if (!any) break;
        // a new tour: every aisle of every order is new to it
        uint32_t c_lo[4], c_hi[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            c_lo[i] = k_lo[i];
            c_hi[i] = k_hi[i];
        }
        // positions with no new aisle
        uint32_t z_lo = ~(c_lo[0] | c_lo[1] | c_lo[2] | c_lo[3]), z_hi = ~(c_hi[0] | c_hi[1] | c_hi[2] | c_hi[3]);
        lds_order();
        for (int w = lane; w < (NA + 31) / 32; w += 64) tbits[w] = 0u;
        lds_order();
        // the seed: the earliest position in no tour
        int b = (int)__builtin_ctzll(any);
        int q = 64 * b + (int)__builtin_ctzll(lane64(free_lo, free_hi, b));
        bool adds = true;                                // the order at q adds an aisle (uniform)
        uint32_t room = Q;
        for (;;) {
            // the order at q joins
            const uint32_t av = adds ? (uint32_t)fwd[SEED_FWD * q + (lane & (SEED_FWD - 1))] : 0u;
            joined = set_lane(joined, (uint32_t)q | ((uint32_t)T << 16), n_join & 63);
            if ((++n_join & 63) == 0) joins[n_join - 64 + lane] = joined;
            const uint32_t bit = 1u << (q & 31);
            uint32_t sz = 0;
            if (q & 32) {
                free_hi &= lane == b ? ~bit : ~0u;
#pragma unroll
                for (int i = 0; i < 4; i++)
                    sz |= (((uint32_t)__builtin_amdgcn_readlane((int)s_hi[i], b) >> (q & 31)) & 1u) << i;
            } else {
                free_lo &= lane == b ? ~bit : ~0u;
#pragma unroll
                for (int i = 0; i < 4; i++)
                    sz |= (((uint32_t)__builtin_amdgcn_readlane((int)s_lo[i], b) >> (q & 31)) & 1u) << i;
            }
            room = sz < room ? room - sz : 0u;           // a larger order rides alone
            if (room == 0u) break;
            uint32_t m_lo = free_lo, m_hi = free_hi;     // in no tour and fitting
            if (room < smax) {
                uint32_t g_lo = 0, g_hi = 0;             // size > room, bit by bit from the lowest
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    if ((room >> i) & 1u) {
                        g_lo &= s_lo[i];
                        g_hi &= s_hi[i];
                    } else {
                        g_lo |= s_lo[i];
                        g_hi |= s_hi[i];
                    }
                }
                m_lo &= ~g_lo;
                m_hi &= ~g_hi;
            }
            if (adds) {
                if (!__ballot((m_lo | m_hi) != 0u)) break;
                // its aisles new to the tour, in lanes of nm
                uint32_t a;
                uint64_t nm;
                if ((uint32_t)__builtin_amdgcn_readlane((int)av, SEED_FWD - 1) != 0xFFFEu) {
                    a = av;
                    const uint32_t ac = min(a, (uint32_t)NA - 1u);
                    nm = __ballot(a != 0xFFFFu && !((tbits[ac >> 5] >> (ac & 31u)) & 1u)) & ((1ull << SEED_FWD) - 1ull);
                } else {
                    // more aisles than the record: from the order's lines,
                    // one per lane (an aisle counts at its first line)
                    const uint32_t o = min((uint32_t)seq[q], (uint32_t)(n - 1));
                    const uint32_t l0 = oo[o], len = min(oo[o + 1] - l0, (uint32_t)SEED_PACKED_LINES);
                    a = (uint32_t)lane < len ? aisle_of(orr[l0 + (uint32_t)lane]) : 0xFFFFFFFFu;
                    const uint32_t ac = min(a, (uint32_t)NA - 1u);
                    bool fresh = (uint32_t)lane < len && !((tbits[ac >> 5] >> (ac & 31u)) & 1u);
                    for (uint32_t i = 0; i + 1 < len; i++)
                        fresh = fresh && !(i < (uint32_t)lane && (uint32_t)__builtin_amdgcn_readlane((int)a, (int)i) == a);
                    nm = __ballot(fresh);
                }
                const uint32_t ac = min(a, (uint32_t)NA - 1u);
                const uint32_t e1 = aend[ac], e0 = ac ? aend[ac - 1u] & 0xFFFFu : 0u;
                lds_order();
                if (lane_in(nm)) atomicOr(&tbits[ac >> 5], 1u << (ac & 31u));
                // two aisles at a time: the mask of each is read, or its
                // (short) position list; the loads carry no condition, so
                // that both are in flight together
                while (nm) {
                    const int j0 = (int)__builtin_ctzll(nm);
                    nm &= nm - 1ull;
                    const bool two = nm != 0ull;
                    const int j1 = two ? (int)__builtin_ctzll(nm) : j0;
                    nm &= two ? nm - 1ull : 0ull;
                    const uint32_t v0 = (uint32_t)__builtin_amdgcn_readlane((int)e1, j0);
                    const uint32_t v1 = (uint32_t)__builtin_amdgcn_readlane((int)e1, j1);
                    const uint32_t s0 = (uint32_t)__builtin_amdgcn_readlane((int)e0, j0);
                    const uint32_t s1 = (uint32_t)__builtin_amdgcn_readlane((int)e0, j1);
                    uint2 w0 = make_uint2(0u, 0u), w1 = make_uint2(0u, 0u);
                    if (v0 >> 16) w0 = hot[64u * ((v0 >> 16) - 1u) + (uint32_t)lane];
                    else w0.x = apos[min(s0 + (uint32_t)lane, n_lines - 1u)];
                    if (two) {
                        if (v1 >> 16) w1 = hot[64u * ((v1 >> 16) - 1u) + (uint32_t)lane];
                        else w1.x = apos[min(s1 + (uint32_t)lane, n_lines - 1u)];
                    }
                    auto to_mask = [&](uint2 &w, uint32_t len) {
                        lds_order();
                        if ((uint32_t)lane < len && w.x < (uint32_t)n) atomicOr(&mask[w.x >> 5], 1u << (w.x & 31u));
                        lds_order();
                        w = ((const uint2 *)mask)[lane];
                        ((uint2 *)mask)[lane] = make_uint2(0u, 0u);
                        lds_order();
                    };
                    // one new aisle fewer at the mask's positions
                    auto subtract = [&](uint2 w) {
#pragma unroll
                        for (int k = 0; k < 4; k++) {
                            const uint32_t x = c_lo[k], y = c_hi[k];
                            c_lo[k] = x ^ w.x;
                            c_hi[k] = y ^ w.y;
                            w.x &= ~x;
                            w.y &= ~y;
                        }
                    };
                    if (!(v0 >> 16)) to_mask(w0, v0 - s0);
                    subtract(w0);
                    if (two) {
                        if (!(v1 >> 16)) to_mask(w1, v1 - s1);
                        subtract(w1);
                    }
                }
                z_lo = ~(c_lo[0] | c_lo[1] | c_lo[2] | c_lo[3]);
                z_hi = ~(c_hi[0] | c_hi[1] | c_hi[2] | c_hi[3]);
            }
            // the next order: the fewest new aisles, then the earliest
            const uint32_t x0 = m_lo & z_lo, y0 = m_hi & z_hi;
            adds = __ballot((x0 | y0) != 0u) == 0ull;
            if (!adds) {
                m_lo = x0;
                m_hi = y0;
            } else {
                if (!__ballot((m_lo | m_hi) != 0u)) break;
#pragma unroll
                for (int k = 3; k >= 0; k--) {
                    const uint32_t x = m_lo & ~c_lo[k], y = m_hi & ~c_hi[k];
                    if (__ballot((x | y) != 0u)) {
                        m_lo = x;
                        m_hi = y;
                    }
                }
            }
            b = (int)__builtin_ctzll(__ballot((m_lo | m_hi) != 0u));
            q = 64 * b + (int)__builtin_ctzll(lane64(m_lo, m_hi, b));
        }
        T++;
    }
    if (lane < (n_join & 63)) joins[(n_join & ~63) + lane] = joined;
    __syncthreads();                                     // the joins are in memory
    for (int i = lane; i < n_join; i += 64) {
        const uint32_t x = joins[i];
        tour_of[min((uint32_t)seq[x & 0xFFFFu], (uint32_t)(n - 1))] = (uint16_t)(x >> 16);
    }
    return T;
}

// Plans under first-fit or seed order batching (the other greedy batching
// rules of the order-picking literature beside next fit; section 5,
// Subproblem 2 leaves the batching of orders into tours open), for each
// route.  One wavefront evaluates one plan (two under first fit by the S-shape route):
//   1. zone starts: each category's start is the total size of the
//      categories in lower zones (one pass over the categories per lane);
//   2. first fit, 64 orders of the sequence at a time, one per lane, tour by
//      tour: an order joins the earliest tour with room, so the first tour
//      takes, in sequence, every order that fits what it has left, the next
//      tour the same of those the first left, and so on.  The open tours come
//      first, in opening order (a tour whose room falls below the instance's
//      smallest order can never take another one), then new tours for the
//      orders left.  A new tour takes all orders up to the first that does not
//      fit by one running sum over the lanes; after that, as for an open tour,
//      one ballot finds the next order that fits.  At the paper scale that is
//      about 20 steps per 64 orders, and 4,096 plans take 0.253 ms, against
//      0.546 when each order looked for its tour in turn; over half of it is
//      this chain of steps, 16 plans per CU in turn.  Lane j also keeps the j-th open tour in
//      opening order and its room; full tours leave the lanes only when the
//      lanes run out.  The open tours stay few (first fit keeps filling the
//      earliest ones), but any beyond 64 wait, in order, in a queue in global
//      memory, which refills the lanes;
//   2'. or seed batching: per position the order's size, aisle count and
//      "new aisles" (for the tour being built) in one word, and per aisle the positions
//      of the orders visiting it, all in LDS.  A tour starts from the
//      earliest position in no tour; each order that joins it marks its
//      aisles in the tour's set, and every order visiting an aisle new to
//      the tour loses one new aisle (an atomic decrement per order and
//      aisle); then one wave-wide minimum over (new aisles, position) of the
//      orders that fit picks the next one;
//   3. tiles of tours: for the S-shape route, every line of an order in the
//      tile sets its aisle bit in the tour's LDS row and the order raises the
//      tour's farthest location, then one lane per tour takes the closed
//      form; for the other routes every line record appends its location to
//      its tour's pick row, then one lane per tour sorts the picks and walks
//      them as the next-fit kernel does;
//   4. the wave's sum, saturated to int32, and the rate over the window.
// Packed seed batching is a chain per plan on 16 plans per CU, which takes four
// waves per SIMD (the optimal route 7.3 ms at three, 4.7 at four); the routes
// with pick rows keep to the same.
// First fit by the S-shape route has a second wave, which waits while the first
// cuts the tours and then takes half of the tile passes: the chain leaves the
// registers of eight waves per SIMD, and 16 plans per CU run as before.  4,096
// paper-scale plans 275 to 253 us.  The other kernels have no registers for it.
static __host__ __device__ constexpr int ff_threads(int route, int batch)
{
    return route == WO_ROUTE_SSHAPE && batch == FF_FIRST_FIT ? 128 : 64;
}

template <int ROUTE, int BATCH>
__global__ __launch_bounds__(ff_threads(ROUTE, BATCH), ff_threads(ROUTE, BATCH) == 128 ? 8
                             : ROUTE != WO_ROUTE_SSHAPE || BATCH == FF_SEED_PACKED ? 4 : 1) void eval_ff_kernel(EvalArgs A)
{
    constexpr int TILE = ff_tile(ROUTE);
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int NT = ff_threads(ROUTE, BATCH), NW = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = NW > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
    for (int64_t p = blockIdx.x; p < A.n_plans; p += gridDim.x) {
        const int ii = instance_of(A, p);
        InstConst &I = as_const(A.inst)[ii];
        const int n = I.n_orders;
        const int C = I.n_cat;
        const int32_t Q = I.capacity;
        const int32_t wsp = A.plan_spacing ? as_const(A.plan_spacing)[p] : I.spacing;   // aisle spacing of this plan
        const int64_t row = p - (A.n_inst > 1 ? as_const(A.plan_begin)[ii] : 0);
        const uint16_t *seq = A.seq + as_const(A.seq_base)[ii] + row * (int64_t)n;
        const uint8_t *cnt = A.cnt + I.cnt_off;
        uint32_t *zs = (uint32_t *)smem;
        uint16_t *tour_of = A.ff_tour + (int64_t)blockIdx.x * A.ff_stride;   // this workgroup's slice
        uint32_t *rows = (uint32_t *)(smem + ff_rows_off());
        const uint32_t RW = (uint32_t)I.row_b / 4u;
        int bad = 0;

        // ---- 1. zone starts ---------------------------------------------
        {
            const uint32_t zc = lane < C ? (uint32_t)A.zone_of[p * 64 + lane] : 0xFFu;
            const uint32_t sz = lane < C ? (uint32_t)I.cat_size[lane] : 0u;
            uint32_t start = 0;
            for (int c = 0; c < C; c++) {
                const uint32_t zo = (uint32_t)__shfl((int)zc, c, 64);
                start += zo < zc ? (uint32_t)I.cat_size[c] : 0u;
            }
            // a malformed row cannot move a category off the warehouse
            start = min(start, (uint32_t)I.n_skus - sz);
            zs[lane] = (start << I.shift) - ((uint32_t)(4 * lane) << 24);
            if (A.validate) {
                uint64_t m = (lane < C && zc < 64u) ? (1ull << zc) : 0ull;
#pragma unroll
                for (int d = 32; d >= 1; d >>= 1) m |= __shfl_xor(m, d, 64);
                const uint64_t want = (C == 64) ? ~0ull : ((1ull << C) - 1ull);
                if (m != want) bad = 1;
            }
        }
        for (int o = tid; o <= n; o += NT) tour_of[o] = 0xFFFFu;   // no tour yet; entry n: padding
        if (A.validate) {
            // every order exactly once: mark them in the tour table, which
            // is then reset
            __syncthreads();
            for (int i = tid; i < n; i += NT) {
                const uint32_t o = seq[i];
                if (o < (uint32_t)n) tour_of[o] = 0; else bad = 1;
            }
            __syncthreads();
            for (int o = tid; o < n; o += NT) {
                bad |= tour_of[o] != 0;
                tour_of[o] = 0xFFFFu;
            }
        }
        __syncthreads();

        // ---- 2. tours ------------------------------------------------------
        // a chain of dependent steps: it issues ahead of other plans' tiles
        __builtin_amdgcn_s_setprio(2);
        int T = 0;                                      // tours opened (uniform)
        if constexpr (BATCH == FF_SEED_PACKED) {
            T = seed_tours_packed(A, I, seq, cnt, zs, tour_of, smem);
        } else if constexpr (BATCH == FF_SEED) {
            // seed batching
            const int NA = I.n_aisles;
            const SeedLayout L = seed_layout(n, NA, I.n_lines);
            // per position: new aisles (bits 0-9), the order's aisles (10-19),
            // its size (20-27), in a tour (bit 31)
            uint32_t *st = (uint32_t *)(smem + L.st);
            uint32_t *aend = (uint32_t *)(smem + L.aend);  // end of each aisle's list of positions
            uint32_t *tbits = (uint32_t *)(smem + L.tbits);
            uint16_t *apos = (uint16_t *)(smem + L.apos);
            const uint32_t *oo = A.ordoff + I.ordoff_off;
            const uint32_t *orr = A.ordrec + I.ordrec_off;
            const uint32_t magic = I.magic;
            auto aisle_of = [&](uint32_t rec) { return mulhi24(rec + zs[rec >> 26], magic); };
            // each distinct aisle of order o's lines, once
            auto for_aisles = [&](uint32_t o, auto f) {
                const uint32_t l0 = oo[o], l1 = oo[o + 1];
                for (uint32_t l = l0; l < l1; l++) {
                    const uint32_t a = aisle_of(orr[l]);
                    bool dup = false;
                    for (uint32_t m = l0; m < l && !dup; m++) dup = aisle_of(orr[m]) == a;
                    if (!dup) f(a);
                }
            };
            for (int a = lane; a < NA; a += 64) aend[a] = 0u;
            __syncthreads();
            // per position: the order's size and aisle count; per aisle: its orders
            for (int q = lane; q < n; q += 64) {
                const uint32_t o = min((uint32_t)seq[q], (uint32_t)(n - 1));
                uint32_t k = 0;
                for_aisles(o, [&](uint32_t a) {
                    k++;
                    atomicAdd(&aend[a], 1u);
                });
                st[q] = k | (k << 10) | ((uint32_t)cnt[o] << 20);
            }
            __syncthreads();
            {
                uint32_t carry = 0;                          // starts of the lists (exclusive scan)
                for (int a0 = 0; a0 < NA; a0 += 64) {
                    const int a = a0 + lane;
                    const uint32_t c = a < NA ? aend[a] : 0u;
                    const uint32_t inc = wave_incl_scan(c) + carry;
                    if (a < NA) aend[a] = inc - c;
                    carry = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
                }
            }
            __syncthreads();
            for (int q = lane; q < n; q += 64) {               // each start advances to its list's end
                const uint32_t o = min((uint32_t)seq[q], (uint32_t)(n - 1));
                // (a malformed sequence, with an order twice, could hold more
                // entries than the table: they are dropped)
                for_aisles(o, [&](uint32_t a) {
                    const uint32_t e = atomicAdd(&aend[a], 1u);
                    if (e < (uint32_t)I.n_lines) apos[e] = (uint16_t)q;
                });
            }
            __syncthreads();
            int next = 0;                                    // positions before it are all in tours (uniform)
            for (;;) {
                // the seed: the earliest position in no tour
                int s = -1;
                for (int b = next; b < n; b += 64) {
                    const uint64_t m = __ballot(b + lane < n && !(st[min(b + lane, n - 1)] >> 31));
                    if (m) {
                        s = b + (int)__builtin_ctzll(m);
                        break;
                    }
                }
                if (s < 0) break;
                next = s;
                // a new tour: every aisle of every later order is new to it
                // (four consecutive positions per lane and access)
                for (int r0 = next & ~3; r0 < n; r0 += 256) {
                    const int i0 = r0 + 4 * lane;
                    if (i0 + 4 <= n) {
                        uint4 w = *(const uint4 *)(st + i0);
                        w.x = (w.x & ~0x3FFu) | ((w.x >> 10) & 0x3FFu);
                        w.y = (w.y & ~0x3FFu) | ((w.y >> 10) & 0x3FFu);
                        w.z = (w.z & ~0x3FFu) | ((w.z >> 10) & 0x3FFu);
                        w.w = (w.w & ~0x3FFu) | ((w.w >> 10) & 0x3FFu);
                        *(uint4 *)(st + i0) = w;
                    } else {
                        for (int q = i0; q < n; q++) st[q] = (st[q] & ~0x3FFu) | ((st[q] >> 10) & 0x3FFu);
                    }
                }
                for (int w = lane; w < (NA + 31) / 32; w += 64) tbits[w] = 0u;
                __syncthreads();
                uint32_t load = 0;
                int q = s;                                   // the order joining the tour (uniform)
                for (;;) {
                    const uint32_t o = min((uint32_t)seq[q], (uint32_t)(n - 1));
                    if (lane == 0) {
                        st[q] |= 1u << 31;
                        tour_of[o] = (uint16_t)T;
                    }
                    load += (st[q] >> 20) & 0xFFu;
                    // each aisle it adds: every order visiting that aisle has
                    // one new aisle fewer.  The order's lines, 64 at a time,
                    // one per lane; a line counts if no earlier line of the
                    // order has its aisle and the tour does not visit it yet.
                    const uint32_t l0 = oo[o], l1 = oo[o + 1];
                    for (uint32_t c0 = l0; c0 < l1; c0 += 64) {
                        const uint32_t l = c0 + lane;
                        const uint32_t a = l < l1 ? aisle_of(orr[l]) : 0xFFFFFFFFu;
                        bool fresh = l < l1 && !((tbits[min(a, (uint32_t)NA - 1u) >> 5] >> (a & 31u)) & 1u);
                        const uint32_t m_c = min(64u, l1 - c0);
                        for (uint32_t i = 0; i < m_c; i++)           // earlier lines of this chunk
                            fresh = fresh && !(i < (uint32_t)lane && (uint32_t)__builtin_amdgcn_readlane((int)a, (int)i) == a);
                        for (uint32_t m = l0; m < c0 && fresh; m++)  // earlier chunks (orders of more than 64 lines)
                            fresh = aisle_of(orr[m]) != a;
                        uint64_t nm = __ballot(fresh);
                        while (nm) {
                            const int j = (int)__builtin_ctzll(nm);
                            nm &= nm - 1ull;
                            const uint32_t aj = (uint32_t)__builtin_amdgcn_readlane((int)a, j);
                            if (lane == 0) tbits[aj >> 5] |= 1u << (aj & 31u);
                            const uint32_t e1 = min(aend[aj], (uint32_t)I.n_lines);
                            for (uint32_t e = (aj ? aend[aj - 1] : 0u) + lane; e < e1; e += 64) {
                                const uint32_t r = apos[e];
                                if ((int)r >= next && (int)r < n) atomicSub(&st[r], 1u);
                            }
                        }
                    }
                    __syncthreads();
                    // the order that fits with the fewest new aisles, the earliest of them
                    // (four consecutive positions per lane and read, branch-free;
                    // positions before `next` are all in tours)
                    uint32_t best = 0xFFFFFFFFu;
                    for (int r0 = next & ~3; r0 < n; r0 += 256) {
                        const int i0 = r0 + 4 * lane;
                        const uint4 w4 = i0 < n ? *(const uint4 *)(st + i0) : make_uint4(~0u, ~0u, ~0u, ~0u);
                        const uint32_t w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                        for (int u = 0; u < 4; u++) {
                            const uint32_t i = (uint32_t)(i0 + u);
                            const bool ok = i < (uint32_t)n && (int32_t)w[u] >= 0 &&
                                            load + ((w[u] >> 20) & 0xFFu) <= (uint32_t)Q;
                            best = min(best, ok ? (((w[u] & 0x3FFu) << 16) | i) : 0xFFFFFFFFu);
                        }
                    }
                    best = wave_min_u32(best);
                    if (best == 0xFFFFFFFFu) break;
                    q = (int)(best & 0xFFFFu);
                }
                T++;
            }
        } else if (wv == 0) {
            // ---- 2. first fit -------------------------------------------------
            const uint32_t mins = (uint32_t)__builtin_amdgcn_readfirstlane(I.min_size);   // a room below it never takes an order
            // Lanes [0, k) hold tours in opening order with their rooms, lanes
            // past k room 0.  A tour whose room falls below mins stays in its
            // lane until the lanes run out (no order fits it, so a ballot never
            // picks it); open tours opened after the lanes' wait in the queue
            // [qh, qt), in order, whenever it is not empty.
            int k = 0;                                      // uniform
            uint32_t room = 0, tour = 0;
            uint32_t *queue = A.ff_queue + (int64_t)blockIdx.x * A.ff_stride;
            int qh = 0, qt = 0;                             // uniform
            // the full tours leave the lanes (the others move down, in order),
            // then the freed lanes take the queue's open tours, in order
            auto compact = [&]() {
                const uint64_t live = __ballot(room >= mins);
                const uint32_t nlive = (uint32_t)__builtin_popcountll(live);
                const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(live >> 32),
                                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)live, 0u));
                // a permutation: open tours to lanes [0, nlive), the rest after them
                const uint32_t dst = lane_in(live) ? below : nlive + (uint32_t)lane - below;
                const uint32_t rr = (uint32_t)__builtin_amdgcn_ds_permute((int)(dst << 2), (int)room);
                const uint32_t tt = (uint32_t)__builtin_amdgcn_ds_permute((int)(dst << 2), (int)tour);
                room = (uint32_t)lane < nlive ? rr : 0u;
                tour = tt;
                k = (int)nlive;
                while (k < 64 && qh < qt) {
                    const uint32_t e = qh + lane < qt ? queue[qh + lane] : 0u;
                    uint64_t lv = __ballot((e >> 16) >= mins);
                    int taken = 0;
                    while (lv && k < 64) {
                        const int f = __builtin_ctzll(lv);
                        const uint32_t ef = (uint32_t)__builtin_amdgcn_readlane((int)e, f);
                        room = set_lane(room, ef >> 16, k);
                        tour = set_lane(tour, ef & 0xFFFFu, k);
                        k++;
                        taken = f + 1;
                        lv &= lv - 1ull;
                    }
                    qh = k < 64 ? min(qh + 64, qt) : qh + taken;
                }
            };
            // orders and sizes of the next windows load ahead: the sequence two
            // windows, the sizes (a gather by order) one
            auto order_at = [&](int i) { return (uint32_t)seq[min(i, n - 1)]; };
            uint32_t o_n = min(order_at(lane), (uint32_t)n), o_n2 = order_at(64 + lane);
            uint32_t s_n = cnt[o_n];
            for (int i0 = 0; i0 < n; i0 += 64) {
                const int i = i0 + lane;
                const uint32_t o_l = i < n ? o_n : (uint32_t)n;
                // min(size, Q + 1); an id out of range (a malformed row, whose
                // result is unspecified) counts as one item and is left out below
                const uint32_t s_l = i < n ? max(s_n, 1u) : 1u;
                o_n = min(o_n2, (uint32_t)n);
                s_n = cnt[o_n];
                o_n2 = order_at(i + 128);
                const int m = __builtin_amdgcn_readfirstlane(min(64, n - i0));
                uint64_t alive = m == 64 ? ~0ull : (1ull << m) - 1ull;   // orders of the window in no tour (uniform)
                uint32_t t_l = 0;                               // lane j: tour of position i0 + j
                // a tour with room r takes, in sequence, every order of `rem`
                // that fits what it then has left; returns that
                auto fill = [&](uint32_t r, uint32_t t, uint64_t rem) -> uint32_t {
                    uint64_t taken = 0;
                    while (r >= mins) {
                        rem &= __ballot(s_l <= r);
                        if (!rem) break;
                        const int j = (int)__builtin_ctzll(rem);
                        r -= (uint32_t)__builtin_amdgcn_readlane((int)s_l, j);
                        taken |= 1ull << j;
                        rem &= rem - 1ull;                      // the next ones come after j
                    }
                    alive &= ~taken;
                    t_l = lane_in(taken) ? t : t_l;
                    return r;
                };
                // the open tours in opening order: those in the lanes, then the queued ones
                for (uint64_t live = __ballot(room >= mins); live && alive; live &= live - 1ull) {
                    const int f = (int)__builtin_ctzll(live);
                    room = set_lane(room, fill((uint32_t)__builtin_amdgcn_readlane((int)room, f),
                                               (uint32_t)__builtin_amdgcn_readlane((int)tour, f), alive), f);
                }
                for (int b = qh; b < qt && alive; b += 64) {
                    const uint32_t e = b + lane < qt ? queue[b + lane] : 0u;
                    uint32_t e_new = e;
                    for (uint64_t live = __ballot((e >> 16) >= mins); live && alive; live &= live - 1ull) {
                        const int f = (int)__builtin_ctzll(live);
                        const uint32_t ef = (uint32_t)__builtin_amdgcn_readlane((int)e, f);
                        e_new = set_lane(e_new, (fill(ef >> 16, ef & 0xFFFFu, alive) << 16) | (ef & 0xFFFFu), f);
                    }
                    if (b + lane < qt) queue[b + lane] = e_new;
                }
                // new tours for the orders left
                while (alive) {
                    const int j = (int)__builtin_ctzll(alive);
                    const uint32_t sz = (uint32_t)__builtin_amdgcn_readlane((int)s_l, j);
                    const uint32_t t = (uint32_t)T++;
                    alive &= alive - 1ull;
                    t_l = lane == j ? t : t_l;
                    uint32_t r = sz <= (uint32_t)Q ? (uint32_t)Q - sz : 0u;   // a larger order rides alone
                    if (r >= mins && alive) {
                        // the orders up to the first that does not fit, at once
                        // by their running sum, then one by one after it
                        const uint32_t cum = wave_incl_scan(lane_in(alive) ? s_l : 0u);
                        const uint64_t run = __ballot(cum <= r) & alive;
                        const uint64_t rest = alive & ~run;
                        if (run) {
                            r -= (uint32_t)__builtin_amdgcn_readlane((int)cum, 63 - (int)__builtin_clzll(run));
                            t_l = lane_in(run) ? t : t_l;
                        }
                        alive = rest;
                        r = fill(r, t, rest & (rest - 1ull));
                    }
                    if (r >= mins) {
                        if (k == 64) compact();
                        if (k < 64 && qh == qt) {
                            room = set_lane(room, r, k);
                            tour = set_lane(tour, t, k);
                            k++;
                        } else {
                            if (lane == 0) queue[qt] = (r << 16) | t;
                            qt++;
                        }
                    }
                }
                // queue stores before later loads of them (not without a queue:
                // the fence would wait for the loads ahead)
                if (qh < qt) __threadfence_block();
                // read after the tile loop's barrier
                if (i < n && o_l < (uint32_t)n) tour_of[o_l] = (uint16_t)t_l;
            }
        }

        __builtin_amdgcn_s_setprio(0);
        if constexpr (NW > 1) {
            if (tid == 0) rows[0] = (uint32_t)T;
            __syncthreads();                             // and the tour table
            T = __builtin_amdgcn_readfirstlane((int)rows[0]);
            __syncthreads();
        }

        // ---- 3. tiles of tours -----------------------------------------------
        int64_t acc = 0;
        for (int t0 = 0; t0 < T; t0 += TILE) {
            for (uint32_t k = tid; k < TILE * RW; k += NT) rows[k] = 0u;
            __syncthreads();
            if (ROUTE == WO_ROUTE_SSHAPE) {
                // aisle sets and farthest locations, one order per lane from
                // the groups of 64 orders of like size: an order outside the
                // tile loads none of its lines
                const uint32_t *grec = A.grec + I.grec_off;
                const uint32_t *gbase = A.gbase + I.gbase_off;
                const uint16_t *gord = A.gord + I.gord_off;
                // the next group's orders, tours and first lines load ahead
                struct Group {
                    uint32_t o, t, x[4], b0, len;
                };
                auto order_of = [&](int g) { return (uint32_t)gord[64 * min(g, I.n_grp - 1) + lane]; };   // 0xFFFF: no order
                auto load = [&](int g, uint32_t o) -> Group {
                    Group r;
                    g = min(g, I.n_grp - 1);
                    r.o = o;
                    r.b0 = gbase[g];
                    r.len = (gbase[g + 1] - r.b0) >> 6;                // lines of the group's longest order
                    r.t = tour_of[min(o, (uint32_t)n)];                // entry n: no tour
#pragma unroll
                    for (int q = 0; q < 4; q++)                         // shorter orders repeat their first line
                        r.x[q] = grec[r.b0 + 64u * min((uint32_t)q, r.len - 1u) + (uint32_t)lane];
                    return r;
                };
                Group nx = load(wv, order_of(wv));
                uint32_t o2 = order_of(wv + NW);
                for (int g = wv; g < I.n_grp; g += NW) {
                    const Group c = nx;
                    nx = load(g + NW, o2);
                    o2 = order_of(g + 2 * NW);
                    const uint32_t t = (c.o < (uint32_t)n ? c.t : 0xFFFFu) - (uint32_t)t0;
                    if (t >= (uint32_t)TILE) continue;
                    uint32_t far = 0;
                    auto add = [&](uint32_t x) {
                        const uint32_t ls = x + zs[x >> 26];
                        const uint32_t a = mulhi24(ls, I.magic);
                        atomicOr(&rows[t * RW + 1u + (a >> 5)], 1u << (a & 31u));
                        far = max(far, ls);
                    };
#pragma unroll
                    for (int q = 0; q < 4; q++)
                        if ((uint32_t)q < c.len) add(c.x[q]);
                    for (uint32_t k = 4; k < c.len; k++) add(grec[c.b0 + 64u * k + (uint32_t)lane]);
                    atomicMax(&rows[t * RW], far);
                }
            } else {
                // pick rows: every line exactly once, from the instance's line
                // records, which name their order by its entry in the
                // next-fit kernel's tour table (the padding records name
                // order n)
                const uint32_t nf_tour = eval_layout(n, I.n_units, (uint32_t)I.row_b, I.t_cap).tour;
                const uint2 *lines = A.lines + I.line_off;
                // eight lines a lane at a time: their records, then their tours, are
                // in flight together (4,096 paper-scale plans in first fit by
                // the optimal route 759 to 585 us; 491 with scalar
                // reads of the instance table)
                constexpr int U = 8;
                static_assert(LINE_PAD % (64 * U) == 0, "whole rounds");
                for (int r0 = lane; r0 < I.n_lines_pad; r0 += 64 * U) {
                    uint32_t x[U], t[U];
#pragma unroll
                    for (int u = 0; u < U; u++) {
                        const uint2 rec = lines[r0 + 64 * u];
                        const uint32_t o = ((rec.y & 0x7FFFFFFFu) - nf_tour) >> 1;
                        x[u] = rec.x;
                        t[u] = o < (uint32_t)n ? o : (uint32_t)n;
                    }
#pragma unroll
                    for (int u = 0; u < U; u++) t[u] = t[u] < (uint32_t)n ? (uint32_t)tour_of[t[u]] : 0xFFFFu;
#pragma unroll
                    for (int u = 0; u < U; u++) {
                        const uint32_t row = t[u] - (uint32_t)t0;
                        if (row >= (uint32_t)TILE) continue;
                        const uint32_t e = atomicAdd(&rows[row * RW], 1u);
                        rows[row * RW + 1u + min(e, (uint32_t)I.pick_slots - 1u)] = x[u] + zs[x[u] >> 26];
                    }
                }
            }
            __syncthreads();
            for (int tt = tid; tt < TILE && t0 + tt < T; tt += NT) {
                const uint32_t *rw = rows + (uint32_t)tt * RW;
                if (ROUTE == WO_ROUTE_SSHAPE) {
                    const uint32_t ls = rw[0];
                    int k = 0;
                    for (int w = 0; w < I.words; w++) k += __popc(rw[1 + w]);
                    const uint32_t a = mulhi24(ls, I.magic);
                    const int64_t y = (int64_t)((ls - a * I.d_s) >> (I.shift + 1)) * I.pitch + I.pitch / 2;
                    acc += 2ll * wsp * a + ((k & 1) ? (int64_t)(k - 1) * I.L + 2 * y : (int64_t)k * I.L);
                } else {
                    const uint32_t np = rw[0];
                    if (np == 0) continue;                  // only a malformed row leaves a tour empty
                    if (np > (uint32_t)I.pick_slots) continue;   // an order routed apart (below)
                    acc += pick_route_cost<ROUTE>(rw + 1, np, wsp, I, I.magic);
                }
            }
            __syncthreads();
        }
        // orders longer than a pick row, each a tour of its own
        if (ROUTE != WO_ROUTE_SSHAPE && I.n_big > 0) acc += big_orders_cost<ROUTE, 64>(A, I, zs, rows, wsp);

        // ---- 4. sum and rate -----------------------------------------------
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) acc += __shfl_xor(acc, d, 64);
        if constexpr (NW > 1) {
            int64_t *part = (int64_t *)rows;             // the last tile's rows are read
            if (tid == 64) *part = acc;
            __syncthreads();
            acc += *part;                                // thread 0's
        }
        if (A.validate && bad) atomicOr(A.err, 1);
        if (tid == 0) {
            A.dist[p] = acc > 2147483647ll ? 2147483647 : (int32_t)acc;
            if (A.thr) A.thr[p] = window_throughput(acc, I);
        }
        __syncthreads();
    }
}

template <int ROUTE, int BATCH>
static hipError_t launch_eval_ff_r(const EvalArgs &a, uint32_t lds_bytes, int grid, hipStream_t s)
{
    static uint32_t attr_bytes = 0;
    if (lds_bytes > attr_bytes) {
        hipError_t e = hipFuncSetAttribute((const void *)eval_ff_kernel<ROUTE, BATCH>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return e;
        }
        attr_bytes = lds_bytes;
    }
    hipLaunchKernelGGL((eval_ff_kernel<ROUTE, BATCH>), dim3(grid), dim3(ff_threads(ROUTE, BATCH)), lds_bytes, s, a);
    return hipGetLastError();
}

template <int BATCH>
static hipError_t launch_eval_ff_s(const EvalArgs &a, uint32_t lds_bytes, int grid, int route, hipStream_t s)
{
    switch (route) {
    case WO_ROUTE_SSHAPE: return launch_eval_ff_r<WO_ROUTE_SSHAPE, BATCH>(a, lds_bytes, grid, s);
    case WO_ROUTE_RETURN: return launch_eval_ff_r<WO_ROUTE_RETURN, BATCH>(a, lds_bytes, grid, s);
    case WO_ROUTE_LARGEST_GAP: return launch_eval_ff_r<WO_ROUTE_LARGEST_GAP, BATCH>(a, lds_bytes, grid, s);
    case WO_ROUTE_OPTIMAL: return launch_eval_ff_r<WO_ROUTE_OPTIMAL, BATCH>(a, lds_bytes, grid, s);
    case WO_ROUTE_COMBINED: return launch_eval_ff_r<WO_ROUTE_COMBINED, BATCH>(a, lds_bytes, grid, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_eval_ff(const EvalArgs &a, uint32_t lds_bytes, int grid, int route, int batch, hipStream_t s)
{
    switch (batch) {
    case FF_FIRST_FIT: return launch_eval_ff_s<FF_FIRST_FIT>(a, lds_bytes, grid, route, s);
    case FF_SEED: return launch_eval_ff_s<FF_SEED>(a, lds_bytes, grid, route, s);
    case FF_SEED_PACKED: return launch_eval_ff_s<FF_SEED_PACKED>(a, lds_bytes, grid, route, s);
    }
    return hipErrorInvalidValue;
}

template <int ROUTE, int BATCH>
static int ff_max_blocks_r(uint32_t lds_bytes)
{
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, eval_ff_kernel<ROUTE, BATCH>, ff_threads(ROUTE, BATCH), lds_bytes) != hipSuccess) {
        (void)hipGetLastError();
        return 1;
    }
    return std::max(1, std::min(n, lds_fit(lds_bytes)));
}

template <int BATCH>
static int ff_max_blocks_s(int route, uint32_t lds_bytes)
{
    switch (route) {
    case WO_ROUTE_RETURN: return ff_max_blocks_r<WO_ROUTE_RETURN, BATCH>(lds_bytes);
    case WO_ROUTE_LARGEST_GAP: return ff_max_blocks_r<WO_ROUTE_LARGEST_GAP, BATCH>(lds_bytes);
    case WO_ROUTE_OPTIMAL: return ff_max_blocks_r<WO_ROUTE_OPTIMAL, BATCH>(lds_bytes);
    case WO_ROUTE_COMBINED: return ff_max_blocks_r<WO_ROUTE_COMBINED, BATCH>(lds_bytes);
    }
    return ff_max_blocks_r<WO_ROUTE_SSHAPE, BATCH>(lds_bytes);
}

int eval_ff_max_blocks_per_cu(int route, int batch, uint32_t lds_bytes)
{
    switch (batch) {
    case FF_SEED: return ff_max_blocks_s<FF_SEED>(route, lds_bytes);
    case FF_SEED_PACKED: return ff_max_blocks_s<FF_SEED_PACKED>(route, lds_bytes);
    }
    return ff_max_blocks_s<FF_FIRST_FIT>(route, lds_bytes);
}

}  // namespace wo
