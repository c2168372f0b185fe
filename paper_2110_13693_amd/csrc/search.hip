// Genetic plan search on gfx950 (the top-level optimiser of the paper's SDO,
// section 5, organising the clustering and sequencing searches of section 6).
//
// Random numbers come from a counter generator: the SplitMix64 finaliser
// (Steele, Lea & Flood 2014) over (seed, stream, generation, child, position),
// so every draw is recomputable anywhere.  Operators:
//   - tournament: `tsize` uniform draws from the population, winner = the
//     smallest (distance, index);
//   - zone swap: for each category position c in turn, with probability
//     thr / 2^32, swap its zone with a uniformly chosen other position;
//   - order insert: for each sequence position i = 0 .. n-1 in turn, with the
//     same probability, move the element currently at i so that it ends at a
//     uniform position j;
//   - uniform integers in [0, m): (r32 * m) >> 32.
#include "eval_device.h"
#include "wo_search.h"

namespace wo {

static __device__ __forceinline__ uint64_t splitmix64(uint64_t x)
{
    uint64_t z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

static __device__ __forceinline__ uint32_t draw(uint64_t seed, uint32_t stream, uint32_t gen, uint32_t child,
                                                uint32_t pos)
{
    uint64_t h = splitmix64(seed + stream);
    h = splitmix64(h ^ (((uint64_t)gen << 32) | child));
    h = splitmix64(h ^ (uint64_t)pos);
    return (uint32_t)(h >> 32);
}

static __device__ __forceinline__ uint32_t uniform(uint32_t r, uint32_t m)
{
    return (uint32_t)(((uint64_t)r * m) >> 32);
}

static __device__ int tournament(const int32_t *dist, int P, int tsize, uint64_t seed, uint32_t gen, uint32_t child)
{
    int best = -1;
    int32_t bd = 0;
    for (int k = 0; k < tsize; k++) {
        const int i = (int)uniform(draw(seed, RS_TOURNAMENT, gen, child, (uint32_t)k), (uint32_t)P);
        const int32_t d = dist[i];
        if (best < 0 || d < bd || (d == bd && i < best)) {
            best = i;
            bd = d;
        }
    }
    return best;
}

static __device__ void mutate_zones(uint8_t *z, int C, uint32_t thr, uint64_t seed, uint32_t gen, uint32_t child)
{
    if (C < 2) return;
    for (int c = 0; c < C; c++) {
        if (draw(seed, RS_ZONE_COIN, gen, child, (uint32_t)c) < thr) {
            uint32_t j = uniform(draw(seed, RS_ZONE_PARTNER, gen, child, (uint32_t)c), (uint32_t)(C - 1));
            if ((int)j >= c) j++;
            const uint8_t t = z[c];
            z[c] = z[j];
            z[j] = t;
        }
    }
}

// Index of the best individual (smallest distance, then index).  One block.
__global__ __launch_bounds__(1024) void argmin_kernel(const int32_t *dist, int P, int32_t *out)
{
    __shared__ unsigned long long best[1024];
    unsigned long long b = ~0ull;
    for (int i = threadIdx.x; i < P; i += 1024) {
        const unsigned long long k = ((unsigned long long)(uint32_t)(dist[i] ^ 0x80000000) << 32) | (uint32_t)i;
        b = k < b ? k : b;
    }
    best[threadIdx.x] = b;
    __syncthreads();
    for (int s = 512; s >= 1; s >>= 1) {
        if ((int)threadIdx.x < s && best[threadIdx.x + s] < best[threadIdx.x]) best[threadIdx.x] = best[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = (int32_t)(best[0] & 0xFFFFFFFFull);
}

// Screened arm: candidate slottings (tournament winner's zones, mutated).
__global__ __launch_bounds__(256) void candidates_kernel(CandArgs a)
{
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b >= a.K) return;
    const int par = tournament(a.pd, a.P, a.tsize, a.seed, a.gen, (uint32_t)b);
    uint8_t z[64];
    for (int c = 0; c < 64; c++) z[c] = a.pz[(int64_t)par * 64 + c];
    mutate_zones(z, a.C, a.thr, a.seed, a.gen, (uint32_t)b);
    for (int c = 0; c < 64; c++) a.cand_zone[(int64_t)b * 64 + c] = z[c];
    a.cand_parent[b] = par;
}

// One workgroup per child: choose the parent, mutate zones and sequence.
//
// The insert moves of a child (about 80 at 4,000 orders and 2 %) are applied
// without shifting the sequence: the elements that never move keep their
// order, so only the moved ones are tracked.  One wave holds them, one per
// lane: O, the element's index in the sequence before the moves; P, its
// position now; R, the number of elements not moved before O.  A move of the
// element at position i to j finds it among the tracked ones (P = i), or as the
// not-moved element of rank i - #(P < i), whose index is that rank + #(R <=
// rank); then the P between i and j shift by one.  After up to BR_TRACK moves
// the sequence is rebuilt in two passes: the elements not moved close up (an
// element's place is its index less the moved ones before it, from a bitmap
// with running counts), then spread over the positions not taken.  A sequence
// of more moves is rebuilt several times, in place in LDS; the first rebuild
// reads the parent and the last writes the child.
//
// The coins, one draw per position, are the largest part of the rest.  The
// moves' targets are drawn 64 at a time, the zone mutation by one lane per
// category.  16,384 children of 4,000 orders: 232 us (the VALU busy 77 % of
// it), against 968 us when every move shifted its range in LDS between
// barriers and one thread drew the zone coins.  Four waves per child instead of
// two, and a longer list: 337 us (8 children per CU instead of 15).
constexpr int BR_THREADS = 128, BR_BLK = 4096;       // positions whose coins are drawn together
constexpr int BR_LIST = 512;                         // moves listed together: at least 8 words of coins
constexpr int BR_TRACK = 128;                        // moves per rebuild: two per lane of the tracking wave

__host__ __device__ inline uint32_t br_words(int n) { return (uint32_t)n / 32u + 1u; }
struct BreedLayout {
    uint32_t coins, list, bits, pre, buf, total;
};
__host__ __device__ inline BreedLayout breed_layout(int n)
{
    BreedLayout L;
    uint32_t b = 0;
    L.coins = b;  b += 8u * (BR_BLK / 64);
    L.list = b;   b += 2u * BR_LIST;
    L.bits = b;   b = align16(b + 4u * br_words(n));
    L.pre = b;    b = align16(b + 2u * br_words(n));
    L.buf = b;    b = align16(b + 2u * (uint32_t)n + 16u);   // whole pieces of 8 entries
    L.total = b;
    return L;
}

// draw() at many positions of one (seed, stream, generation, child).  The
// position changes the low word of the last finaliser's argument only, so
// after the addition the high word is one of two values (with and without the
// carry): its part of the first shift and product is made once for both.  The
// 32 result bits then need 5 multiplications of 32 bits instead of 7.
struct DrawKey {
    uint32_t lo, s0, s1, t0, t1;
};
static __device__ __forceinline__ DrawKey draw_key(uint64_t seed, uint32_t stream, uint32_t gen, uint32_t child)
{
    const uint64_t key = splitmix64(splitmix64(seed + stream) ^ (((uint64_t)gen << 32) | child));
    const uint32_t h0 = (uint32_t)(key >> 32) + 0x9E3779B9u, h1 = h0 + 1u;
    return {(uint32_t)key, h0 << 2, h1 << 2, (h0 ^ (h0 >> 30)) * 0x1CE4E5B9u, (h1 ^ (h1 >> 30)) * 0x1CE4E5B9u};
}
static __device__ __forceinline__ uint32_t draw_at(const DrawKey &k, uint32_t pos)
{
    const uint32_t lo = (k.lo ^ pos) + 0x7F4A7C15u;
    const bool carry = lo < 0x7F4A7C15u;
    const uint32_t z = lo ^ (lo >> 30) ^ (carry ? k.s1 : k.s0);
    const uint64_t p = (uint64_t)z * 0x1CE4E5B9u;
    const uint32_t ph = (uint32_t)(p >> 32) + z * 0xBF58476Du + (carry ? k.t1 : k.t0), pl = (uint32_t)p;
    const uint32_t yl = pl ^ ((pl >> 27) | (ph << 5)), yh = ph ^ (ph >> 27);
    const uint32_t r = __umulhi(yl, 0x133111EBu) + yl * 0x94D049BBu + yh * 0x133111EBu;
    return r ^ (r >> 31);
}

__global__ __launch_bounds__(BR_THREADS) void breed_kernel(BreedArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_par, s_cid, s_m, s_next;
    const int c = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = a.n;
    const BreedLayout L = breed_layout(n);
    uint64_t *coins = (uint64_t *)(smem + L.coins);
    uint16_t *list = (uint16_t *)(smem + L.list);
    uint32_t *bits = (uint32_t *)(smem + L.bits);
    uint16_t *pre = (uint16_t *)(smem + L.pre);
    uint16_t *buf = (uint16_t *)(smem + L.buf);
    const bool elite = a.mode == 0 && c == 0;
    // ---- parent and zones: one wave -------------------------------------
    if (w == 0) {
        uint32_t cid = (uint32_t)c;
        int par;
        if (a.mode != 0) {
            cid = (uint32_t)__builtin_amdgcn_readfirstlane(a.kept[c]);
            par = a.cand_parent[cid];
        } else if (elite) {
            par = a.best[0];
        } else {
            // tournament, one draw per lane: smallest (distance, index)
            unsigned long long best = ~0ull;
            if (lane < a.tsize) {
                const DrawKey key = draw_key(a.seed, RS_TOURNAMENT, a.gen, cid);
                const uint32_t i = uniform(draw_at(key, (uint32_t)lane), (uint32_t)a.P);
                best = ((unsigned long long)((uint32_t)a.pd[i] ^ 0x80000000u) << 32) | i;
            }
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) {
                const unsigned long long o = __shfl_xor(best, d, 64);
                best = o < best ? o : best;
            }
            par = (int)(uint32_t)best;
        }
        par = __builtin_amdgcn_readfirstlane(par);
        uint32_t z = a.mode == 0 ? a.pz[(int64_t)par * 64 + lane] : a.cand_zone[(int64_t)cid * 64 + lane];
        if (a.mode == 0 && !elite && a.C >= 2) {
            const DrawKey kc = draw_key(a.seed, RS_ZONE_COIN, a.gen, cid), kp = draw_key(a.seed, RS_ZONE_PARTNER, a.gen, cid);
            uint64_t m = __ballot(lane < a.C && draw_at(kc, (uint32_t)lane) < a.thr);
            uint32_t j = uniform(draw_at(kp, (uint32_t)lane), (uint32_t)(a.C - 1));
            j += (int)j >= lane;
            while (m) {                              // the swaps in category order
                const int x = (int)__builtin_ctzll(m);
                m &= m - 1ull;
                const int y = __builtin_amdgcn_readlane((int)j, x);
                const int zx = __builtin_amdgcn_readlane((int)z, x), zy = __builtin_amdgcn_readlane((int)z, y);
                z = lane == x ? (uint32_t)zy : (lane == y ? (uint32_t)zx : z);
            }
        }
        a.cz[(int64_t)c * 64 + lane] = (uint8_t)z;
        if (lane == 0) {
            s_par = par;
            s_cid = (int)cid;
        }
    }
    __syncthreads();
    const int par = __builtin_amdgcn_readfirstlane(s_par);
    const uint32_t cid = (uint32_t)__builtin_amdgcn_readfirstlane(s_cid);
    const uint16_t *src = a.ps + (int64_t)par * n;
    uint16_t *dst = a.cs + (int64_t)c * n;
    const bool whole = n % 8 == 0;                   // rows of whole 16-byte pieces
    if (elite) {
        if (whole)
            for (int i = tid; i < n / 8; i += BR_THREADS) ((uint4 *)dst)[i] = ((const uint4 *)src)[i];
        else
            for (int i = tid; i < n; i += BR_THREADS) dst[i] = src[i];
        return;
    }
    const DrawKey k_coin = draw_key(a.seed, RS_INSERT_COIN, a.gen, cid);
    const DrawKey k_to = draw_key(a.seed, RS_INSERT_TARGET, a.gen, cid);

    bool first = true;                               // the sequence is still the parent's
    for (int blk = 0; blk < n; blk += BR_BLK) {
        // ---- the block's coins, then the positions with a move -------------
        const int nb = min(BR_BLK, n - blk), words = (nb + 63) / 64;
        for (int x = w; x < words; x += BR_THREADS / 64) {
            const int i = blk + 64 * x + lane;
            const uint64_t b = __ballot(i < n && draw_at(k_coin, (uint32_t)i) < a.thr);
            if (lane == 0) coins[x] = b;
        }
        __syncthreads();
        for (int w0 = 0; w0 < words;) {
            if (w == 0) {
                // the moves of words w0 and on, as many as the list holds
                const bool in = lane >= w0 && lane < words;
                uint64_t b = in ? coins[lane] : 0ull;
                const uint32_t k = (uint32_t)__popcll(b), inc = wave_incl_scan(k);
                const uint64_t take = __ballot(in && inc <= (uint32_t)BR_LIST);   // consecutive words from w0
                uint32_t at = inc - k;
                if (!lane_in(take)) b = 0ull;
                while (b) {
                    list[at++] = (uint16_t)(blk + 64 * lane + (int)__builtin_ctzll(b));
                    b &= b - 1ull;
                }
                const int nx = w0 + (int)__builtin_popcountll(take);
                if (lane == nx - 1) s_m = (int)inc;
                if (lane == 0) s_next = nx;
            }
            __syncthreads();
            const int m = __builtin_amdgcn_readfirstlane(s_m);
            w0 = __builtin_amdgcn_readfirstlane(s_next);
            const bool end = blk + BR_BLK >= n && w0 >= words;   // the last moves write the child, moves or not
            for (int t0 = 0; t0 < m || (end && t0 == 0); t0 += BR_TRACK) {
                const bool last = end && t0 + BR_TRACK >= m;
                uint32_t O[2] = {0, 0}, P[2] = {~0u, ~0u}, V[2] = {0, 0};
                int count = 0;                           // tracked elements (uniform in the tracking wave)
                // the tracked elements' bits at `at`, and the bits before each word
                auto mark = [&](const uint32_t (&at)[2]) {
                    const int nw = (int)br_words(n);
                    for (int x = lane; x < nw; x += 64) bits[x] = 0u;
                    lds_order();
                    if (lane < count) atomicOr(&bits[at[0] >> 5], 1u << (at[0] & 31u));
                    if (lane + 64 < count) atomicOr(&bits[at[1] >> 5], 1u << (at[1] & 31u));
                    lds_order();
                    uint32_t carry = 0;
                    for (int x0 = 0; x0 < nw; x0 += 64) {
                        const uint32_t k = x0 + lane < nw ? (uint32_t)__popc(bits[x0 + lane]) : 0u;
                        const uint32_t inc = wave_incl_scan(k) + carry;
                        if (x0 + lane < nw) pre[x0 + lane] = (uint16_t)(inc - k);
                        carry = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
                    }
                };
                if (w == 0) {
                    __builtin_amdgcn_s_setprio(2);   // a chain the other waves wait for
                    uint32_t R[2] = {~0u, ~0u};
                    const int g1 = min(m, t0 + BR_TRACK);
                    for (int g0 = t0; g0 < g1; g0 += 64) {
                        // position and target of the next (at most 64) moves, one per lane
                        const uint32_t vi = list[min(g0 + lane, m - 1)];
                        const uint32_t vj = uniform(draw_at(k_to, vi), (uint32_t)n);
                        const int g = min(64, g1 - g0);
                        for (int t = 0; t < g; t++) {
                            const uint32_t i = (uint32_t)__builtin_amdgcn_readlane((int)vi, t);
                            const uint32_t j = (uint32_t)__builtin_amdgcn_readlane((int)vj, t);
                            if (i == j) continue;
                            // (lanes not yet used hold values that match nothing)
                            const uint64_t h0 = __ballot(P[0] == i);
                            const uint64_t h1 = count > 64 ? __ballot(P[1] == i) : 0ull;
                            int k;
                            if (h0 | h1) {
                                k = h0 ? (int)__builtin_ctzll(h0) : 64 + (int)__builtin_ctzll(h1);
                            } else {
                                uint32_t u = i - (uint32_t)__builtin_popcountll(__ballot(P[0] < i));
                                if (count > 64) u -= (uint32_t)__builtin_popcountll(__ballot(P[1] < i));
                                uint32_t o = u + (uint32_t)__builtin_popcountll(__ballot(R[0] <= u));
                                R[0] -= R[0] > u;
                                if (count > 64) {
                                    o += (uint32_t)__builtin_popcountll(__ballot(R[1] <= u));
                                    R[1] -= R[1] > u;
                                }
                                k = count++;
                                if (k < 64) {
                                    O[0] = set_lane(O[0], o, k);
                                    R[0] = set_lane(R[0], u, k);
                                } else {
                                    O[1] = set_lane(O[1], o, k - 64);
                                    R[1] = set_lane(R[1], u, k - 64);
                                }
                            }
                            // the tracked positions between i and j shift by one
                            const uint32_t lo = i < j ? i + 1u : j, len = i < j ? j - i : i - j;
                            const uint32_t by = i < j ? ~0u : 1u;
                            P[0] += P[0] - lo < len ? by : 0u;
                            if (count > 64) P[1] += P[1] - lo < len ? by : 0u;
                            if (k < 64) P[0] = set_lane(P[0], j, k);
                            else P[1] = set_lane(P[1], j, k - 64);
                        }
                    }
                    // the tracked elements themselves (count is 0 where no move was made)
                    if (lane < count) V[0] = first ? src[O[0]] : buf[O[0]];
                    if (lane + 64 < count) V[1] = first ? src[O[1]] : buf[O[1]];
                    mark(O);
                    __builtin_amdgcn_s_setprio(0);
                }
                __syncthreads();
                // ---- the elements not moved close up ---------------------------
                for (int b0 = 0; b0 < n; b0 += 8 * BR_THREADS) {
                    const int p0 = b0 + 8 * tid;
                    uint32_t v[8];
                    if (p0 < n) {
                        if (!first || whole) {
                            const uint4 q = *(const uint4 *)((first ? src : buf) + p0);
                            v[0] = q.x & 0xFFFFu; v[1] = q.x >> 16; v[2] = q.y & 0xFFFFu; v[3] = q.y >> 16;
                            v[4] = q.z & 0xFFFFu; v[5] = q.z >> 16; v[6] = q.w & 0xFFFFu; v[7] = q.w >> 16;
                        } else {
    #pragma unroll
                            for (int q = 0; q < 8; q++) v[q] = src[min(p0 + q, n - 1)];
                        }
                    }
                    if (!first) __syncthreads();         // in place: a piece is read before it is written
                    if (p0 < n) {
                        const uint32_t x = bits[p0 >> 5];
                        uint32_t d = (uint32_t)p0 - pre[p0 >> 5] - (uint32_t)__popc(x & ((1u << (p0 & 31)) - 1u));
                        const uint32_t gone = x >> (p0 & 31);
    #pragma unroll
                        for (int q = 0; q < 8; q++)
                            if (p0 + q < n && !((gone >> q) & 1u)) buf[d++] = (uint16_t)v[q];
                    }
                    if (!first) __syncthreads();
                }
                __syncthreads();
                if (w == 0) mark(P);
                __syncthreads();
                // ---- and spread over the positions not taken, from the top -----
                for (int b0 = (n - 1) / (8 * BR_THREADS) * (8 * BR_THREADS); b0 >= 0; b0 -= 8 * BR_THREADS) {
                    const int p0 = b0 + 8 * tid;
                    uint32_t v[8];
                    if (p0 < n) {
                        const uint32_t x = bits[p0 >> 5];
                        uint32_t d = (uint32_t)p0 - pre[p0 >> 5] - (uint32_t)__popc(x & ((1u << (p0 & 31)) - 1u));
                        const uint32_t taken = x >> (p0 & 31);
    #pragma unroll
                        for (int q = 0; q < 8; q++) {
                            v[q] = buf[min(d, (uint32_t)(n - 1))];
                            d += !((taken >> q) & 1u);
                        }
                    }
                    if (!last) __syncthreads();
                    if (p0 < n) {
                        if (!last || whole) {
                            *(uint4 *)((last ? dst : buf) + p0) =
                                make_uint4(v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16));
                        } else {
    #pragma unroll
                            for (int q = 0; q < 8; q++)
                                if (p0 + q < n) dst[p0 + q] = (uint16_t)v[q];
                        }
                    }
                    if (!last) __syncthreads();
                }
                __syncthreads();
                if (w == 0) {
                    uint16_t *to = last ? dst : buf;
                    if (lane < count) to[P[0]] = (uint16_t)V[0];
                    if (lane + 64 < count) to[P[1]] = (uint16_t)V[1];
                }
                __syncthreads();
                first = false;
            }
            __syncthreads();                         // the list is read
        }
    }
}

// Screened arm: the evaluated children replace the worst individuals.
__global__ __launch_bounds__(256) void replace_kernel(ReplaceArgs a)
{
    const int r = blockIdx.x;
    const int dst = a.worst[r];
    for (int k = threadIdx.x; k < 64; k += 256) a.pz[(int64_t)dst * 64 + k] = a.cz[(int64_t)r * 64 + k];
    for (int k = threadIdx.x; k < a.n; k += 256) a.ps[(int64_t)dst * a.n + k] = a.cs[(int64_t)r * a.n + k];
    if (threadIdx.x == 0) a.pd[dst] = a.cd[r];
}

hipError_t launch_argmin(const int32_t *dist, int P, int32_t *out, hipStream_t s)
{
    hipLaunchKernelGGL(argmin_kernel, dim3(1), dim3(1024), 0, s, dist, P, out);
    return hipGetLastError();
}

hipError_t launch_candidates(const CandArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(candidates_kernel, dim3((a.K + 255) / 256), dim3(256), 0, s, a);
    return hipGetLastError();
}

uint32_t breed_lds_bytes(int n) { return breed_layout(n).total; }

hipError_t launch_breed(const BreedArgs &a, int n_children, hipStream_t s)
{
    static uint32_t attr_bytes = 0;
    const uint32_t need = breed_lds_bytes(a.n);
    if (need > attr_bytes) {
        hipError_t e = hipFuncSetAttribute((const void *)breed_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)need);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return e;
        }
        attr_bytes = need;
    }
    hipLaunchKernelGGL(breed_kernel, dim3(n_children), dim3(BR_THREADS), breed_lds_bytes(a.n), s, a);
    return hipGetLastError();
}

hipError_t launch_replace(const ReplaceArgs &a, int keep, hipStream_t s)
{
    hipLaunchKernelGGL(replace_kernel, dim3(keep), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace wo
