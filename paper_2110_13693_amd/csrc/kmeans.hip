// Class-based storage by K-means on pick frequency (section 5, Subproblem 3:
// products are placed by how often they are picked, with an unsupervised
// clustering such as K-means, MacQueen 1967).  The feature of a SKU is the
// number of order lines naming it; Lloyd's iteration clusters the SKUs into
// k classes, numbered by descending mean frequency, which become the
// categories the zones hold.
//
// SKUs of equal frequency always share a cluster, so after the frequencies
// and their histogram the iteration runs over the histogram's non-empty bins,
// all of it in one workgroup (km_lloyd_kernel).  The arithmetic is exact: a centroid is the
// rational S / N, and f is nearer to S_j / N_j than to S_k / N_k iff
// |f N_j - S_j| N_k < |f N_k - S_k| N_j, compared in 128 bits (ties to the
// lower index).  Start: centroid c is the distinct frequency of rank
// floor((2c + 1) D / (2k)) among the D distinct ones.  A step assigns every
// bin and moves each non-empty cluster's centroid to its members' mean; the
// iteration ends at the first assignment equal to the previous one or after
// max_iter assignments.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "wo_common.h"

namespace {

constexpr int KM_MAX = 64;

struct KmState {
    int k_used, n_iter, err, pad;         // the results a caller reads, together
    int rank[KM_MAX];
};

// a * b < c * d for a, c < 2^47 and b, d < 2^23 (products up to 2^70: 128 bits)
__device__ __forceinline__ bool less_prod(unsigned long long a, unsigned long long b, unsigned long long c,
                                          unsigned long long d)
{
    const unsigned long long h1 = __umul64hi(a, b), h2 = __umul64hi(c, d);
    return h1 < h2 || (h1 == h2 && a * b < c * d);
}

__device__ __forceinline__ unsigned long long absdiff(long long x, long long y) { return x > y ? x - y : y - x; }

// SKU ids are popularity ranks, so the low ids take most lines: their counts
// gather in the workgroup's LDS first and reach memory once per workgroup.
constexpr int KM_HOT_SKUS = 2048;
__global__ __launch_bounds__(1024) void km_freq_kernel(const int32_t *skus, int64_t n_lines, int32_t n_skus,
                                                       int32_t *freq, KmState *st)
{
    __shared__ int32_t hot[KM_HOT_SKUS];
    for (int i = threadIdx.x; i < KM_HOT_SKUS; i += blockDim.x) hot[i] = 0;
    __syncthreads();
    for (int64_t l = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; l < n_lines; l += (int64_t)gridDim.x * blockDim.x) {
        const int32_t s = skus[l];
        if (s < 0 || s >= n_skus) atomicOr(&st->err, 1);
        else if (s < KM_HOT_SKUS) atomicAdd(&hot[s], 1);
        else atomicAdd(&freq[s], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < KM_HOT_SKUS && i < n_skus; i += blockDim.x)
        if (hot[i]) atomicAdd(&freq[i], hot[i]);
}

// Most SKUs share a few low frequencies (most are never picked), so the
// counts of frequencies below KM_HOT gather in the workgroup's LDS first (the
// lanes of a wave holding the first active lane's frequency add theirs with
// one atomic), and each workgroup adds them to memory once; higher
// frequencies, few SKUs each, go to memory directly.
constexpr int KM_HOT = 64;
__global__ __launch_bounds__(1024) void km_hist_kernel(const int32_t *freq, int32_t n_skus, int32_t *hist)
{
    __shared__ int32_t hot[KM_HOT];
    if (threadIdx.x < KM_HOT) hot[threadIdx.x] = 0;
    __syncthreads();
    for (int32_t s0 = blockIdx.x * blockDim.x; s0 < n_skus; s0 += gridDim.x * blockDim.x) {
        const int32_t s = s0 + threadIdx.x;
        const bool act = s < n_skus;
        const int32_t f = act ? freq[s] : -1;
        const uint64_t live = __ballot(act);
        if (!live) continue;
        const int32_t f0 = __shfl(f, __builtin_ctzll(live), 64);
        const uint64_t same = __ballot(act && f == f0);
        if (act && f == f0) {
            if ((threadIdx.x & 63) == __builtin_ctzll(same)) {
                if (f0 < KM_HOT) atomicAdd(&hot[f0], __popcll(same));
                else atomicAdd(&hist[f0], __popcll(same));
            }
        } else if (act) {
            if (f < KM_HOT) atomicAdd(&hot[f], 1);
            else atomicAdd(&hist[f], 1);
        }
    }
    __syncthreads();
    if (threadIdx.x < KM_HOT && hot[threadIdx.x]) atomicAdd(&hist[threadIdx.x], hot[threadIdx.x]);
}

__global__ void km_label_kernel(const int32_t *freq, int32_t n_skus, const int32_t *label, const KmState *st,
                                int32_t *category)
{
    for (int32_t s = blockIdx.x * blockDim.x + threadIdx.x; s < n_skus; s += gridDim.x * blockDim.x)
        category[s] = st->rank[label[freq[s]]];
}

// The whole iteration in one workgroup: the non-empty bins (the distinct
// frequencies, at most sqrt(2 n_lines) + 1 <= KM_MAX_BINS of them since the
// positive ones sum to at most n_lines) are compacted in order into LDS, 8
// bins per thread and pass; then the start, every assignment and centroid
// move, and the ranking run with block barriers between them, and the bins'
// labels and the results go to memory once.
//
// There are about a hundred bins at the paper scale, and the assignment is a
// chain of comparisons per bin: G = 2^g lanes share a bin, each taking every
// G-th cluster, and the best of them follows in g exchanges (smallest distance,
// ties to the lower index: associative, as the distances are exact).
// EXACT64: n_lines * n_skus^2 < 2^53, which bounds every product of a
// comparison, so that doubles hold them exactly; else 128-bit products.  10,006
// lines over 150,000 SKUs, 16 classes, 9 assignments: 21 us, against 41 with one
// lane per bin and 128-bit products throughout.
constexpr int KM_MAX_BINS = 5800;
constexpr int KM_BLOCK = 1024;

template <bool EXACT64>
__global__ __launch_bounds__(KM_BLOCK) void km_lloyd_kernel(const int32_t *hist, int32_t n_bins, int32_t k,
                                                           int32_t max_iter, int32_t *label, KmState *st)
{
    __shared__ int32_t bv[KM_MAX_BINS], bm[KM_MAX_BINS];
    __shared__ uint8_t bl[KM_MAX_BINS];
    __shared__ unsigned long long S2[KM_MAX];       // the assignment's sums: frequency total << 32 | members
    __shared__ long long S[KM_MAX], N[KM_MAX], cnt[KM_MAX];
    __shared__ double Sd[KM_MAX], Nd[KM_MAX];
    __shared__ int part[2][KM_BLOCK / 64];
    __shared__ int changed_s[2];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // ---- compaction of the non-empty bins, in order of frequency
    int D = 0;
    for (int v0 = 0, par = 0; v0 < n_bins; v0 += 8 * KM_BLOCK, par ^= 1) {
        const int v = v0 + 8 * tid;                  // the array is padded to whole pieces of zeros
        int m[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        if (v < n_bins) {
            const int4 x = *(const int4 *)(hist + v), y = *(const int4 *)(hist + v + 4);
            m[0] = x.x; m[1] = x.y; m[2] = x.z; m[3] = x.w;
            m[4] = y.x; m[5] = y.y; m[6] = y.z; m[7] = y.w;
        }
        int own = 0;
#pragma unroll
        for (int j = 0; j < 8; j++) own += m[j] > 0;
        int inc = own;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int u = __shfl_up(inc, d, 64);
            if (lane >= d) inc += u;
        }
        if (lane == 63) part[par][w] = inc;
        __syncthreads();                             // the other half is read before it is written again
        int off = D + inc - own;
#pragma unroll
        for (int i = 0; i < KM_BLOCK / 64; i++) {
            off += i < w ? part[par][i] : 0;
            D += part[par][i];
        }
#pragma unroll
        for (int j = 0; j < 8; j++)
            if (m[j] > 0) {
                if (off < KM_MAX_BINS) {
                    bv[off] = v + j;
                    bm[off] = m[j];
                    bl[off] = 0xFF;
                }
                off++;
            }
    }
    D = min(D, KM_MAX_BINS);
    if (tid < KM_MAX) {
        S2[tid] = 0;
        cnt[tid] = 0;
    }
    if (tid < 2) changed_s[tid] = 0;
    __syncthreads();
    // ---- start: centroid c is the distinct frequency of rank (2c + 1) D / (2k)
    if (tid < k) {
        const long long r = (2ll * tid + 1) * D / (2ll * k);
        S[tid] = bv[r];
        N[tid] = 1;
        Sd[tid] = (double)bv[r];
        Nd[tid] = 1.0;
    }
    int g = 0;                                       // lanes per bin: 2^g, every one with a cluster
    while (g < 6 && (2 << g) <= k && (D << (g + 1)) <= KM_BLOCK) g++;
    const int G = 1 << g, sub = tid & (G - 1);
    __syncthreads();
    int n_iter = 0;
    for (;;) {
        // ---- assignment: the nearest centroid, exactly; ties to the lower index
        for (int i0 = 0; i0 < D; i0 += KM_BLOCK >> g) {
            const int i = i0 + (tid >> g);
            const int ic = min(i, D - 1);
            int best = sub;
            if (EXACT64) {
                const double v = (double)bv[ic];
                double bd = fabs(v * Nd[sub] - Sd[sub]), bn = Nd[sub];
                for (int c = sub + G; c < k; c += G) {
                    const double nc = Nd[c], dc = fabs(v * nc - Sd[c]);
                    if (dc * bn < bd * nc) {
                        best = c;
                        bd = dc;
                        bn = nc;
                    }
                }
                for (int d = 1; d < G; d <<= 1) {
                    const double pd = __shfl_xor(bd, d, 64), pn = __shfl_xor(bn, d, 64);
                    const int pb = __shfl_xor(best, d, 64);
                    const double x = pd * bn, y = bd * pn;
                    if (x < y || (x == y && pb < best)) {
                        best = pb;
                        bd = pd;
                        bn = pn;
                    }
                }
            } else {
                const long long v = bv[ic];
                unsigned long long bd = absdiff(v * N[sub], S[sub]), bn = (unsigned long long)N[sub];
                for (int c = sub + G; c < k; c += G) {
                    const unsigned long long nc = (unsigned long long)N[c], dc = absdiff(v * N[c], S[c]);
                    if (less_prod(dc, bn, bd, nc)) {
                        best = c;
                        bd = dc;
                        bn = nc;
                    }
                }
                for (int d = 1; d < G; d <<= 1) {
                    const unsigned long long pd = __shfl_xor(bd, d, 64), pn = __shfl_xor(bn, d, 64);
                    const int pb = __shfl_xor(best, d, 64);
                    if (less_prod(pd, bn, bd, pn) || (pb < best && !less_prod(bd, pn, pd, bn))) {
                        best = pb;
                        bd = pd;
                        bn = pn;
                    }
                }
            }
            if (i < D && sub == 0) {
                if (bl[i] != best) {
                    changed_s[n_iter & 1] = 1;         // benign race: every writer stores 1
                    bl[i] = (uint8_t)best;
                }
                // frequencies sum to at most 2^24 and members to 2^22: both in one addition
                atomicAdd(&S2[best], ((unsigned long long)bv[i] * (unsigned long long)bm[i]) << 32 | (unsigned long long)bm[i]);
            }
        }
        __syncthreads();
        const int changed = changed_s[n_iter & 1];
        n_iter++;
        // ---- centroids: each non-empty cluster moves to its members' mean
        if (tid < k) {
            const unsigned long long s2 = S2[tid];
            const long long ns = (long long)(s2 >> 32), nn = (long long)(s2 & 0xFFFFFFFFull);
            if (changed) {
                cnt[tid] = nn;
                if (nn > 0) {
                    S[tid] = ns;
                    N[tid] = nn;
                    Sd[tid] = (double)ns;
                    Nd[tid] = (double)nn;
                }
            }
            S2[tid] = 0;
        }
        if (tid == 0) changed_s[n_iter & 1] = 0;       // the next assignment's flag
        __syncthreads();
        if (!changed || n_iter >= max_iter) break;
    }
    // ---- results: bin labels, ranks of the non-empty clusters
    for (int i = tid; i < D; i += KM_BLOCK) label[bv[i]] = bl[i];
    if (tid < KM_MAX) {
        const bool used = tid < k && cnt[tid] > 0;
        int r = 0;
        for (int d = 0; d < k; d++) {
            if (cnt[d] <= 0 || !used) continue;
            const long long a = S[d] * N[tid], b = S[tid] * N[d];
            r += a > b || (a == b && d < tid);
        }
        st->rank[tid] = used ? r : -1;
        const unsigned long long u = __ballot(used);
        if (tid == 0) {
            st->k_used = __popcll(u);
            st->n_iter = n_iter;
        }
    }
}

int grid_for(int64_t n, int block) { return (int)std::min<int64_t>(std::max<int64_t>((n + block - 1) / block, 1), 4096); }

// Scratch layout of one call: frequencies [n_skus], histogram [n_bins], the
// state (these start at zero), then bin labels [n_bins] (those of the bins in use
// are written before they are read); each part starts on 256 bytes.
struct KmLayout {
    size_t o_hist, o_state, o_label, bytes;
};

KmLayout km_layout(int32_t n_skus, int32_t n_bins)
{
    KmLayout L;
    L.o_hist = ((size_t)n_skus * 4 + 255) & ~(size_t)255;
    L.o_state = L.o_hist + (((size_t)n_bins * 4 + 255) & ~(size_t)255);
    L.o_label = L.o_state + ((sizeof(KmState) + 255) & ~(size_t)255);
    L.bytes = L.o_label + (((size_t)n_bins * 4 + 255) & ~(size_t)255);
    return L;
}

// Clears n 16-byte pieces: the scratch, inside the stream (a kernel rather
// than a memset, so that a call can sit in a captured graph).
__global__ void km_clear_kernel(uint4 *p, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = make_uint4(0u, 0u, 0u, 0u);
}

// Results of the allocation-free variant, written on the device.
__global__ void km_finish_kernel(const KmState *st, int32_t *k_used, int32_t *n_iter)
{
    if (threadIdx.x != 0) return;
    if (k_used) *k_used = st->err ? -1 : st->k_used;
    if (n_iter) *n_iter = st->n_iter;
}

// The launches of a call on its scratch.
hipError_t km_launch(char *buf, const KmLayout &L, const int32_t *skus, int64_t n_lines, int32_t n_skus, int32_t k,
                     int32_t max_iter, int32_t *category, hipStream_t s)
{
    int32_t *freq = (int32_t *)buf, *hist = (int32_t *)(buf + L.o_hist), *label = (int32_t *)(buf + L.o_label);
    KmState *st = (KmState *)(buf + L.o_state);
    const int32_t n_bins = (int32_t)n_lines + 1;
    const bool exact64 = (double)n_lines * (double)n_skus * (double)n_skus < 9007199254740992.0;
    hipLaunchKernelGGL(km_clear_kernel, dim3(grid_for((int64_t)L.o_label / 16, 256)), dim3(256), 0, s, (uint4 *)buf,
                       (int64_t)L.o_label / 16);
    hipLaunchKernelGGL(km_freq_kernel, dim3(std::min(grid_for(n_lines, 1024), 64)), dim3(1024), 0, s, skus, n_lines, n_skus,
                       freq, st);
    hipLaunchKernelGGL(km_hist_kernel, dim3(std::min(grid_for(n_skus, 1024), 128)), dim3(1024), 0, s, freq, n_skus, hist);
    if (exact64)
        hipLaunchKernelGGL(km_lloyd_kernel<true>, dim3(1), dim3(KM_BLOCK), 0, s, hist, n_bins, k, max_iter, label, st);
    else
        hipLaunchKernelGGL(km_lloyd_kernel<false>, dim3(1), dim3(KM_BLOCK), 0, s, hist, n_bins, k, max_iter, label, st);
    hipLaunchKernelGGL(km_label_kernel, dim3(grid_for(n_skus, 256)), dim3(256), 0, s, freq, n_skus, label, st, category);
    return hipGetLastError();
}

}  // namespace

// The allocation-free variant keeps its scratch in this array: one copy per
// device, held until the process ends.  In host code the name is only a
// stand-in: the device address comes from hipGetSymbolAddress, taken once
// per device with that device current, and is what the launches receive.
static __device__ __align__(256) unsigned char km_scratch[WO_KMEANS_NOALLOC_SCRATCH];

namespace {

constexpr int KM_MAX_DEVICES = 64;
std::mutex km_scratch_mu;
void *km_scratch_dev[KM_MAX_DEVICES];

wo_status km_scratch_address(void **out)
{
    int dev = 0;
    WO_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= KM_MAX_DEVICES) return wo_fail(WO_E_UNSUPPORTED, "device %d beyond %d", dev, KM_MAX_DEVICES);
    std::lock_guard<std::mutex> g(km_scratch_mu);
    if (!km_scratch_dev[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(km_scratch));
        if (e != hipSuccess || !p) {
            (void)hipGetLastError();
            return wo_fail(WO_E_DEVICE, "hipGetSymbolAddress of the K-means scratch failed: %s", hipGetErrorString(e));
        }
        km_scratch_dev[dev] = p;
    }
    *out = km_scratch_dev[dev];
    return WO_OK;
}

}  // namespace

extern "C" wo_status wo_kmeans_categories(const int32_t *d_order_skus, int64_t n_lines, int32_t n_skus, int32_t k,
                                          int32_t max_iter, int32_t *d_category, int32_t *k_used, int32_t *n_iter,
                                          void *stream)
{
    if (!d_order_skus || !d_category) return wo_fail(WO_E_INVAL, "NULL device buffer");
    if (n_lines < 1 || n_lines > WO_MAX_LINES)
        return wo_fail(WO_E_RANGE, "n_lines must be in 1 .. %d", WO_MAX_LINES);
    if (n_skus < 1 || n_skus > WO_MAX_LOCATIONS)
        return wo_fail(WO_E_RANGE, "n_skus must be in 1 .. %d", WO_MAX_LOCATIONS);
    if (k < 1 || k > KM_MAX) return wo_fail(WO_E_RANGE, "k must be in 1 .. %d", KM_MAX);
    if (max_iter < 1) return wo_fail(WO_E_INVAL, "max_iter must be >= 1");
    hipStream_t s = (hipStream_t)stream;
    const int32_t n_bins = (int32_t)n_lines + 1;      // a frequency is at most n_lines
    char *buf = nullptr;
    const KmLayout Ly = km_layout(n_skus, n_bins);
    if (wo_fault_injected()) return wo_fail(WO_E_NOMEM, "injected allocation failure");
    if (hipMalloc((void **)&buf, Ly.bytes) != hipSuccess) {
        (void)hipGetLastError();
        return wo_fail(WO_E_NOMEM, "hipMalloc(%zu) failed", Ly.bytes);
    }
    wo_status ret = WO_OK;
    int32_t h[3] = {0, 0, 0};                         // k_used, n_iter, err
    auto run = [&]() -> wo_status {
        WO_HIP(km_launch(buf, Ly, d_order_skus, n_lines, n_skus, k, max_iter, d_category, s));
        WO_HIP(hipMemcpyAsync(h, buf + Ly.o_state, sizeof h, hipMemcpyDeviceToHost, s));
        WO_HIP(hipStreamSynchronize(s));
        if (h[2]) return wo_fail(WO_E_INVAL, "an order line names a SKU outside 0 .. %d", n_skus - 1);
        return WO_OK;
    };
    ret = run();
    if (ret != WO_OK) (void)hipStreamSynchronize(s);
    (void)hipFree(buf);
    if (ret == WO_OK) {
        if (k_used) *k_used = h[0];
        if (n_iter) *n_iter = h[1];
    }
    return ret;
}

extern "C" wo_status wo_kmeans_categories_noalloc(const int32_t *d_order_skus, int64_t n_lines, int32_t n_skus,
                                                  int32_t k, int32_t max_iter, int32_t *d_category,
                                                  int32_t *d_k_used, int32_t *d_n_iter, void *stream)
{
    if (!d_order_skus || !d_category) return wo_fail(WO_E_INVAL, "NULL device buffer");
    if (n_lines < 1 || n_lines > WO_MAX_LINES)
        return wo_fail(WO_E_RANGE, "n_lines must be in 1 .. %d", WO_MAX_LINES);
    if (n_skus < 1 || n_skus > WO_MAX_LOCATIONS)
        return wo_fail(WO_E_RANGE, "n_skus must be in 1 .. %d", WO_MAX_LOCATIONS);
    if (k < 1 || k > KM_MAX) return wo_fail(WO_E_RANGE, "k must be in 1 .. %d", KM_MAX);
    if (max_iter < 1 || max_iter > WO_KMEANS_NOALLOC_MAX_ITER)
        return wo_fail(WO_E_RANGE, "max_iter must be in 1 .. %d", WO_KMEANS_NOALLOC_MAX_ITER);
    const int32_t n_bins = (int32_t)n_lines + 1;
    const KmLayout Ly = km_layout(n_skus, n_bins);
    if (Ly.bytes > (size_t)WO_KMEANS_NOALLOC_SCRATCH)
        return wo_fail(WO_E_RANGE, "%d SKUs and %lld lines need %zu bytes of scratch, more than the %d it has",
                       n_skus, (long long)n_lines, Ly.bytes, WO_KMEANS_NOALLOC_SCRATCH);
    void *base = nullptr;
    wo_status st0 = km_scratch_address(&base);
    if (st0) return st0;
    hipStream_t s = (hipStream_t)stream;
    char *buf = (char *)base;
    // the previous call's contents stay in the array: what starts at zero is
    // cleared first
    WO_HIP(km_launch(buf, Ly, d_order_skus, n_lines, n_skus, k, max_iter, d_category, s));
    const KmState *st = (const KmState *)(buf + Ly.o_state);
    hipLaunchKernelGGL(km_finish_kernel, dim3(1), dim3(64), 0, s, st, d_k_used, d_n_iter);
    WO_HIP(hipGetLastError());
    return WO_OK;
}
