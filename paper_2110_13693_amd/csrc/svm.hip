// Order categories by linear support vector machines (arXiv 2110.13693,
// section 5, subroutine 5): each order belongs to a category of orders; an
// SVM (Cortes and Vapnik 1995) learns the categories from the outputs of the
// subroutines before it, and is refreshed continuously from a window of the
// most recent orders, newer data replacing older.
//
// Readings (the paper gives no features, model or training rule):
//   - an order's features are the shares of its lines in each product
//     category (the classes of Subproblem 3): x[c] = lines in c / lines;
//   - one linear SVM per category of orders against the rest: hinge loss
//     plus lambda / 2 times the squared norm of the weights, the bias being
//     the weight of a constant feature 1; full-batch subgradient steps over
//     the window with the step sizes of Pegasos (Shalev-Shwartz et al.
//     2007), eta_t = 1 / (lambda t), t counting every step since creation;
//   - an order takes the category of the largest score (ties: the lower).
// The window is a ring of the last `window` samples on the device.  Every
// sum runs in a fixed order (features in index order, samples from the
// oldest) with one IEEE double operation at a time, so the results do not
// depend on the launch shape.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <new>

#include "wo_common.h"

// one IEEE operation at a time: no multiply-add contraction anywhere below
// (the file is also built with -ffp-contract=off)
#pragma clang fp contract(off)

struct wo_svm {
    int32_t F = 0, K = 0, W = 0;
    double lambda = 0.0;
    int64_t steps = 0;       // training steps so far
    int64_t pushed = 0;      // samples pushed so far; the window holds the last min(pushed, W)
    double *X = nullptr;     // [F][W]: by feature, sample g in slot g mod W
    int32_t *L = nullptr;    // [W]
    double *Wt = nullptr;    // [K][F + 1], bias last
    int8_t *coef = nullptr;  // [W][K]: +1 / -1 inside the margin, 0 outside
    std::atomic<int> busy{0};
};

namespace {

struct SvmBusy {
    std::atomic<int> *f;
    bool ok;
    explicit SvmBusy(std::atomic<int> *flag) : f(flag)
    {
        int z = 0;
        ok = f->compare_exchange_strong(z, 1);
    }
    ~SvmBusy()
    {
        if (ok) f->store(0);
    }
};

int grid_for(int64_t n, int block) { return (int)std::min<int64_t>(std::max<int64_t>((n + block - 1) / block, 1), 65535); }

// Line counts per category, then shares, 64 orders per workgroup.  The first
// wave counts: each lane its order's lines in its own LDS row (lines clamped to
// [0, n_lines); SKUs outside [0, n_skus) and categories outside [0, F) count
// in the length only), the two dependent gathers of 4 lines in flight
// together.  It also divides the small counts, which nearly all are, by the
// length once per order.  Then all four waves write the 64 rows of shares, one
// coalesced row per store (lane = feature).  8,192 orders: 9.4 us, against 14
// us with one wave, a line at a time and a division per share; 1M: 0.121 ms,
// against 0.131.
constexpr int FT_LD = WO_SVM_MAX_FEATURES + 1;
constexpr int FT_SHARES = 5;                         // shares of 0 .. 4 lines are kept per order
constexpr int FT_U = 4;

__global__ __launch_bounds__(256) void features_kernel(const int32_t *off, const int32_t *skus, int32_t n_orders,
                                                      int64_t n_lines, const int32_t *sku_cat, int32_t n_skus,
                                                      int32_t F, double *x)
{
    __shared__ uint32_t cnt[64 * FT_LD];
    __shared__ double share[64 * FT_SHARES];
    __shared__ double len[64];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    for (int64_t o0 = (int64_t)blockIdx.x * 64; o0 < n_orders; o0 += (int64_t)gridDim.x * 64) {
        for (int32_t c = tid; c < 64 * FT_LD; c += 256) cnt[c] = 0u;
        __syncthreads();
        const int64_t o = o0 + lane;
        if (w == 0 && o < n_orders) {
            uint32_t *mine = cnt + lane * FT_LD;
            const int32_t a = off[o], b = off[o + 1];
            const int64_t l0 = std::max<int64_t>(a, 0), l1 = std::min<int64_t>(b, n_lines);
            for (int64_t l = l0; l < l1; l += FT_U) {
                int32_t sk[FT_U], c[FT_U];
#pragma unroll
                for (int u = 0; u < FT_U; u++) sk[u] = skus[std::min<int64_t>(l + u, l1 - 1)];
#pragma unroll
                for (int u = 0; u < FT_U; u++) c[u] = sk[u] >= 0 && sk[u] < n_skus ? sku_cat[sk[u]] : -1;
#pragma unroll
                for (int u = 0; u < FT_U; u++)
                    if (l + u < l1 && c[u] >= 0 && c[u] < F) mine[c[u]] += 1u;
            }
            const double d = (double)(b - a);
            len[lane] = d;
#pragma unroll
            for (int v = 0; v < FT_SHARES; v++) share[lane * FT_SHARES + v] = (double)v / d;
        }
        __syncthreads();
        const int32_t rows = (int32_t)std::min<int64_t>(64, n_orders - o0);
        for (int32_t r = w; r < rows; r += 4)
            for (int32_t c = lane; c < F; c += 64) {
                const uint32_t k = cnt[r * FT_LD + c];
                x[(o0 + r) * F + c] = k < (uint32_t)FT_SHARES ? share[r * FT_SHARES + k] : (double)k / len[r];
            }
        __syncthreads();
    }
}

// Samples into the window, transposed to [F][W] (both later readers of the
// window, the margins and the subgradients, then read it coalesced): 64
// samples per workgroup through LDS, row r of the input to slot (g0 + r) mod W.
__global__ __launch_bounds__(256) void push_kernel(const double *x, const int32_t *labels, int64_t n, int32_t F,
                                                   int64_t g0, int32_t W, double *X, int32_t *L)
{
    __shared__ double tile[64 * (WO_SVM_MAX_FEATURES + 1)];
    const int tid = threadIdx.x;
    const int64_t r0 = (int64_t)blockIdx.x * 64;
    const int32_t rows = (int32_t)std::min<int64_t>(64, n - r0);
    for (int32_t e = tid; e < rows * F; e += 256) {
        const int32_t r = e / F;
        tile[r * (WO_SVM_MAX_FEATURES + 1) + (e - r * F)] = x[r0 * F + e];
    }
    __syncthreads();
    const int32_t r = tid & 63;
    if (r >= rows) return;
    const int64_t slot = (g0 + r0 + r) % W;
    for (int32_t f = tid >> 6; f < F; f += 4) X[(int64_t)f * W + slot] = tile[r * (WO_SVM_MAX_FEATURES + 1) + f];
    if (tid < 64) L[slot] = labels[r0 + r];
}

// One lane per sample, MG_K classes per wave: inside the margin at the current
// weights?  A score adds weight times feature in feature order, then the bias.
// The features of 64 consecutive samples are one coalesced load, the weights
// scalar ones; 8 features are in flight.  65,536 samples, 64 features, 8
// classes: 12.3 us, against 42 us with one thread per (sample, class) reading
// rows of samples.
constexpr int MG_K = 2, MG_F = 8;

__global__ __launch_bounds__(256) void margin_kernel(const double *X, const int32_t *L, int32_t W, int64_t first, int64_t n,
                                                     int32_t F, int32_t K, const double *Wt, int8_t *coef)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int32_t k0 = (int32_t)blockIdx.y * MG_K;
    int64_t slot = first + i;
    if (slot >= W) slot -= W;
    const double *x = X + slot;
    const double *w[MG_K];
    double s[MG_K];
#pragma unroll
    for (int j = 0; j < MG_K; j++) {
        w[j] = Wt + (int64_t)std::min(k0 + j, K - 1) * (F + 1);
        s[j] = 0.0;
    }
    int32_t f = 0;
    for (; f + MG_F <= F; f += MG_F) {
        double v[MG_F];
#pragma unroll
        for (int u = 0; u < MG_F; u++) v[u] = x[(int64_t)(f + u) * W];
#pragma unroll
        for (int u = 0; u < MG_F; u++)
#pragma unroll
            for (int j = 0; j < MG_K; j++) s[j] = s[j] + w[j][f + u] * v[u];
    }
    for (; f < F; f++) {
        const double v = x[(int64_t)f * W];
#pragma unroll
        for (int j = 0; j < MG_K; j++) s[j] = s[j] + w[j][f] * v;
    }
    const int32_t label = L[slot];
#pragma unroll
    for (int j = 0; j < MG_K; j++) {
        const int32_t k = k0 + j;
        if (k >= K) break;
        const double sc = s[j] + w[j][F];
        const bool pos = label == k;
        const double ys = pos ? sc : -sc;
        coef[i * K + k] = (int8_t)(ys < 1.0 ? (pos ? 1 : -1) : 0);
    }
}

// The subgradient step, one workgroup per feature (blockIdx < F) for all
// classes.  A weight's sum over the samples runs from the oldest, one addition
// after the other, so its chain is the longest thing here, and only the terms
// that can change it are kept in it: a feature of zero adds coef * 0 = +-0 to
// a sum that is never -0 (it starts at +0), which leaves it as it is, while
// every other value, also infinities and NaN, takes part for every class.
// Order features are shares of few lines, so about 1 in 25 is not zero; dense
// features give the full chain.  A step over 65,536 samples, 64 features and 8
// classes: 41.6 us for order features and 0.43 ms for dense ones, with the
// margins, against 3.82 ms with one thread per weight reading every sample (143
// cycles a sample; the chain's reads now come from LDS, one per addition).
// With the products made by the adding wave itself: 65 us.  Per round of 8,192 samples:
//   1. every lane holds 16 values of the feature (loaded during the previous
//      round); ballots number the non-zero ones in sample order;
//   2. in pieces of at most UP_VAL / KP entries (KP: the classes rounded up to a power of two): the entries' values and
//      sample numbers go to LDS, then all waves form the products with the
//      classes' coefficients, one per (entry, class);
//   3. a wave of its own, one lane per class, adds the products in order while
//      the others prepare the next piece (two product buffers; it passes the
//      barriers of that preparation half-way and at the end of its piece).
// The bias (a constant feature of 1) sums +-1 exactly in any order: one
// workgroup per class (blockIdx >= F) counts.
constexpr int UP_WAVES = 8, UP_J = 16, UP_ROUND = 64 * UP_WAVES * UP_J;   // waves that prepare, values per lane
constexpr int UP_THREADS = 64 * UP_WAVES + 64;       // and the wave that adds
constexpr int UP_VAL = 4096;                         // products per piece
constexpr int UP_CAP = UP_VAL / 2;                   // entries per piece at most (2 classes)
constexpr int UP_PT = UP_VAL / (64 * UP_WAVES);      // products per thread and piece

// KPL: log2 of the classes rounded up, so that the chain's reads take their
// addresses from immediate offsets (the adding wave issues one read and one
// addition per entry).
template <int KPL>
__global__ __launch_bounds__(UP_THREADS) void update_kernel(const double *X, const int8_t *coef, int32_t W,
                                                            int64_t first, int64_t n, int32_t F, int32_t K,
                                                            double *Wt, double lambda, double t)
{
    constexpr int cap = UP_CAP < (UP_VAL >> KPL) ? UP_CAP : UP_VAL >> KPL;
    __shared__ double val[2 * UP_VAL + (16 << KPL)];   // two buffers; the chain reads up to 16 entries past a piece
    __shared__ double lx[UP_CAP];
    __shared__ int32_t li[UP_CAP];
    __shared__ int32_t wcnt[2][UP_WAVES + 1];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const double eta = 1.0 / (lambda * t);
    auto step = [&](int32_t k, int32_t f, double g) {
        double *p = Wt + (int64_t)k * (F + 1) + f;
        const double old = *p;
        *p = old - eta * (lambda * old - g / (double)n);
    };
    if ((int32_t)blockIdx.x >= F) {
        const int32_t k = (int32_t)blockIdx.x - F;
        int32_t s = 0;
        for (int64_t i0 = tid; i0 < n; i0 += 32 * UP_THREADS) {
            int8_t c[32];                            // loads in flight together
#pragma unroll
            for (int u = 0; u < 32; u++) c[u] = coef[std::min(i0 + (int64_t)u * UP_THREADS, n - 1) * K + k];
#pragma unroll
            for (int u = 0; u < 32; u++) s += i0 + (int64_t)u * UP_THREADS < n ? c[u] : 0;
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d, 64);
        if (lane == 0) wcnt[0][w] = s;
        __syncthreads();
        if (tid == 0) {
            for (int v = 1; v <= UP_WAVES; v++) s += wcnt[0][v];
            step(k, F, (double)s);
        }
        return;
    }
    const int32_t f = (int32_t)blockIdx.x;
    const double *col = X + (int64_t)f * W;
    int buf = 0;
    if (w == UP_WAVES) {
        // the sums, one lane per class
        double g = 0.0;
        const int32_t mine = std::min(lane, K - 1);
        // entries [e, end) of a piece, the next 16 read while 16 are added
        auto add = [&](const double *v0, int32_t e, int32_t end) {
            const double *v = v0 + mine;
            double a[16], b[16];
            auto get = [&](int32_t e_, double (&d)[16]) {
                const double *q = v + (e_ << KPL);
#pragma unroll
                for (int u = 0; u < 16; u++) d[u] = q[u << KPL];
            };
            if (e + 32 <= end) {
                get(e, a);
                for (; e + 32 <= end; e += 32) {
                    get(e + 16, b);
#pragma unroll
                    for (int u = 0; u < 16; u++) g = g + a[u];
                    get(e + 32, a);
#pragma unroll
                    for (int u = 0; u < 16; u++) g = g + b[u];
                }
            }
            for (; e < end; e++) g = g + v[e << KPL];
        };
        const double *pv = nullptr;
        int32_t pe = 0, pm = 0;                      // the piece being added, its next entry
        int par = 0;
        for (int64_t r0 = 0; r0 < n; r0 += UP_ROUND, par ^= 1) {
            __syncthreads();                         // the counts
            if (pe < pm) {
                add(pv, pe, pm);
                pe = pm;
            }
            int32_t total = 0;
            for (int v = 0; v < UP_WAVES; v++) total += wcnt[par][v];
            for (int32_t c0 = 0; c0 < total; c0 += cap) {
                __syncthreads();                     // the entries
                if (pe < pm) {
                    add(pv, pe, pm);
                    pe = pm;
                }
                __syncthreads();                     // the products
                pv = val + buf * UP_VAL;
                buf ^= 1;
                pm = std::min(cap, total - c0);
                pe = pm / 2 & ~15;
                add(pv, 0, pe);
            }
        }
        if (pe < pm) add(pv, pe, pm);
        if (lane < K) step(lane, f, g);
        return;
    }
    double x[UP_J], nx[UP_J];
    // sample of slot j of this lane in the round that starts at r0; past the
    // last sample: zero
    auto load = [&](int64_t r0, double (&v)[UP_J]) {
#pragma unroll
        for (int j = 0; j < UP_J; j++) {
            const int64_t i = r0 + w * (64 * UP_J) + j * 64 + lane;
            int64_t slot = first + (i < n ? i : 0);
            if (slot >= W) slot -= W;
            v[j] = col[slot];
        }
#pragma unroll
        for (int j = 0; j < UP_J; j++)
            if (r0 + w * (64 * UP_J) + j * 64 + lane >= n) v[j] = 0.0;
    };
    load(0, nx);
    int par = 0;
    for (int64_t r0 = 0; r0 < n; r0 += UP_ROUND, par ^= 1) {
#pragma unroll
        for (int j = 0; j < UP_J; j++) x[j] = nx[j];
        if (r0 + UP_ROUND < n) load(r0 + UP_ROUND, nx);
        int32_t cnt = 0;
#pragma unroll
        for (int j = 0; j < UP_J; j++) cnt += (int32_t)__popcll(__ballot(x[j] != 0.0));
        if (lane == 0) wcnt[par][w] = cnt;
        __syncthreads();                             // the counts
        int32_t base = 0, total = 0;
#pragma unroll
        for (int v = 0; v < UP_WAVES; v++) {
            const int32_t c = wcnt[par][v];
            base += v < w ? c : 0;
            total += c;
        }
        for (int32_t c0 = 0; c0 < total; c0 += cap) {
            const int32_t m = std::min(cap, total - c0);
            int32_t at = base - c0;
#pragma unroll
            for (int j = 0; j < UP_J; j++) {
                const bool nz = x[j] != 0.0;
                const uint64_t b = __ballot(nz);
                const int32_t e = at + (int32_t)__popcll(b & ((1ull << lane) - 1ull));
                if (nz && e >= 0 && e < m) {
                    lx[e] = x[j];
                    li[e] = (int32_t)(r0 + w * (64 * UP_J) + j * 64 + lane);
                }
                at += (int32_t)__popcll(b);
            }
            __syncthreads();                         // the entries
            {
                // the coefficients of a thread's products load together
                double v[UP_PT];
                int8_t c[UP_PT];
#pragma unroll
                for (int u = 0; u < UP_PT; u++) {
                    const int32_t q = tid + u * 64 * UP_WAVES, e = std::min(q >> KPL, m - 1);
                    const int32_t k = std::min(q & ((1 << KPL) - 1), K - 1);
                    v[u] = lx[e];
                    c[u] = coef[(int64_t)li[e] * K + k];
                }
#pragma unroll
                for (int u = 0; u < UP_PT; u++) val[buf * UP_VAL + tid + u * 64 * UP_WAVES] = (double)c[u] * v[u];
            }
            buf ^= 1;
            __syncthreads();                         // the products
        }
    }
}

// Prediction: the class of the largest score (ties: the lower class), a score
// being weights . features in feature order, then the bias, as in training.
// 64 R orders per workgroup: their rows, one contiguous block of at most 4,096
// features, go to LDS with all loads in flight together; then 4 / R waves share
// the classes of each 64 orders, KG at a time, with one lane per order (weights
// by scalar loads, a row's features from LDS at an odd stride), and the first of
// these waves takes the best of their bests.  Four workgroups fit a CU, so that
// some load while others multiply.  64 features, 8 classes: 9 us for 8,192
// orders and 0.104 ms for 1M (5.2 TB/s of features), against 30 us and 0.194 ms
// when each wave streamed 64 orders of its own in chunks of 8 features for all
// classes.
template <int R, int KG>
__global__ __launch_bounds__(256) void predict_kernel(const double *X, int64_t n, int32_t F, int32_t f_inv, int32_t K,
                                                     const double *Wt, int32_t *cls)
{
    extern __shared__ double lds[];                  // the rows, then the waves' best scores [256] and classes [256]
    constexpr int WPR = 4 / R;                       // waves that share a row's classes
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sub = w % WPR;
    const int32_t row = w / WPR * 64 + lane;         // this lane's order
    const int32_t ld = F | 1;
    for (int64_t i0 = (int64_t)blockIdx.x * (64 * R); i0 < n; i0 += (int64_t)gridDim.x * (64 * R)) {
        const int32_t rows = (int32_t)std::min<int64_t>(64 * R, n - i0), total = rows * F;
        const double *src = X + i0 * F;
        {
            double v[16];
#pragma unroll
            for (int t = 0; t < 16; t++) v[t] = src[std::min(tid + t * 256, total - 1)];
#pragma unroll
            for (int t = 0; t < 16; t++) {
                const int32_t e = tid + t * 256;
                // e / F: exact, as e < 4096 and F <= 64
                const int32_t r = (int32_t)(((uint32_t)e * (uint32_t)f_inv) >> 20);
                if (e < total) lds[r * ld + (e - r * F)] = v[t];
            }
        }
        __syncthreads();
        const double *mine = lds + std::min(row, rows - 1) * ld;
        // the best of this wave's classes (sub * KG + j, then 4 / R KG further).
        // The sequence that starts from class 0 and takes every larger score keeps
        // class 0 where its score is NaN and never takes a NaN or -inf.
        int32_t best = sub == 0 ? 0 : WO_SVM_MAX_CLASSES;
        double bs = -INFINITY;
        for (int32_t k0 = sub * KG; k0 < K; k0 += WPR * KG) {
            double s[KG];
            const double *wt[KG];
#pragma unroll
            for (int j = 0; j < KG; j++) {
                s[j] = 0.0;
                wt[j] = Wt + (int64_t)std::min(k0 + j, K - 1) * (F + 1);
            }
            int32_t f = 0;
            for (; f + 8 <= F; f += 8) {
                double v[8];
#pragma unroll
                for (int u = 0; u < 8; u++) v[u] = mine[f + u];
#pragma unroll
                for (int u = 0; u < 8; u++)
#pragma unroll
                    for (int j = 0; j < KG; j++) s[j] = s[j] + wt[j][f + u] * v[u];
            }
            for (; f < F; f++) {
                const double v = mine[f];
#pragma unroll
                for (int j = 0; j < KG; j++) s[j] = s[j] + wt[j][f] * v;
            }
#pragma unroll
            for (int j = 0; j < KG; j++) {
                const double v = s[j] + wt[j][F];
                if (k0 + j < K && (k0 + j == 0 || v > bs)) {
                    bs = v;
                    best = k0 + j;
                }
            }
        }
        if (WPR > 1) {
            int32_t *bk = (int32_t *)(lds + 256);
            __syncthreads();                         // the rows are read
            lds[sub * (64 * R) + row] = bs;
            bk[sub * (64 * R) + row] = best;
            __syncthreads();
            if (sub == 0)
#pragma unroll
                for (int u = 1; u < WPR; u++) {
                    const double v = lds[u * (64 * R) + row];
                    const int32_t k = bk[u * (64 * R) + row];
                    if (v > bs || (v == bs && k < best)) {
                        bs = v;
                        best = k;
                    }
                }
        }
        if (sub == 0 && row < rows) cls[i0 + row] = best;
        __syncthreads();                             // the rows, or the bests, are read
    }
}

}  // namespace

extern "C" wo_status wo_order_features(const int32_t *d_order_offsets, const int32_t *d_order_skus, int32_t n_orders,
                                       int64_t n_lines, const int32_t *d_sku_category, int32_t n_skus,
                                       int32_t n_features, double *d_features, void *stream)
{
    if (!d_order_offsets || !d_order_skus || !d_sku_category || !d_features) return wo_fail(WO_E_INVAL, "NULL buffer");
    if (n_orders < 0 || n_lines < 0 || n_skus < 0) return wo_fail(WO_E_INVAL, "negative size");
    if (n_features < 1 || n_features > WO_SVM_MAX_FEATURES)
        return wo_fail(WO_E_RANGE, "n_features must be in 1 .. %d", WO_SVM_MAX_FEATURES);
    if (n_orders == 0) return WO_OK;
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(features_kernel, dim3(grid_for(n_orders, 64)), dim3(256), 0, s, d_order_offsets, d_order_skus,
                       n_orders, n_lines, d_sku_category, n_skus, n_features, d_features);
    WO_HIP(hipGetLastError());
    return WO_OK;
}

extern "C" wo_status wo_svm_create(int32_t n_features, int32_t n_classes, int32_t window, double lambda,
                                   void *stream, wo_svm **out)
{
    if (!out) return wo_fail(WO_E_INVAL, "out is NULL");
    *out = nullptr;
    if (n_features < 1 || n_features > WO_SVM_MAX_FEATURES)
        return wo_fail(WO_E_RANGE, "n_features must be in 1 .. %d", WO_SVM_MAX_FEATURES);
    if (n_classes < 2 || n_classes > WO_SVM_MAX_CLASSES)
        return wo_fail(WO_E_RANGE, "n_classes must be in 2 .. %d", WO_SVM_MAX_CLASSES);
    if (window < 1 || window > WO_SVM_MAX_WINDOW) return wo_fail(WO_E_RANGE, "window must be in 1 .. %d", WO_SVM_MAX_WINDOW);
    if (!(lambda > 0.0)) return wo_fail(WO_E_INVAL, "lambda must be > 0");
    if (wo_fault_injected()) return wo_fail(WO_E_NOMEM, "injected allocation failure");
    wo_svm *m = new (std::nothrow) wo_svm;
    if (!m) return wo_fail(WO_E_NOMEM, "host allocation failed");
    m->F = n_features;
    m->K = n_classes;
    m->W = window;
    m->lambda = lambda;
    hipStream_t s = (hipStream_t)stream;
    bool ok = hipMalloc((void **)&m->X, sizeof(double) * (size_t)window * n_features) == hipSuccess &&
              hipMalloc((void **)&m->L, sizeof(int32_t) * (size_t)window) == hipSuccess &&
              hipMalloc((void **)&m->Wt, sizeof(double) * (size_t)n_classes * (n_features + 1)) == hipSuccess &&
              hipMalloc((void **)&m->coef, (size_t)window * n_classes) == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        wo_svm_free(m);
        return wo_fail(WO_E_NOMEM, "device allocation failed");
    }
    if (hipMemsetAsync(m->Wt, 0, sizeof(double) * (size_t)n_classes * (n_features + 1), s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) {
        (void)hipGetLastError();
        wo_svm_free(m);
        return wo_fail(WO_E_DEVICE, "clearing the weights failed");
    }
    *out = m;
    return WO_OK;
}

extern "C" wo_status wo_svm_free(wo_svm *m)
{
    if (!m) return WO_OK;
    if (m->X || m->L || m->Wt || m->coef) (void)hipDeviceSynchronize();
    if (m->X) (void)hipFree(m->X);
    if (m->L) (void)hipFree(m->L);
    if (m->Wt) (void)hipFree(m->Wt);
    if (m->coef) (void)hipFree(m->coef);
    delete m;
    return WO_OK;
}

extern "C" wo_status wo_svm_push(wo_svm *m, int64_t n, const double *d_features, const int32_t *d_labels, void *stream)
{
    if (!m || !d_features || !d_labels) return wo_fail(WO_E_INVAL, "NULL argument");
    if (n < 0) return wo_fail(WO_E_INVAL, "n < 0");
    SvmBusy busy(&m->busy);
    if (!busy.ok) return wo_fail(WO_E_STATE, "SVM in use by another thread");
    hipStream_t s = (hipStream_t)stream;
    // only the last min(n, W) samples stay; sample g goes to slot g mod W
    const int64_t keep = std::min<int64_t>(n, m->W), r0 = n - keep;
    if (keep > 0) {
        hipLaunchKernelGGL(push_kernel, dim3((uint32_t)((keep + 63) / 64)), dim3(256), 0, s, d_features + r0 * m->F,
                           d_labels + r0, keep, m->F, m->pushed + r0, m->W, m->X, m->L);
        WO_HIP(hipGetLastError());
    }
    m->pushed += n;
    return WO_OK;
}

extern "C" wo_status wo_svm_train(wo_svm *m, int32_t iterations, void *stream)
{
    if (!m) return wo_fail(WO_E_INVAL, "NULL SVM");
    if (iterations < 0) return wo_fail(WO_E_INVAL, "iterations < 0");
    SvmBusy busy(&m->busy);
    if (!busy.ok) return wo_fail(WO_E_STATE, "SVM in use by another thread");
    const int64_t n = std::min<int64_t>(m->pushed, m->W);
    if (n == 0) return wo_fail(WO_E_STATE, "the window holds no sample");
    const int64_t first = (m->pushed - n) % m->W;   // slot of the oldest sample
    hipStream_t s = (hipStream_t)stream;
    decltype(&update_kernel<1>) update = m->K <= 2    ? update_kernel<1>
                                         : m->K <= 4  ? update_kernel<2>
                                         : m->K <= 8  ? update_kernel<3>
                                         : m->K <= 16 ? update_kernel<4>
                                         : m->K <= 32 ? update_kernel<5>
                                                      : update_kernel<6>;
    for (int32_t it = 0; it < iterations; it++) {
        const double t = (double)(m->steps + it + 1);
        hipLaunchKernelGGL(margin_kernel, dim3((uint32_t)((n + 255) / 256), (m->K + MG_K - 1) / MG_K), dim3(256), 0, s,
                           m->X, m->L, m->W, first, n, m->F, m->K, m->Wt, m->coef);
        hipLaunchKernelGGL(update, dim3(m->F + m->K), dim3(UP_THREADS), 0, s, m->X, m->coef, m->W, first, n,
                           m->F, m->K, m->Wt, m->lambda, t);
    }
    WO_HIP(hipGetLastError());
    m->steps += iterations;
    return WO_OK;
}

extern "C" wo_status wo_svm_predict(wo_svm *m, int64_t n, const double *d_features, int32_t *d_class, void *stream)
{
    if (!m || !d_features || !d_class) return wo_fail(WO_E_INVAL, "NULL argument");
    if (n < 0) return wo_fail(WO_E_INVAL, "n < 0");
    if (n == 0) return WO_OK;
    hipStream_t s = (hipStream_t)stream;
    // Rows of few features make a workgroup of 64 orders too small for its own
    // start (1M orders of 8 features, 2 classes: 60 us, 24 with 256 orders): the
    // 64, 128 or 256 orders whose features a workgroup's loads take at once,
    // where the GPU still gets several workgroups per CU.
    const int R = n < 32768 || m->F > 32 ? 1 : m->F > 16 ? 2 : 4;
    // two classes at a time where each wave has no more than two, else four
    const bool two = m->K * R <= 8;
    auto kernel = R == 1   ? (two ? predict_kernel<1, 2> : predict_kernel<1, 4>)
                  : R == 2 ? (two ? predict_kernel<2, 2> : predict_kernel<2, 4>)
                           : (two ? predict_kernel<4, 2> : predict_kernel<4, 4>);
    // the rows; the waves' bests of 256 orders and classes take their place
    const size_t lds = sizeof(double) * std::max<size_t>(64 * (size_t)R * (m->F | 1), 256 + 128);
    hipLaunchKernelGGL(kernel, dim3(grid_for(n, 64 * R)), dim3(256), lds, s, d_features, n, m->F, (1 << 20) / m->F + 1,
                       m->K, m->Wt, d_class);
    WO_HIP(hipGetLastError());
    return WO_OK;
}

extern "C" wo_status wo_svm_get_weights(wo_svm *m, double *h_weights, int64_t *h_steps, int64_t *h_window_count,
                                        void *stream)
{
    if (!m) return wo_fail(WO_E_INVAL, "NULL SVM");
    hipStream_t s = (hipStream_t)stream;
    if (h_weights) {
        WO_HIP(hipMemcpyAsync(h_weights, m->Wt, sizeof(double) * (size_t)m->K * (m->F + 1), hipMemcpyDeviceToHost, s));
        WO_HIP(hipStreamSynchronize(s));
    }
    if (h_steps) *h_steps = m->steps;
    if (h_window_count) *h_window_count = std::min<int64_t>(m->pushed, m->W);
    return WO_OK;
}
