// Aisle width design (arXiv 2110.13693, section 5, Subproblem 1, Eq. (1)):
// maximise the share of the floor the racks take, A_ind / A_max, subject to
// k * delta - a <= 0, where a is the width between racks and delta the
// picking frequency that Subproblem 2 returns for the picking plan
// (delta = f(d), Eq. (2)).  The two subproblems couple through a and delta:
// a narrower aisle shortens every route, raises delta and so the width the
// flow needs.
//
// Geometry of the single block: every aisle is a corridor of width a with a
// rack face of depth r on each side (racks of neighbouring aisles stand back
// to back), so aisles are a + 2r apart centre to centre; racks are L = S p
// long; a cross aisle of width c runs along the front and the back.  Then
//     A_ind / A_max = 2 r L / ((a + 2 r) (L + 2 c)),
// which falls with a, so the optimum is the narrowest feasible width.  delta
// falls as a grows (routes lengthen), so k delta(a) <= a holds from one width
// on: the optimum is the smallest width in [a_min, a_max] that meets it.
//
// Widths are whole decimetres, like every distance here.  Tours do not depend on
// the spacing, and under every route but the optimal one a tour's cost does only
// through 2 spacing a_max, the way to its farthest aisle and back: the plan's
// distance is affine in the spacing, exactly, so two widths are evaluated and
// the others follow in 64-bit integers (saturated as the evaluator does; it
// grows with the spacing, so past a saturated width every one is).  The optimal
// route is evaluated at every width.  (400 widths at the paper scale: 48 us, 114
// when each was evaluated, in five buffers.)  Either way it is one launch of the exact
// evaluator, each copy of the plan with its own aisle spacing; the host then
// takes the first width that meets the constraint, deciding it in IEEE double
// from the integer distance.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "wo_common.h"
#include "wo_internal.h"

namespace {

// The plan once per width: zone rows, sequence rows back to back (n ids each)
// and the widths' spacings.
__global__ void replicate_kernel(uint8_t *zone, uint16_t *seq, int32_t *spacing, const uint8_t *zone0,
                                 const uint16_t *seq0, int64_t n, int32_t spacing0)
{
    const int64_t j = blockIdx.y;
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) seq[j * n + i] = seq0[i];
    if (i < 64) zone[j * 64 + i] = zone0[i];
    if (i == 0) spacing[j] = spacing0 + (int32_t)j;
}

}  // namespace

using namespace wo;

extern "C" wo_status wo_aisle_width(wo_wh *wh, int32_t inst, const uint8_t *d_zone_of, const uint16_t *d_order_seq,
                                    const wo_aisle_params *prm, int32_t *h_dist, void *stream, wo_aisle_result *out)
{
    if (!wh || !d_zone_of || !d_order_seq || !prm || !out) return wo_fail(WO_E_INVAL, "NULL argument");
    if (inst < 0 || inst >= instance_count(wh)) return wo_fail(WO_E_RANGE, "instance %d out of range", inst);
    const wo_aisle_params p = *prm;
    if (p.rack_depth_dm < 1 || p.cross_aisle_dm < 0 || p.min_width_dm < 1 || p.max_width_dm < p.min_width_dm ||
        !(p.k_dm >= 0.0))
        return wo_fail(WO_E_INVAL, "need rack depth >= 1, cross aisle >= 0, 1 <= min width <= max width, k >= 0");
    const int64_t G = (int64_t)p.max_width_dm - p.min_width_dm + 1;
    if (G > WO_AISLE_MAX_WIDTHS)
        return wo_fail(WO_E_RANGE, "%lld widths in the range, at most %d", (long long)G, WO_AISLE_MAX_WIDTHS);
    const InstDev &I = instance_dev(wh, inst);
    const int64_t w_max = (int64_t)p.max_width_dm + 2ll * p.rack_depth_dm;
    if (w_max >= (1ll << 24)) return wo_fail(WO_E_RANGE, "aisle spacing of %lld dm too large", (long long)w_max);
    if (I.route == WO_ROUTE_OPTIMAL &&
        4ll * w_max * (I.n_aisles + 2) + 4ll * I.L * (I.n_aisles + 1) >= (1ll << 30))
        return wo_fail(WO_E_RANGE, "the optimal route's 32-bit distances do not reach a spacing of %lld dm",
                       (long long)w_max);
    hipStream_t s = (hipStream_t)stream;
    const int64_t n = I.n_orders;
    // widths evaluated, in the order of the range; the others follow
    const int64_t E = I.route == WO_ROUTE_OPTIMAL ? G : std::min<int64_t>(G, 2);
    std::vector<int32_t> dist((size_t)G);
    if (wo_fault_injected()) return wo_fail(WO_E_NOMEM, "injected allocation failure");
    // distances, spacings, zone rows, sequence rows
    const size_t o_sp = ((size_t)E * 4 + 255) & ~(size_t)255, o_z = 2 * o_sp, o_q = o_z + (size_t)E * 64;
    unsigned char *buf = nullptr;
    if (hipMalloc((void **)&buf, o_q + (size_t)E * n * 2) != hipSuccess) {
        (void)hipGetLastError();
        return wo_fail(WO_E_NOMEM, "device allocation for %lld widths failed", (long long)G);
    }
    int32_t *dd = (int32_t *)buf, *dsp = (int32_t *)(buf + o_sp);
    uint8_t *dz = buf + o_z;
    uint16_t *dq = (uint16_t *)(buf + o_q);
    auto run = [&]() -> wo_status {
        hipLaunchKernelGGL(replicate_kernel, dim3((unsigned)((std::max<int64_t>(n, 64) + 255) / 256), (unsigned)E), dim3(256),
                           0, s, dz, dq, dsp, d_zone_of, d_order_seq, n, p.min_width_dm + 2 * p.rack_depth_dm);
        WO_HIP(hipGetLastError());
        wo_status r = eval_instance(wh, inst, E, dz, dq, dd, nullptr, s, dsp);
        if (r) return r;
        WO_HIP(hipMemcpyAsync(dist.data(), dd, (size_t)E * 4, hipMemcpyDeviceToHost, s));
        WO_HIP(hipStreamSynchronize(s));
        return WO_OK;
    };
    const wo_status st = run();
    if (st) (void)hipStreamSynchronize(s);
    (void)hipFree(buf);
    if (st) return st;
    if (E < G) {
        const int64_t d0 = dist[0], slope = (int64_t)dist[1] - d0;
        for (int64_t j = 2; j < G; j++)
            dist[(size_t)j] = dist[1] == INT32_MAX ? INT32_MAX : (int32_t)std::min<int64_t>(d0 + j * slope, INT32_MAX);
    }
    if (h_dist) std::copy(dist.begin(), dist.end(), h_dist);
    // delta(a) = n_orders * window / (D / walk + t_item * items), one
    // operation per statement (no contraction), as the rate of the evaluator
    auto delta_of = [&](int32_t D) {
        const double q = (double)D / I.walk;
        const double u = I.t_item * (double)I.n_lines;
        const double T = q + u;
        const double num = (double)I.n_orders * I.window;
        return num / T;
    };
    int64_t pick = G - 1;
    bool feasible = false;
    for (int64_t j = 0; j < G; j++) {
        const double need = p.k_dm * delta_of(dist[(size_t)j]);
        if (need <= (double)(p.min_width_dm + j)) {
            pick = j;
            feasible = true;
            break;
        }
    }
    const int32_t a = p.min_width_dm + (int32_t)pick;
    const double L = (double)I.L, r = (double)p.rack_depth_dm, c = (double)p.cross_aisle_dm;
    const double num = 2.0 * r * L;
    const double den1 = (double)a + 2.0 * r;
    const double den2 = L + 2.0 * c;
    const double den = den1 * den2;
    out->width_dm = a;
    out->spacing_dm = a + 2 * p.rack_depth_dm;
    out->feasible = feasible ? 1 : 0;
    out->widths_evaluated = (int32_t)G;
    out->distance = dist[(size_t)pick];
    out->orders_per_window = delta_of(dist[(size_t)pick]);
    out->utilization = num / den;
    return WO_OK;
}
