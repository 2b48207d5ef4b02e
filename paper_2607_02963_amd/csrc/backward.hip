// C ABI of the whole-branch attention backward (include/pdec.h): argument
// checks, the plan of tiles and splits, and the launches of kernel_bwd.h and
// kernel_bwd_small.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "pdec.h"
#include "kernel_bwd.h"
#include "kernel_bwd_small.h"

namespace {

bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

int check_dims(const pdec_dims* d)
{
    if (!d) return PDEC_ERR_INVALID_ARG;
    if (d->num_events < 1 || d->num_q_heads < 1 || d->num_kv_heads < 1 || d->event_cap < 1 ||
        d->max_prefix_len < 0 || d->queries_per_stream < 0)
        return PDEC_ERR_INVALID_ARG;
    if (d->num_q_heads % d->num_kv_heads != 0) return PDEC_ERR_INVALID_ARG;
    // as for the forward: a scale <= 0 selects 1/sqrt(D); a positive one must be finite
    if (!(d->softmax_scale <= 0.f) && !std::isfinite(d->softmax_scale)) return PDEC_ERR_INVALID_ARG;
    if (d->dtype != PDEC_DTYPE_BF16 || (d->head_dim != 64 && d->head_dim != 128)) return PDEC_ERR_UNSUPPORTED;
    if (d->plan_mask != 0 || d->cross_causal != 0) return PDEC_ERR_UNSUPPORTED;
    const long N = d->queries_per_stream > 0 ? d->queries_per_stream : 1;
    const long rows = (long)d->num_events * N * d->num_q_heads;
    if (rows > (1L << 30) || (long)d->num_events * N * (d->num_q_heads / d->num_kv_heads) > (1L << 30) ||
        (long)d->num_events * ((d->event_cap + 63) / 64) + (d->max_prefix_len + 63) / 64 > (1L << 30))
        return PDEC_ERR_UNSUPPORTED;
    return PDEC_OK;
}

long ceil_div(long a, long b) { return (a + b - 1) / b; }

size_t workspace_for(const pdec_dims* d)
{
    const long N = d->queries_per_stream > 0 ? d->queries_per_stream : 1;
    return (size_t)d->num_events * N * d->num_q_heads * sizeof(float);
}

// Splits of the two passes: at most one of them is above 1 (kernel_bwd.h).
struct BwdPlan {
    int row_splits, key_splits, unit_per_chunk;
    long kv_elems, dq_elems;  // elements of one tensor that a split pass writes
    long part_n;              // dq splits that one prefix gradient holds
    bool small;               // the small tiles (kernel_bwd_small.h), without splits
};

// A stage of the dk, dv pass takes about 2.4 us, a unit of the dq pass about 2.5,
// an item a few of either to start and end, the sum a launch and its bytes.
constexpr double kStageUs = 2.4, kUnitUs = 2.5, kItemUs = 6.0, kSumUs = 16.0, kBytesPerUs = 4.0e6;

BwdPlan make_plan(const pdec_dims* d)
{
    BwdPlan p{};
    const long N = d->queries_per_stream > 0 ? d->queries_per_stream : 1;
    const long E = d->num_events, D = d->head_dim, H_kv = d->num_kv_heads, G = d->num_q_heads / H_kv;
    const long L = d->max_prefix_len, cap = d->event_cap, NG = N * G, R = E * NG;
    const double cus = 256.0;  // one work-group per compute unit

    // dk, dv: tiles of 128 keys, each walking the rows in 64-row stages; the
    // splits cut the prefix's rows (a pure causal sequence's own rows, where
    // a tile sees half of them on average)
    const long tiles = (L > 0 ? ceil_div(L, 128) : E * ceil_div(cap, 128)) * H_kv;
    const long stages = ceil_div(L > 0 ? R : NG, 64), kv_keys = L > 0 ? L : E * cap;
    p.kv_elems = kv_keys * H_kv * D;
    auto kv_us = [&](long n) {
        const double item = ceil_div(stages, n) * kStageUs + kItemUs;
        const double t = L > 0 ? std::ceil(tiles * n / cus) * item
                               : std::max(item, tiles * n / cus * (0.5 * stages / n * kStageUs + kItemUs));
        return n > 1 ? t + kSumUs + 16.0 * p.kv_elems * n / kBytesPerUs : t;
    };
    // dq: groups of 256 rows, each walking its 64-key units
    const long groups = ceil_div(R, 256) * H_kv;
    const long full = ceil_div(std::min(cap, N), 64), spans = std::min<long>(E, 254 / NG + 2);
    const long own = spans >= 2 ? (spans - 1) * full + std::min(full, ceil_div(256 / G + 2, 64)) : full;
    const long upre = ceil_div(L, 64), units = std::max<long>(upre + own, 1);
    p.dq_elems = R * H_kv * D;
    auto dq_us = [&](long n) {
        const double item = ceil_div(units, n) * kUnitUs + kItemUs;
        const double t = own > upre ? std::max(item, groups * n / cus * ((upre + 0.5 * own) / n * kUnitUs + kItemUs))
                                    : std::ceil(groups * n / cus) * item;
        return n > 1 ? t + kSumUs + 8.0 * p.dq_elems * n / kBytesPerUs : t;
    };
    // Later splits of dk, dv fit in dq, those of dq in dk_prefix and dv_prefix.
    p.part_n = L / R;
    p.row_splits = p.key_splits = 1;
    double best = kv_us(1) + dq_us(1);
    for (long n = 2; n <= std::min<long>({stages, 32, 1 + R / (2 * kv_keys)}); ++n) {
        const double t = kv_us(n) + dq_us(1);
        if (t >= best) continue;
        best = t;
        p.row_splits = (int)n;
    }
    for (long n = 2; n <= std::min<long>({units, 64, 1 + 2 * p.part_n}); ++n) {
        if (ceil_div(units, ceil_div(units, n)) != n) continue;
        const double t = kv_us(1) + dq_us(n);
        if (t >= best) continue;
        best = t;
        p.row_splits = 1;
        p.key_splits = (int)n;
    }
    p.unit_per_chunk = (int)std::min<long>(ceil_div(units, p.key_splits), 1L << 24);

    // The small tiles, for calls that leave the chip idle and whose splits the
    // output buffers do not hold.  Both times as fitted to measurements of the two
    // (4 to 24 streams of 10 to 80 tokens over 300 to 4000 keys, five head
    // layouts: within 10%): the launches, the longest work-group's row stages and
    // key tiles times the rounds, and the sums of splits.
    if (L > 0) {
        const bool wide = d->head_dim == 128;
        const bool split = p.row_splits > 1 || p.key_splits > 1;
        const double split_bytes = p.row_splits > 1 ? 16.0 * p.kv_elems * p.row_splits : split ? 8.0 * p.dq_elems * p.key_splits : 0.0;
        const double large_us = (wide ? 18.0 : 14.0) +
                                (wide ? 1.9 : 1.2) * std::ceil(tiles * p.row_splits / cus) * ceil_div(stages, p.row_splits) +
                                (wide ? 3.9 : 2.5) * std::ceil(groups * p.key_splits / cus) * p.unit_per_chunk +
                                (split ? 5.0 : 0.0) + 2.2 * split_bytes / kBytesPerUs;
        const long own_tiles = std::min<long>(E, 62 / NG + 2) * ceil_div(std::min(cap, N), 128);
        const double kv_wgs = (ceil_div(L, 64) + E * ceil_div(cap, 64)) * H_kv, dq_wgs = ceil_div(R, 64) * H_kv;
        const double small_us = (wide ? 7.0 : 5.0) + (wide ? 4.2 : 2.7) * ceil_div(R, 64) * std::max(1.0, kv_wgs / cus) +
                                (wide ? 2.8 : 1.7) * (ceil_div(L, 128) + own_tiles) * std::max(1.0, dq_wgs / cus);
        p.small = small_us < large_us;
        if (p.small) p.row_splits = p.key_splits = 1;
    }
    return p;
}

int launch_status() { return hipGetLastError() == hipSuccess ? PDEC_OK : PDEC_ERR_HIP; }

int launch_sum(float* out0, float* out1, const pdec::BwdArgs& a, int splits, hipStream_t s)
{
    const int tensors = out1 ? 2 : 1;
    const long n4 = a.part_elems / 4;
    hipLaunchKernelGGL(pdec::bwd_sum_kernel, dim3((unsigned)ceil_div(n4, 256), tensors), dim3(256), 0, s,
                       reinterpret_cast<pdec::f32x4_t*>(out0), reinterpret_cast<pdec::f32x4_t*>(out1),
                       reinterpret_cast<const pdec::f32x4_t*>(a.part0), reinterpret_cast<const pdec::f32x4_t*>(a.part1),
                       n4, tensors, (int)a.part_n, splits);
    return launch_status();
}

template <int D>
int launch_dkdv(pdec::BwdArgs a, const BwdPlan& p, hipStream_t s)
{
    a.part0 = a.dq;
    a.part_elems = p.kv_elems;
    a.part_n = p.row_splits;
    const long tiles = ceil_div(a.Lmax, 128) + a.E * ceil_div(a.cap, 128);
    hipLaunchKernelGGL((pdec::bwd_dkdv_kernel<D>), dim3((unsigned)tiles, a.H_kv, p.row_splits), dim3(256), 0, s, a);
    const int rc = launch_status();
    if (rc != PDEC_OK || p.row_splits == 1) return rc;
    return a.Lmax > 0 ? launch_sum(a.dkp, a.dvp, a, p.row_splits, s) : launch_sum(a.dke, a.dve, a, p.row_splits, s);
}

template <int D>
int launch_dq(pdec::BwdArgs a, const BwdPlan& p, hipStream_t s)
{
    a.part0 = a.dkp;
    a.part1 = a.dvp;
    a.part_elems = p.dq_elems;
    a.part_n = p.part_n;
    hipLaunchKernelGGL((pdec::bwd_dq_kernel<D>), dim3((unsigned)ceil_div(a.R, 256), a.H_kv, p.key_splits), dim3(256), 0,
                       s, a);
    const int rc = launch_status();
    return rc != PDEC_OK || p.key_splits == 1 ? rc : launch_sum(a.dq, nullptr, a, p.key_splits, s);
}

template <int D>
int launch_drow(const pdec::BwdArgs& a, hipStream_t s)
{
    const long rows = (long)a.E * a.N * a.H_q;
    hipLaunchKernelGGL((pdec::bwd_drow_kernel<D>), dim3((unsigned)ceil_div(rows, 16)), dim3(256), 0, s, a);
    return launch_status();
}

template <int D>
int launch_small(const pdec::BwdArgs& a, hipStream_t s)
{
    int rc = launch_drow<D>(a, s);
    if (rc != PDEC_OK) return rc;
    const long units = ceil_div(a.Lmax, 64) + a.E * ceil_div(a.cap, 64);
    hipLaunchKernelGGL((pdec::bwd_small_dkdv_kernel<D>), dim3((unsigned)units, a.H_kv), dim3(256), 0, s, a);
    if ((rc = launch_status()) != PDEC_OK) return rc;
    hipLaunchKernelGGL((pdec::bwd_small_dq_kernel<D>), dim3((unsigned)ceil_div(a.R, 64), a.H_kv), dim3(512), 0, s, a);
    return launch_status();
}

template <int D>
int launch(const pdec::BwdArgs& a, const BwdPlan& p, hipStream_t s)
{
    if (p.small) return launch_small<D>(a, s);
    int rc = PDEC_OK;
    if (p.row_splits > 1) {
        // dk, dv first, whose later splits dq holds: D in a pass of its own
        rc = launch_drow<D>(a, s);
        if (rc == PDEC_OK) rc = launch_dkdv<D>(a, p, s);
        if (rc == PDEC_OK) rc = launch_dq<D>(a, p, s);
    } else {
        rc = launch_dq<D>(a, p, s);
        if (rc == PDEC_OK) rc = launch_dkdv<D>(a, p, s);
    }
    return rc;
}

}  // namespace

extern "C" {

size_t pdec_backward_workspace_size(const pdec_dims* dims)
{
    return check_dims(dims) == PDEC_OK ? workspace_for(dims) : 0;
}

int pdec_query_backward_plan(const pdec_dims* dims, int32_t* small_tiles, int32_t* row_splits, int32_t* key_splits)
{
    const int rc = check_dims(dims);
    if (rc != PDEC_OK) return rc;
    const BwdPlan p = make_plan(dims);
    if (small_tiles) *small_tiles = p.small;
    if (row_splits) *row_splits = p.row_splits;
    if (key_splits) *key_splits = p.key_splits;
    return PDEC_OK;
}

int pdec_attn_prefill_backward(const pdec_dims* dims, const void* q, const void* k_prefix, const void* v_prefix,
                               const void* k_event, const void* v_event, const int32_t* event_lens,
                               const int32_t* prefix_lens, const void* out, const float* lse, const void* dout,
                               float* dq, float* dk_prefix, float* dv_prefix, float* dk_event, float* dv_event,
                               void* workspace, size_t workspace_bytes, void* stream)
{
    const int rc = check_dims(dims);
    if (rc != PDEC_OK) return rc;
    for (const void* p : {q, k_event, v_event, out, dout})
        if (!p || !aligned(p, 16)) return PDEC_ERR_INVALID_ARG;
    for (const void* p : {(const void*)dq, (const void*)dk_event, (const void*)dv_event})
        if (!p || !aligned(p, 16)) return PDEC_ERR_INVALID_ARG;
    for (const void* p : {k_prefix, v_prefix, (const void*)dk_prefix, (const void*)dv_prefix})
        if ((!p && dims->max_prefix_len > 0) || !aligned(p, 16)) return PDEC_ERR_INVALID_ARG;
    if (!event_lens || !aligned(event_lens, 4) || !prefix_lens || !aligned(prefix_lens, 4)) return PDEC_ERR_INVALID_ARG;
    if (!lse || !aligned(lse, 4)) return PDEC_ERR_INVALID_ARG;
    if (!workspace || !aligned(workspace, 16)) return PDEC_ERR_INVALID_ARG;
    if (workspace_bytes < workspace_for(dims)) return PDEC_ERR_WORKSPACE;

    const BwdPlan p = make_plan(dims);
    pdec::BwdArgs a{};
    a.q = static_cast<const uint16_t*>(q);
    a.kp = static_cast<const uint16_t*>(k_prefix);
    a.vp = static_cast<const uint16_t*>(v_prefix);
    a.ke = static_cast<const uint16_t*>(k_event);
    a.ve = static_cast<const uint16_t*>(v_event);
    a.event_lens = event_lens;
    a.prefix_len = prefix_lens;
    a.out = static_cast<const uint16_t*>(out);
    a.lse = lse;
    a.dout = static_cast<const uint16_t*>(dout);
    a.dq = dq;
    a.dkp = dk_prefix;
    a.dvp = dv_prefix;
    a.dke = dk_event;
    a.dve = dv_event;
    a.drow = static_cast<float*>(workspace);
    a.E = dims->num_events;
    a.N = dims->queries_per_stream > 0 ? dims->queries_per_stream : 1;
    a.H_q = dims->num_q_heads;
    a.H_kv = dims->num_kv_heads;
    a.G = a.H_q / a.H_kv;
    a.cap = dims->event_cap;
    a.R = a.E * a.N * a.G;
    a.row_splits = p.row_splits;
    a.key_splits = p.key_splits;
    a.unit_per_chunk = p.unit_per_chunk;
    a.Lmax = dims->max_prefix_len;
    a.tau = dims->softmax_scale > 0.f ? dims->softmax_scale : 1.f / std::sqrt((float)dims->head_dim);
    a.c = a.tau * pdec::kLog2eF;
    hipStream_t s = static_cast<hipStream_t>(stream);
    return dims->head_dim == 128 ? launch<128>(a, p, s) : launch<64>(a, p, s);
}

}  // extern "C"
