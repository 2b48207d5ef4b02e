// float32 split pass, on v_mfma_f32_16x16x4_f32.
//
// Same work items as the other split passes: (video, kv head, chunk of the
// virtual key sequence, row group; pdec_common.h), with 16 NT rows per group.
// The work-group is 4 waves; wave w takes keys 16 w .. 16 w + 15 of every unit
// of the chunk with its own online-softmax state, and the four states are
// merged in LDS at the end.
//
//   S^T  = K  Q^T    A = 16 keys x 4 d, B = 4 d x 16 rows, D / 4 steps: lane
//                    (l % 16, k = l / 16) holds elements k D/4 + t of its key
//                    (row) at step t, D/4 consecutive floats of one row
//   O^T += V^T P^T   A = 16 d x 4 keys, B = 4 keys x 16 rows: step i takes keys
//                    4 k + i, so the S^T accumulator's register i (row l % 16,
//                    key 4 (l / 16) + i) is the B operand; tile dt takes
//                    d = DT (l % 16) + dt, DT consecutive floats of a value
//                    row, and leaves a lane D/4 consecutive d of its row
//
// K, V and Q go straight from memory to registers in 16-byte loads, the next
// unit's K requested after this one's scores and its V after this one's P V;
// nothing is staged.  Two work-groups share a compute unit.  Products and sums are float32, as in a
// vector kernel.
//
// What bounds it: a small step is a chain of memory round trips, so a chunk
// may be a single unit, spread over four waves, with V requested beside K; a
// larger one the float32 products, which read every operand from registers
// where a vector kernel reads the query rows from LDS once per multiply-add
// quartet, and serve 16 NT rows per key read where it served 8.
#pragma once

#include "kernel_mfma.h"
#include "kernel_valu.h"

namespace pdec {

__device__ inline f32x4_t mfma_16x16x4(float a, float b, f32x4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <int D, int NT, bool PLAN>
__global__ __launch_bounds__(256, 2) void split_f32_kernel(StepArgs a)
{
    constexpr int NW = 4;
    constexpr int RT = 16 * NT;   // rows per item
    constexpr int KPL = D / 4;    // floats of a key (query) row per lane
    constexpr int DT = D / 16;    // 16-wide d tiles
    constexpr int VQ = DT / 4;    // 16-byte words per value row and lane
    constexpr int OROW = D + 4;   // row pitch of the merge buffer, in floats
    // the unit table, and after the last unit the waves' outputs in its place
    constexpr int TAB = (2 * kMaxStreamsPerVideo + 1) * 4, MERGE = NW * RT * OROW * 4;
    __shared__ __attribute__((aligned(16))) unsigned char buf[TAB > MERGE ? TAB : MERGE];
    __shared__ float m_s[NW][RT], l_s[NW][RT];
    __shared__ int s_total;
    int* const tab_start = reinterpret_cast<int*>(buf);
    int* const tab_nlen = tab_start + kMaxStreamsPerVideo + 1;
    float* const o_s = reinterpret_cast<float*>(buf);

    ValuItem it;
    if (!valu_item<RT>(a, it, tab_start, tab_nlen, &s_total)) return;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
    const float c = a.qscale;
    const uint32_t stride_b = (uint32_t)a.H_kv * D * 4;

    // the next unit at or after u that some row of the item sees (an own unit
    // concerns its stream's rows)
    auto next_unit = [&](int u, UnitInfo& ui) {
        for (; u < it.u1; ++u) {
            ui = uniform_unit(unit_info(a, it.vi, it.upre, tab_start, tab_nlen, it.id.g, u));
            if (ui.stream < 0 || (ui.stream * a.G < it.row0 + it.nrows && (ui.stream + 1) * a.G > it.row0)) break;
        }
        return u;
    };
    // this wave's operands of a unit; keys past the last valid one re-read it
    // (their scores are masked)
    f32x4_t kx[KPL / 4], vx[4][VQ];
    auto load_k = [&](const UnitInfo& ui) {
        const unsigned char* kb =
            static_cast<const unsigned char*>(ui.stream < 0 ? a.k_prefix : a.k_event) + ui.key_off * 4;
        const AppendedKey ak = appended_key(a, it.vi, ui, it.id.g, 4);  // fused append: key from k_new / v_new
        const int kk = min(16 * w + l16, ui.nk - 1);
        const unsigned char* kr = (kk == ak.key ? ak.krow : kb + (size_t)kk * stride_b) + 4 * KPL * lg;
#pragma unroll
        for (int j = 0; j < KPL / 4; ++j) kx[j] = *reinterpret_cast<const f32x4_t*>(kr + 16 * j);
    };
    auto load_v = [&](const UnitInfo& ui) {
        const unsigned char* vb =
            static_cast<const unsigned char*>(ui.stream < 0 ? a.v_prefix : a.v_event) + ui.key_off * 4;
        const AppendedKey ak = appended_key(a, it.vi, ui, it.id.g, 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int kv = min(16 * w + 4 * lg + i, ui.nk - 1);
            const unsigned char* vr = (kv == ak.key ? ak.vrow : vb + (size_t)kv * stride_b) + 4 * DT * l16;
#pragma unroll
            for (int j = 0; j < VQ; ++j) vx[i][j] = *reinterpret_cast<const f32x4_t*>(vr + 16 * j);
        }
    };
    UnitInfo ui;
    int u = next_unit(it.u0, ui);
    if (u < it.u1) {
        load_k(ui);
        load_v(ui);
    }

    int row_stream[NT];
    f32x4_t qv[NT][KPL / 4];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int r = 16 * nt + l16;
        row_stream[nt] = r < it.nrows ? (it.row0 + r) / a.G : -2;
        const float* q = static_cast<const float*>(a.q) +
                         (long)row_qrow(a, it.vi, it.id.g, it.row0 + min(r, it.nrows - 1)) * D + KPL * lg;
#pragma unroll
        for (int j = 0; j < KPL / 4; ++j) qv[nt][j] = *reinterpret_cast<const f32x4_t*>(q + 4 * j);
    }

    f32x4_t o[NT][DT];
    float m_ref[NT], l_lane[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        m_ref[nt] = kMinRef;
        l_lane[nt] = 0.f;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[nt][dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }

    // Units of which a row may see nothing, streams' own and those of the plan
    // segment under the self-only mask, come last.  There a row that sees none of
    // the wave's keys keeps its sums as they are: 0 times an infinite or NaN
    // value of another stream would be NaN.
    auto apart_unit = [&](const UnitInfo& x) { return x.stream >= 0 || (PLAN && x.k0 + kUnit > it.vi.plan0); };
    auto unit_pass = [&](auto apart) __attribute__((always_inline)) {
        constexpr bool APART = decltype(apart)::value;
        const UnitInfo cur = ui;
        f32x4_t s[NT][2];  // two sums per tile: the products of one wait for each other
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) s[nt][0] = s[nt][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < KPL; ++t)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                s[nt][t & 1] = mfma_16x16x4(kx[t >> 2][t & 3], qv[nt][t >> 2][t & 3], s[nt][t & 1]);
        u = next_unit(u + 1, ui);
        if (u < it.u1) load_k(ui);  // in flight under this unit's softmax and P V

        if (16 * w < cur.nk) {
            const bool plan_unit = PLAN && APART && cur.stream < 0;  // self-only mask
            bool none[NT];
            float p[NT][4], mx[NT];
            bool need = false;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const bool row_sees =
                    row_stream[nt] != -2 && (!APART || cur.stream < 0 || row_stream[nt] == cur.stream);
                bool sees[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int key = 16 * w + 4 * lg + i;
                    sees[i] = row_sees & (key < cur.nk);
                    if (plan_unit) sees[i] = sees[i] & !plan_key_hidden(a, it.vi, cur.k0 + key, row_stream[nt]);
                    p[nt][i] = sees[i] ? (s[nt][0][i] + s[nt][1][i]) * c : kNegInf;
                }
                mx[nt] = fmaxf(fmaxf(p[nt][0], p[nt][1]), fmaxf(p[nt][2], p[nt][3]));
                need |= mx[nt] > m_ref[nt] + 8.f;
                none[nt] = !row_sees;
                if (plan_unit) {  // some lane of the row (one of four) sees a key
                    uint64_t b = 0;
#pragma unroll
                    for (int i = 0; i < 4; ++i) b |= __ballot(sees[i]);
                    b |= b >> 32;
                    none[nt] = ((b | (b >> 16)) >> l16 & 1) == 0;
                }
            }
            if (__any(need)) {  // rare after a row's first keys
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const float mt = max_over_groups(mx[nt]);
                    const bool up = mt > m_ref[nt] + 8.f;
                    const float alpha = up ? fast_exp2(m_ref[nt] - mt) : 1.f;
                    m_ref[nt] = up ? mt : m_ref[nt];
                    l_lane[nt] *= alpha;
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt) o[nt][dt] *= alpha;
                }
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    p[nt][i] = fast_exp2(p[nt][i] - m_ref[nt]);  // 0 for a hidden key
                    l_lane[nt] += p[nt][i];
                }
            if constexpr (!APART) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt)
                            o[nt][dt] = mfma_16x16x4(vx[i][dt >> 2][dt & 3], p[nt][i], o[nt][dt]);
            } else {
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        f32x4_t x = o[nt][dt];
#pragma unroll
                        for (int i = 0; i < 4; ++i) x = mfma_16x16x4(vx[i][dt >> 2][dt & 3], p[nt][i], x);
#pragma unroll
                        for (int j = 0; j < 4; ++j) o[nt][dt][j] = none[nt] ? o[nt][dt][j] : x[j];
                    }
                    __builtin_amdgcn_sched_barrier(0);  // one d tile at a time: few registers
                }
            }
        }
        if (u < it.u1) load_v(ui);  // under the next scores
    };
    while (u < it.u1 && !apart_unit(ui)) unit_pass(std::false_type{});
    while (u < it.u1) unit_pass(std::true_type{});

    // ---- merge of the four waves, and the item's slot ----
    // lane: row l % 16 of tile nt, d = D/4 (l / 16) + DT j + dt
    __syncthreads();  // the table is no longer read
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        float l = l_lane[nt];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        const int r = 16 * nt + l16;
        if (lg == 0) {
            m_s[w][r] = m_ref[nt];
            l_s[w][r] = l;
        }
        float* dst = o_s + (w * RT + r) * OROW + KPL * lg;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int k = 0; k < VQ; ++k)
                *reinterpret_cast<f32x4_t*>(dst + DT * j + 4 * k) =
                    f32x4_t{o[nt][4 * k][j], o[nt][4 * k + 1][j], o[nt][4 * k + 2][j], o[nt][4 * k + 3][j]};
    }
    __syncthreads();
    for (int i = tid; i < it.nrows * (D / 4); i += 256) {
        const int r = i / (D / 4), d4 = i % (D / 4);
        float M = m_s[0][r];
#pragma unroll
        for (int x = 1; x < NW; ++x) M = fmaxf(M, m_s[x][r]);
        float L = 0.f;
        f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int x = 0; x < NW; ++x) {
            const float f = fast_exp2(m_s[x][r] - M);  // 0 for a wave that saw none of the row's keys
            L += f * l_s[x][r];
            acc += f * *reinterpret_cast<const f32x4_t*>(o_s + (x * RT + r) * OROW + 4 * d4);
        }
        const long slot = (long)row_qrow(a, it.vi, it.id.g, it.row0 + r) * a.max_chunks + it.id.c;
        const float inv = L > 0.f ? 1.f / L : 0.f;  // stored normalised
        *reinterpret_cast<f32x4_t*>(static_cast<float*>(a.part_o) + slot * D + 4 * d4) = acc * inv;
        if (d4 == 0) *reinterpret_cast<float2*>(a.part_ml + 2 * slot) = make_float2(M, L);
    }
}

}  // namespace pdec
