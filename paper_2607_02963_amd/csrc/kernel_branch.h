// Whole-branch attention (several query tokens per stream: the training /
// prefill form of the §3.4 mask, and with one stream and no prefix a causal
// prefill), bf16, on v_mfma_f32_32x32x16_bf16.
//
// Query token j of stream f sees every prefix key and the rows t <= j of its
// own cache; with the causal-attention variant also the rows t < j of the
// video's other streams.  A work item is (video, kv head, chunk, row group):
// 128 * NT consecutive query rows (stream-major, then token, then head of the
// group), NT 32-row tiles in each of four waves, against a chunk of the row
// group's own key sequence
//
//   [ prefix units ] [ units of the caches that some row of the group sees ]
//
// in 64-key units.  Each unit is one stage of a four-slot LDS ring filled by
// global_load_lds_dwordx4.
//
// Per 32-key block:
//   S^T  = K  Q^T    A = 32 keys x 16 d (LDS), B = Q^T (registers)
//   O^T += V^T P^T   A = V^T via ds_read_b64_tr_b16, B = P^T (registers)
// The S^T accumulator gives lane l the scores of row l % 32 for keys
// 8 (i / 4) + 4 (l / 32) + i % 4, register i: registers 8 s .. 8 s + 7 are the
// B operand of the s-th 16-key step of the second product, the transposing
// read fetching V^T with the same key order.
//
// What bounds it and why this shape: a dense contraction, so the matrix
// cores (512 cycles per SIMD for 16 rows x 64 keys at D = 128) should.  Two
// other units come close: the LDS serves 128 bytes per cycle, and 32 rows per
// wave would read the K and V stage eight times per 256 rows (2048 cycles,
// the products' own time), 64 rows per wave four times; and the softmax takes
// 3.5 vector instructions per score.  So a wave holds 64 rows (one wave per
// SIMD, 512 registers), and the loop is software-pipelined: the scores of
// block b + 1 are multiplied under the exponentials of block b, and the P V
// products of block b run under the maxima of block b + 1, with scheduling
// groups interleaving the two kinds of instruction.
#pragma once

#include "kernel_mfma.h"
#include "ring.h"

namespace pdec {

typedef __attribute__((ext_vector_type(16))) float bf32x16_t;

__device__ inline bf32x16_t branch_mfma(u32x4_t a, u32x4_t b, bf32x16_t c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a), as_bf16x8(b), c, 0, 0, 0);
}

// Index of the work-group and of the lane within it.  blockIdx and threadIdx
// are device library functions; this translation unit is compiled without the
// IEEE mode bit, which keeps them as calls here, and a call's stack would put
// the kernel's arguments in private memory.  (The decode step's kernels are
// faster with the calls: without them the compiler moves their index work
// into the loop's registers, and the sixteen-wave form spills.)
__device__ inline int wg_id() { return (int)__builtin_amdgcn_workgroup_id_x(); }
__device__ inline int wi_id() { return (int)__builtin_amdgcn_workitem_id_x(); }

// Chunk permutations of the staged rows (16-byte chunk ch of key k sits at
// ch ^ swizzle(k)): the 16 lanes of one LDS phase of the K read hold 16 keys
// of one chunk, the 32 lanes of one phase of the transposing V read hold four
// keys of four chunks.
template <int D>
__device__ inline int branch_kswz(int key) { return D == 128 ? (key & 15) : ((key >> 1) & 7); }
template <int D>
__device__ inline int branch_vswz(int key)
{
    return D == 128 ? ((6 * (key & 1)) ^ (12 * ((key >> 1) & 1))) : 4 * ((key >> 1) & 1);
}

// One wave-wide 16-byte-per-lane DMA from a scalar base plus 32-bit lane
// offsets into LDS, M0 left changed (dma_16B_sbase restores it; a reserved
// register, which the compiler sets right before each instruction of its own
// that reads it).
// lanes is the set of lanes that load, never empty (ring.h).  Called with every
// lane of the wave active.
// Its base comes from scalar arithmetic, far from any vector write of an SGPR
// (which the load would have to follow by five wait states).
__device__ inline void dma_16B_m0(const void* base, uint32_t off, uint32_t lds_base, uint64_t lanes)
{
    const uint64_t sb = sgpr_base(base);
    asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 exec, %3\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b64 exec, -1" :
                 : "s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(off), "s"(sb), "s"(sgpr_base(reinterpret_cast<const void*>(lanes)))
                 : "memory");
}

template <int D, int NT, int NW>
struct BranchCfg {
    static constexpr int ROWB = 2 * D;
    static constexpr int CH = D / 8;                      // 16-byte chunks per key row
    static constexpr int STAGE_K = kUnit * ROWB;
    static constexpr int STAGE = 2 * STAGE_K;             // K, then V
    static constexpr int NSTAGE = 4;
    static constexpr int PIECES = STAGE / 1024;           // 1 KB per wave DMA instruction
    static constexpr int PPW = PIECES / NW;               // pieces per wave: the lower half of the waves K, the upper half V
    static constexpr int KPI = 1024 / ROWB;               // keys per piece
    static constexpr int KS = D / 16;                     // 16-wide d steps of the scores
    static constexpr int DT = D / 32;                     // 32-wide d tiles of O
    static constexpr int WROWS = 32 * NT;                 // rows per wave
    static constexpr int RT = NW * WROWS;                 // rows per item
};

// own_bound: a bound on the own units that one row group sees; rows_first: the
// order in which work-groups take the items.
template <int D, int NT, int NW, bool CROSS>
__global__ __launch_bounds__(64 * NW) void branch_kernel(StepArgs a, int own_bound, int rows_first)
{
    using C = BranchCfg<D, NT, NW>;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[C::NSTAGE * C::STAGE];
    // units of the streams a row group may see, when it may see several:
    // start[i] = first unit of stream fa + i, nlen[i] = its visible rows
    __shared__ int tab_start[kMaxStreamsPerVideo + 1];
    __shared__ int tab_nlen[kMaxStreamsPerVideo];

    // ---- which item; every branch is uniform over the work-group ----
    // Row groups of one chunk read the same keys.  They are numbered one after
    // another and the items cut into eight contiguous runs, one per XCD (block b
    // runs on XCD b % 8), so that they meet in one L2 and every XCD gets as many.
    // The items of a causal sequence, whose row groups differ in length, are taken
    // in another order instead: the (chunk, head) pairs in turn, the longest row
    // groups first, so that the long items are spread over the XCDs.  A batch's
    // videos differ in their numbers of row groups and chunks: there the items
    // that exist are counted first.
    const int upc = a.unit_per_chunk;
    auto chunks_of = [&](const VideoInfo& x) __attribute__((always_inline)) {  // slots that hold states
        return min(max(((x.L + kUnit - 1) / kUnit + own_bound + upc - 1) / upc, 1), a.max_chunks);
    };
    int v = 0, c_idx, g, rg;
    if (a.num_videos > 1) {
        const int l = wi_id() & 63;
        auto items_of = [&](int x) __attribute__((always_inline)) {
            if (x >= a.num_videos) return 0;
            const VideoInfo xi = video_info(a, x);
            return a.H_kv * chunks_of(xi) * ((xi.E * a.G * a.qps + C::RT - 1) / C::RT);
        };
        auto scan = [&](int x) __attribute__((always_inline)) {  // inclusive, over the lanes
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int y = __shfl_up(x, off);
                if (l >= off) x += y;
            }
            return x;
        };
        int total = 0;
        for (int v0 = 0; v0 < a.num_videos; v0 += 64) total += __shfl(scan(items_of(v0 + l)), 63);
        const int per = (total + 7) / 8;
        int i = (wg_id() % 8) * per + wg_id() / 8;
        if (wg_id() / 8 >= per || i >= total) return;
        for (int v0 = 0;; v0 += 64) {
            const int n = items_of(v0 + l), incl = scan(n), all = __shfl(incl, 63);
            if (i >= all) {
                i -= all;
                continue;
            }
            const int at = __builtin_ctzll(__ballot(incl > i));
            v = v0 + at;
            i -= __shfl(incl - n, at);
            break;
        }
        v = __builtin_amdgcn_readfirstlane(v);
        i = __builtin_amdgcn_readfirstlane(i);
        const int groups = (video_info(a, v).E * a.G * a.qps + C::RT - 1) / C::RT;
        rg = i % groups;
        g = i / groups % a.H_kv;
        c_idx = i / groups / a.H_kv;
    } else {
        const int b = wg_id(), P = a.n_items / a.rg_max, per = (a.n_items + 7) / 8;
        int p;
        if (rows_first) {
            if (b >= a.n_items) return;
            // where the eight XCDs would each meet the same pairs in every step, the
            // chunks move on by one, so that each gets early ones and late, short ones
            const int step = b / P;
            p = (b % P + a.H_kv * (P % 8 == 0 ? step : 8 % P == 0 ? step * P / 8 : 0)) % P;
            rg = a.rg_max - 1 - step;
        } else {
            const int i = (b % 8) * per + b / 8;
            if (i >= a.n_items || b / 8 >= per) return;
            p = i / a.rg_max;
            rg = i % a.rg_max;
        }
        g = p % a.H_kv;
        c_idx = p / a.H_kv;
    }
    const VideoInfo vi = video_info(a, v);
    const int per_stream = a.G * a.qps;
    const int R = vi.E * per_stream;
    const int row0 = rg * C::RT;
    const int upre = (vi.L + kUnit - 1) / kUnit;
    const int nch = chunks_of(vi);
    if (c_idx == 0 && g == 0 && rg == 0 && wi_id() == 0) a.video_chunks[v] = nch;
    if (row0 >= R || c_idx >= nch) return;
    const int nrows = min(C::RT, R - row0);

    const int tid = wi_id();
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
    const float c = a.qscale;

    // streams whose caches some row of the group sees, and their visible rows
    const int f_lo = row0 / per_stream, f_hi = (row0 + nrows - 1) / per_stream;
    const int tok_last = ((row0 + nrows - 1) / a.G) % a.qps;  // token of the group's last row
    const int fa = CROSS ? 0 : f_lo, fb = CROSS ? vi.E - 1 : f_hi;
    const bool one = fa == fb;  // one stream: no table
    int own;                    // own units of the group
    int n_one = 0;
    if (one) {
        n_one = min(max(a.event_lens[vi.e0 + fa], 0), tok_last + 1);
        own = (n_one + kUnit - 1) / kUnit;
    } else {
        if (w == 0) {
            int base = 0;
            for (int f0 = fa; f0 <= fb; f0 += 64) {
                const int f = f0 + lane;
                // rows of stream f at or above the largest token that sees
                // them are left out (CROSS: any row of the group may)
                const int lim = f_lo < f_hi && (CROSS || f < f_hi) ? a.qps : tok_last + 1;
                const int n = f <= fb ? min(max(a.event_lens[vi.e0 + f], 0), lim) : 0;
                const int units = (n + kUnit - 1) / kUnit;
                int incl = units;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const int y = __shfl_up(incl, off);
                    if (lane >= off) incl += y;
                }
                if (f <= fb) {
                    tab_start[f - fa] = base + incl - units;
                    tab_nlen[f - fa] = n;
                }
                base += __shfl(incl, 63);
            }
            if (lane == 0) tab_start[fb - fa + 1] = base;
        }
        __syncthreads();
        own = __builtin_amdgcn_readfirstlane(tab_start[fb - fa + 1]);
    }
    const int u0 = c_idx * upc;
    // the last slot takes whatever is left
    const int u1 = c_idx == nch - 1 ? upre + own : min(u0 + upc, upre + own);
    const int nst = __builtin_amdgcn_readfirstlane(max(0, u1 - u0));

    auto unit = [&](int u) __attribute__((always_inline)) {
        const bool prefix = u < upre;
        int f = 0, t0 = (prefix ? u : u - upre) * kUnit, n = prefix ? vi.L : n_one;
        if (!prefix && !one) {
            int lo = 0, top = fb - fa;
            while (lo < top) {
                const int mid = (lo + top + 1) >> 1;
                if (tab_start[mid] <= u - upre) lo = mid; else top = mid - 1;
            }
            f = __builtin_amdgcn_readfirstlane(lo);
            t0 = (u - upre - __builtin_amdgcn_readfirstlane(tab_start[f])) * kUnit;
            n = __builtin_amdgcn_readfirstlane(tab_nlen[f]);
        }
        const long row = prefix ? (long)(vi.p0 + t0) : (long)(vi.e0 + fa + f) * a.cap + t0;
        return UnitInfo{(row * a.H_kv + g) * D, min(kUnit, n - t0), prefix ? -1 : fa + f, t0};
    };

    // ---- DMA of one stage: this wave's PPW pieces, all of K or all of V ----
    const bool w_is_v = w >= NW / 2;
    const int pk0 = (w % (NW / 2)) * C::PPW;
    // (selected as integers: a select over the argument struct's members
    // would put it in private memory)
    const uint64_t kpre = sgpr_base(a.k_prefix), vpre = sgpr_base(a.v_prefix);
    const uint64_t kevt = sgpr_base(a.k_event), vevt = sgpr_base(a.v_event);
    const uint64_t pre = w_is_v ? vpre : kpre, evt_pre = (w_is_v ? vevt : kevt) - pre;
    const uint32_t strideB = (uint32_t)a.H_kv * D * 2;
    const int pkey = lane / C::CH;  // key of the lane within a piece
    const int key0 = pk0 * C::KPI + pkey;
    const uint32_t k0off = (uint32_t)key0 * strideB;
    uint32_t choff[4];  // byte offset of the lane's chunk in piece i, of period 4 in i
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int key = key0 + i * C::KPI;
        choff[i] = 16u * ((lane % C::CH) ^ (w_is_v ? branch_vswz<D>(key) : branch_kswz<D>(key)));
    }
    const uint32_t m_base = lds_u32(lds) + (w_is_v ? C::STAGE_K : 0) + pk0 * 1024;
    // Stages past the last are pieces of one lane, so that every wait below
    // counts the same pieces.
    struct Pending { const uint16_t* base; uint32_t dst; int nk; uint64_t lanes; };
    auto pending = [&](int st) __attribute__((always_inline)) {
        const UnitInfo ui = unit(u0 + min(st, nst - 1));
        return Pending{reinterpret_cast<const uint16_t*>(pre + (ui.stream < 0 ? 0 : evt_pre) + 2 * ui.key_off),
                       m_base + (st % C::NSTAGE) * C::STAGE, ui.nk, ring_lanes(st, nst)};
    };
    auto issue_piece = [&](const Pending& pd, int i) __attribute__((always_inline)) {
        // keys past the last valid one re-read it (their scores are masked)
        const uint32_t row = key0 < pd.nk - i * C::KPI ? k0off + i * C::KPI * strideB : (uint32_t)(pd.nk - 1) * strideB;
        dma_16B_m0(pd.base, row + choff[i & 3], pd.dst + 1024 * i, pd.lanes);
    };
    auto issue_stage = [&](const Pending& pd) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < C::PPW; ++i) issue_piece(pd, i);
    };

    // ---- this lane's rows: 32 nt + l % 32 of the wave ----
    const int wrow0 = C::WROWS * w;
    const bool active = wrow0 < nrows;
    int r_tok[NT], r_stream[NT];
    u32x4_t qf[NT][C::KS];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        // rows past the item's last repeat it; their results are not stored
        const int r = row0 + min(wrow0 + 32 * nt + l32, nrows - 1);
        r_stream[nt] = r / per_stream;
        r_tok[nt] = (r / a.G) % a.qps;
        const uint16_t* q = static_cast<const uint16_t*>(a.q) + (long)row_qrow(a, vi, g, r) * D + 8 * hi;
#pragma unroll
        for (int t = 0; t < C::KS; ++t) qf[nt][t] = *reinterpret_cast<const u32x4_t*>(q + 16 * t);
    }
#pragma unroll
    for (int st = 0; st < C::NSTAGE - 1; ++st)
        if (nst > 0) issue_stage(pending(st));
    // the query loads and the DMA complete in no order relative to each other
    wait_vmcnt<0>();
    // the queries live in accumulation registers, which the products read
    // directly: the vector registers are for the scores, P and the operands
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int t = 0; t < C::KS; ++t) asm volatile("" : "+a"(qf[nt][t]));

    bf32x16_t o[NT][C::DT];
    f32x4_t lsum[NT];  // four times the lane's sum
    float m_ref[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        m_ref[nt] = kMinRef;
        lsum[nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
            for (int i = 0; i < 16; ++i) o[nt][dt][i] = 0.f;
    }

    // operand reads: K step t: key l % 32, chunk 2 t + l / 32; V d tile dt:
    // key 4 (q / 2) + (l % 16) / 4 (+ 16 s + 8 r), d 32 dt + 16 (q % 2) + 4 (l % 4) .. +3, q = l / 16
    // (2 t + l / 32 has no bits in common with the row offset: step t is koff ^ 32 t)
    const int koff = l32 * C::ROWB + 16 * (hi ^ branch_kswz<D>(l32));
    int voff[C::DT];
    {
        const int q = lane >> 4, i = lane & 15;
        const int key = 4 * (q >> 1) + (i >> 2);
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt)
            voff[dt] = key * C::ROWB + 16 * ((4 * dt + 2 * (q & 1) + ((i & 3) >> 1)) ^ branch_vswz<D>(key)) + 8 * (i & 1);
    }
    auto slot = [&](int st) __attribute__((always_inline)) { return lds + (st % C::NSTAGE) * C::STAGE; };
    auto read_k = [&](u32x4_t (&kf)[C::KS], const unsigned char* buf, int kb, int t) __attribute__((always_inline)) {
        kf[t] = *reinterpret_cast<const u32x4_t*>(buf + kb * C::ROWB + (koff ^ (32 * t)));
    };
    // half r (8 keys) of V operand (s, dt), index j = 2 (DT s + dt) + r
    auto read_v = [&](u32x2_t (&vf)[4 * C::DT], const unsigned char* buf, int kb, int j) __attribute__((always_inline)) {
        const int s = j / (2 * C::DT), dt = (j / 2) % C::DT;
        const unsigned char* va = buf + C::STAGE_K + (kb + 16 * s + 8 * (j & 1)) * C::ROWB + voff[dt];
        vf[j] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                                (__attribute__((address_space(3))) s16x4_t*)va));
    };
    auto v_op = [&](const u32x2_t (&vf)[4 * C::DT], int s, int dt) __attribute__((always_inline)) {
        const u32x2_t x0 = vf[2 * (C::DT * s + dt)], x1 = vf[2 * (C::DT * s + dt) + 1];
        return u32x4_t{x0.x, x0.y, x1.x, x1.y};
    };
    auto score_step = [&](bf32x16_t (&s)[NT], const u32x4_t (&kf)[C::KS], int i) __attribute__((always_inline)) {
        const int t = i / NT, nt = i % NT;
        if (t == 0) {
#pragma unroll
            for (int k = 0; k < 16; ++k) s[nt][k] = 0.f;
        }
        s[nt] = branch_mfma(kf[t], qf[nt][t], s[nt]);
    };
    auto pv_step = [&](const u32x4_t (&pk)[NT][2], const u32x2_t (&vf)[4 * C::DT], int i) __attribute__((always_inline)) {
        const int s = i / (C::DT * NT), dt = (i / NT) % C::DT, nt = i % NT;
        o[nt][dt] = branch_mfma(v_op(vf, s, dt), pk[nt][s], o[nt][dt]);
    };
    // The row sums of P (the rounded P, the one that meets V), each lane over
    // its own keys, four at a time, i = 0 .. 4 NT - 1: products of sixteen 4x4
    // blocks with ones, lane l being column l % 4 of block l / 4, so that no
    // lane's P meets another's (0 times a NaN of another row would be NaN).
    // Measured in a prefill 32768 x 13 x 48: these 337 us, adds of the unpacked P
    // 345.  (v_dot2_f32_bf16 holds up the matrix cores: four of them beside a
    // 32x32x16 product take 29 ns, four v_fma_f32 17 ns.)
    const s16x4_t ones = {0x3f80, 0x3f80, 0x3f80, 0x3f80};
    auto sum_step = [&](const u32x4_t (&pk)[NT][2], int i) __attribute__((always_inline)) {
        const int nt = i % NT, k = i / NT;
        const u32x4_t x = pk[nt][k >> 1];
        const u32x2_t h = (k & 1) ? u32x2_t{x.z, x.w} : u32x2_t{x.x, x.y};
        lsum[nt] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones, __builtin_bit_cast(s16x4_t, h), lsum[nt], 0, 0, 0);
    };
    // visible keys of a lane's row within its unit: keys k0 + .. < lim
    auto row_limit = [&](const UnitInfo& ui, int nt) __attribute__((always_inline)) {
        const int seen = ui.stream < 0 || r_stream[nt] == ui.stream ? (ui.stream < 0 ? kUnit : r_tok[nt] + 1 - ui.k0)
                                                                    : (CROSS ? r_tok[nt] - ui.k0 : 0);
        return min(ui.nk, seen);
    };
    auto mask_tile = [&](bf32x16_t& s, int lim) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 8 * (i >> 2) + (i & 3) >= lim - 4 * hi ? kNegInf : s[i];
    };
    auto mask = [&](bf32x16_t (&s)[NT], int kb, const UnitInfo& ui) __attribute__((always_inline)) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) mask_tile(s[nt], row_limit(ui, nt) - kb);
    };
    // max of element pair i (0 .. 8 NT - 1) into mx
    auto max_step = [&](float (&mx)[NT], const bf32x16_t (&s)[NT], int i) __attribute__((always_inline)) {
        const int nt = i / 8, k = 2 * (i % 8);
        mx[nt] = k == 0 ? fmaxf(s[nt][0], s[nt][1]) : fmaxf(fmaxf(mx[nt], s[nt][k]), s[nt][k + 1]);
    };
    // A row's reference max moves only when its block max exceeds it by more
    // than 8 (every p is at most 2^8, and the final ratio is exact).  Each
    // lane tests its own keys; the max over the two lanes of a row is formed
    // only when some row moves.
    auto rescale_tile = [&](float mx, int nt) __attribute__((always_inline)) {
        const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
        const float mt = fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1])) * c;
        const bool up = mt > m_ref[nt] + 8.f;
        const float alpha = up ? fast_exp2(m_ref[nt] - mt) : 1.f;
        m_ref[nt] = up ? mt : m_ref[nt];
        lsum[nt] *= alpha;
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt) o[nt][dt] *= alpha;
    };
    auto rescale = [&](const float (&mx)[NT]) __attribute__((always_inline)) {
        bool need = false;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) need |= mx[nt] * c > m_ref[nt] + 8.f;
        if (__any(need)) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) rescale_tile(mx[nt], nt);
        }
    };
    // P of element pair i (0 .. 8 NT - 1), rounded to bf16
    auto prob_step = [&](u32x4_t (&pk)[NT][2], const bf32x16_t (&s)[NT], int i) __attribute__((always_inline)) {
        const int nt = i / 8, k = i % 8;
        pk[nt][k >> 2][k & 3] = pack_bf16x2(fast_exp2(fmaf(s[nt][2 * k], c, -m_ref[nt])),
                                            fast_exp2(fmaf(s[nt][2 * k + 1], c, -m_ref[nt])));
        // keeps P in the phase that computes it: without a use there the
        // compiler sinks the exponentials into the phase that multiplies it
        if ((k & 3) == 3) asm volatile("" : "+v"(pk[nt][k >> 2]));
    };

    // The two phases of a block, in a fixed order (scheduling barriers): one
    // 32x32x16 product per step, with the vector and LDS work that fits under
    // it (up to six vector instructions are free under one product).
    // A: the next block's scores sn under this block's exponentials, this
    // block's V operands on their way.
    auto phase_a = [&](bf32x16_t (&sn)[NT], const bf32x16_t (&sc)[NT], u32x4_t (&pk)[NT][2],
                       const u32x4_t (&kf)[C::KS], u32x2_t (&vf)[4 * C::DT], const unsigned char* buf,
                       int kb) __attribute__((always_inline)) {
        constexpr int STEPS = NT * C::KS;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            score_step(sn, kf, i);
#pragma unroll
            for (int j = i * 4 * C::DT / STEPS; j < (i + 1) * 4 * C::DT / STEPS; ++j) read_v(vf, buf, kb, j);
#pragma unroll
            for (int j = i * 8 * NT / STEPS; j < (i + 1) * 8 * NT / STEPS; ++j) prob_step(pk, sc, j);
        }
    };
    // B: this block's P V products and row sums under the next block's
    // maxima, the K operands of the block after it and, with DMA, the pieces
    // of a later stage.
    auto phase_b = [&](auto dma, const u32x4_t (&pk)[NT][2], const u32x2_t (&vf)[4 * C::DT],
                       const bf32x16_t (&sn)[NT], float (&mx)[NT], u32x4_t (&kf)[C::KS], const unsigned char* nbuf,
                       int nkb, const Pending& pd) __attribute__((always_inline)) {
        constexpr int STEPS = 2 * C::DT * NT;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            pv_step(pk, vf, i);
#pragma unroll
            for (int j = i * C::KS / STEPS; j < (i + 1) * C::KS / STEPS; ++j) read_k(kf, nbuf, nkb, j);
            if constexpr (decltype(dma)::value) {
#pragma unroll
                for (int j = i * C::PPW / STEPS; j < (i + 1) * C::PPW / STEPS; ++j)
                    issue_piece(pd, j);
            }
#pragma unroll
            for (int j = i * 8 * NT / STEPS; j < (i + 1) * 8 * NT / STEPS; ++j) max_step(mx, sn, j);
#pragma unroll
            for (int j = i * 4 * NT / STEPS; j < (i + 1) * 4 * NT / STEPS; ++j) sum_step(pk, j);
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) asm volatile("" : "+v"(mx[nt]));
    };

    // B where no row of the wave sees the block (other streams' rows visible):
    // no products.
    auto phase_b_idle = [&](auto dma, const bf32x16_t (&sn)[NT], float (&mx)[NT], u32x4_t (&kf)[C::KS],
                            const unsigned char* nbuf, int nkb, const Pending& pd) __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < C::KS; ++t) read_k(kf, nbuf, nkb, t);
        if constexpr (decltype(dma)::value) issue_stage(pd);
#pragma unroll
        for (int i = 0; i < 8 * NT; ++i) max_step(mx, sn, i);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) asm volatile("" : "+v"(mx[nt]));
    };

    // A masked key has p = 0, but 0 times an infinite or NaN value is NaN, so a
    // unit's products may only meet rows that see some of it.  The pipelined
    // loop takes the wave's first nd stages: the prefix's and, where every own
    // unit belongs to the rows' one stream, those up to its first row's token,
    // of which every row sees a part.  The plain loop takes the others, tile by
    // tile and block by block, and keeps the rows that see nothing of a block as
    // they were.  With other streams' rows visible nearly every row of a wave
    // sees some of nearly every unit: the one-tile form takes them all in the
    // pipelined loop, without products where its tile sees nothing of a block,
    // and the plain loop leaves out tiles only.  (Videos of at most 64 rows, most
    // of which are one tile, keep rows apart; branches of one block stay in the
    // plain loop, which skips the unit's second one.)
    const bool others = CROSS && NT == 1 && !one && R > 64 && a.qps > 32;
    const int nd = !active ? 0
                   : others ? nst
                            : min(max(upre + (one ? ((row0 + wrow0) / a.G) % a.qps / kUnit + 1 : 0) - u0, 0), nst);
    // bit b: some row of the wave sees some of block b of the unit
    auto sees_blocks = [&](const UnitInfo& ui) __attribute__((always_inline)) {
        if (!others || ui.stream < 0) return 3;
        const int lim = row_limit(ui, 0);
        return (__any(lim > 0) ? 1 : 0) | (__any(lim > 32) ? 2 : 0);
    };

    // a unit that some row of this wave does not see whole
    auto masked = [&](const UnitInfo& ui) __attribute__((always_inline)) {
        bool m = ui.nk < kUnit;
        if (ui.stream >= 0) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) m |= row_limit(ui, nt) < kUnit;
        }
        return __any(m) != 0;
    };

    // Every wave passes one barrier per stage; behind the one of stage st,
    // stage st + 1 has landed and stage st - 1 been consumed for all of them, and
    // the slot of the latter takes stage st + 3.
    if (nst > 0) lds_barrier();  // the first three stages have landed
    if (nd > 0) {
        // Entering stage st: sa holds block 0's scores (masked, reference set),
        // kf block 1's K operands.
        bf32x16_t sa[NT], sb[NT];
        u32x4_t kf[C::KS], pk[NT][2];
        u32x2_t vf[4 * C::DT];
        float mx[NT];
        UnitInfo ui = unit(u0);
#pragma unroll
        for (int t = 0; t < C::KS; ++t) read_k(kf, slot(0), 0, t);
#pragma unroll
        for (int i = 0; i < NT * C::KS; ++i) score_step(sa, kf, i);
        bool msk = masked(ui);
        int sees = sees_blocks(ui);
        if (msk) mask(sa, 0, ui);
#pragma unroll
        for (int i = 0; i < 8 * NT; ++i) max_step(mx, sa, i);
        rescale(mx);
#pragma unroll
        for (int t = 0; t < C::KS; ++t) read_k(kf, slot(0), 32, t);
        for (int st = 0; st < nd; ++st) {
            const unsigned char* buf = slot(st);
            const unsigned char* nbuf = slot(st + 1);
            phase_a(sb, sa, pk, kf, vf, buf, 0);
            if (msk) mask(sb, 32, ui);
            const Pending pd = pending(st + 3);
            stage_barrier<C::PPW>();
            if (sees & 1) phase_b(std::true_type{}, pk, vf, sb, mx, kf, nbuf, 0, pd);
            else phase_b_idle(std::true_type{}, sb, mx, kf, nbuf, 0, pd);
            rescale(mx);
            phase_a(sa, sb, pk, kf, vf, buf, 32);
            const bool more = st + 1 < nd;
            const int saw = sees;
            if (more) {
                ui = unit(u0 + st + 1);
                msk = masked(ui);
                sees = sees_blocks(ui);
                if (msk) mask(sa, 0, ui);
            }
            if (saw & 2) phase_b(std::false_type{}, pk, vf, sa, mx, kf, nbuf, 32, pd);
            else phase_b_idle(std::false_type{}, sa, mx, kf, nbuf, 32, pd);
            if (more) rescale(mx);
        }
    }
    for (int st = nd; st < nst; ++st) {
        stage_barrier<C::PPW>();
        issue_stage(pending(st + 3));
        const unsigned char* buf = slot(st);
        const UnitInfo ui = unit(u0 + st);
        int lim[NT], most = 0;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            lim[nt] = row_limit(ui, nt);
            most = max(most, lim[nt]);
        }
        if (!active) continue;
#pragma unroll 1
        for (int kb = 0; kb < kUnit; kb += 32) {
            if (!__any(most > kb)) continue;
            u32x4_t kf[C::KS], pk[NT][2];
            u32x2_t vf[4 * C::DT];
            bf32x16_t s[NT];
            float mx[NT];
#pragma unroll
            for (int t = 0; t < C::KS; ++t) read_k(kf, buf, kb, t);
#pragma unroll
            for (int j = 0; j < 4 * C::DT; ++j) read_v(vf, buf, kb, j);
            // other streams' rows visible: both tiles at once, without the products
            // of a tile that sees nothing
            if (CROSS && (NT > 1 || R > 64)) {
#pragma unroll
                for (int i = 0; i < NT * C::KS; ++i) score_step(s, kf, i);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) mask_tile(s[nt], lim[nt] - kb);
#pragma unroll
                for (int i = 0; i < 8 * NT; ++i) max_step(mx, s, i);
                rescale(mx);
#pragma unroll
                for (int i = 0; i < 8 * NT; ++i) prob_step(pk, s, i);
#pragma unroll
                for (int i = 0; i < 4 * NT; ++i) sum_step(pk, i);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    if (!__any(lim[nt] > kb)) continue;
#pragma unroll
                    for (int i = 0; i < 2 * C::DT; ++i) pv_step(pk, vf, i * NT + nt);
                }
                continue;
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const bool sees = lim[nt] > kb;
                __builtin_amdgcn_sched_barrier(0);
                if (!__any(sees)) continue;
#pragma unroll
                for (int t = 0; t < C::KS; ++t) score_step(s, kf, t * NT + nt);
                mask_tile(s[nt], lim[nt] - kb);
#pragma unroll
                for (int i = 0; i < 8; ++i) max_step(mx, s, 8 * nt + i);
                if (__any(mx[nt] * c > m_ref[nt] + 8.f)) rescale_tile(mx[nt], nt);
#pragma unroll
                for (int i = 0; i < 8; ++i) prob_step(pk, s, 8 * nt + i);
#pragma unroll
                for (int i = 0; i < 4; ++i) sum_step(pk, i * NT + nt);
#pragma unroll
                for (int dt = 0; dt < C::DT; ++dt) {
                    bf32x16_t x = branch_mfma(v_op(vf, 0, dt), pk[nt][0], o[nt][dt]);
                    x = branch_mfma(v_op(vf, 1, dt), pk[nt][1], x);
#pragma unroll
                    for (int i = 0; i < 16; ++i) o[nt][dt][i] = sees ? x[i] : o[nt][dt][i];
                }
            }
        }
    }
    wait_vmcnt<0>();  // no DMA into the LDS outlives the work-group

    if (!active) return;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const float l = lsum[nt][0] + __shfl_xor(lsum[nt][0], 32);  // both lanes of the row
        const int r = wrow0 + 32 * nt + l32;
        if (r >= nrows) continue;
        const long qr = row_qrow(a, vi, g, row0 + r);
        const long sl = qr * a.max_chunks + c_idx;
        const float inv = l > 0.f ? 1.f / l : 0.f;
        // one slot: the row's result itself, an ended stream giving 0 and -inf
        const bool single = a.max_chunks == 1;
        const bool ended = single && a.event_lens[vi.e0 + r_stream[nt]] <= 0;
        const uint64_t obase = sgpr_base(a.out), pbase = sgpr_base(a.part_o);
        uint16_t* dst = reinterpret_cast<uint16_t*>(single ? obase + 2 * qr * D : pbase + 2 * sl * D);
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint2 val = make_uint2(pack_bf16x2(o[nt][dt][4 * k] * inv, o[nt][dt][4 * k + 1] * inv),
                                             pack_bf16x2(o[nt][dt][4 * k + 2] * inv, o[nt][dt][4 * k + 3] * inv));
                *reinterpret_cast<uint2*>(dst + 32 * dt + 8 * k + 4 * hi) = ended ? make_uint2(0u, 0u) : val;
            }
        if (hi == 0) {
            if (!single) *reinterpret_cast<float2*>(a.part_ml + 2 * sl) = make_float2(m_ref[nt], l);
            else if (a.lse) a.lse[qr] = ended ? kNegInf : kLn2 * (m_ref[nt] + __log2f(l));
        }
    }
}

}  // namespace pdec
