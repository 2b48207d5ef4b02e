// Backward pass of event-factorized attention over whole branches (the
// training form of the §3.4 mask: query token j of branch e sees every prefix
// token and its own rows 0 .. min(j, n_e - 1)), for one video.
//
// With the forward's O and lse and the incoming dO, for a live query row i
// and a key k it sees:
//   p_ik = 2^(c <q_i, k_k> - lse_i log2 e),  D_i = <dO_i, O_i>,
//   ds_ik = p_ik (<dO_i, v_k> - D_i),
//   dq_i = tau sum_k ds_ik k_k,  dk_k = tau sum_i ds_ik q_i,  dv_k = sum_i p_ik dO_i.
// Rows of ended streams (n_e <= 0) have no output and add nothing.
//
// Passes, on v_mfma_f32_32x32x16_bf16 (1 only where 2 runs before 3, which
// otherwise leaves D itself):
//  1. per row: D_i, a mark for the rows of ended streams (bwd_drow_word);
//  2. dk, dv: a work-group holds 128 keys of one kv head (32 per wave, K and V
//     as B operands in registers) and walks the rows that see them in stages
//     of 64.  S = Q K^T and dP = dO V^T give a lane one key and 16 rows of a
//     32-row tile, which is the A operand (keys x rows) of dV += P^T dO and
//     dK += dS^T Q; their B operands (rows x d) are transposing LDS reads of
//     the same stage;
//  3. dq: a work-group holds 256 rows of one kv head (64 per wave, Q and dO as
//     B operands in registers) and walks 64-key units, as the forward does.
//     S^T = K Q^T and dP^T = V dO^T give a lane one row and 16 keys, the B
//     operand of dQ^T += K^T dS^T, whose A operand is the transposing read;
//  4. where 2 is split over rows or 3 over keys to fill the chip, the sum of
//     the splits, in a fixed order.  Only one of the two is split: it runs
//     first, its splits after the first in the output buffers that the other
//     pass writes afterwards, so the workspace is the row values alone.
// P and dS meet the matrix cores in bf16 (as the forward's P does); every sum
// is float32.  Every output element is written, so nothing needs clearing, and
// repeated calls agree bit for bit.
//
// What bounds 2 and 3 and why these tiles: dense contractions, so the matrix
// cores should.  32 keys (or 64 rows) per wave keep the LDS reads at or below
// the products' time, which 16 did not, and the 32x32x16 product runs at the
// full rate where the 16x16x16 one of the earlier form ran at half.  One wave
// per SIMD holds the operands and sums in 512 registers; the vector work of
// one 32-row tile is issued under the products of the other.
#pragma once

#include "kernel_branch.h"

namespace pdec {

constexpr float kLog2eF = 1.44269504088896340736f;

struct BwdArgs {
    const uint16_t* q;     // [E, N, H_q, D]
    const uint16_t* kp;    // [Lmax, H_kv, D]
    const uint16_t* vp;
    const uint16_t* ke;    // [E, cap, H_kv, D]
    const uint16_t* ve;
    const int32_t* event_lens;  // [E]
    const int32_t* prefix_len;  // [1], <= Lmax
    const uint16_t* out;   // [E, N, H_q, D]
    const float* lse;      // [E, N, H_q]
    const uint16_t* dout;  // [E, N, H_q, D]
    float* drow;           // [E, N, H_q]: D, or the mark of an ended stream's row
    float* dq;             // [E, N, H_q, D]
    float* dkp;            // [Lmax, H_kv, D]
    float* dvp;
    float* dke;            // [E, cap, H_kv, D]
    float* dve;
    // Splits after the first of the split pass: split k of dk, dv at part0 +
    // (2 k - 2) and (2 k - 1) tensors; split k of dq in part0, then part1,
    // part_n tensors in each.
    float* part0;
    float* part1;
    long part_n;
    long part_elems;       // elements of one split tensor
    int row_splits, key_splits;
    int E, N, H_q, H_kv, G, cap, Lmax;
    int R;                 // rows per kv head: E N G
    int unit_per_chunk;    // 64-key units per key split
    float c;    // tau * log2(e)
    float tau;  // softmax scale
};

// Row r (0 .. R - 1) of kv head g: stream r / (N G), token (r / G) % N, head
// g G + r % G; its index in q, out, dout and lse.
__device__ inline long bwd_qrow(const BwdArgs& a, int g, int r)
{
    return (long)(r / a.G) * a.H_q + g * a.G + r % a.G;
}

// Row values between the passes: D, or kEndedRow for the row of an ended
// stream.  The mark is a NaN that no D is: a live row may have any D, infinite
// or NaN, and its NaN is stored as the plain quiet one.
constexpr uint32_t kEndedRow = 0x7fc00001u;
__device__ inline float bwd_drow_word(float D, bool live)
{
    const uint32_t u = __float_as_uint(D);
    return __uint_as_float(!live ? kEndedRow : (u & 0x7fffffffu) > 0x7f800000u ? 0x7fc00000u : u);
}

// One float per lane straight into LDS, lane l's at lds_base + 4 l; as
// dma_16B_m0 otherwise.
__device__ inline void dma_4B_m0(const void* base, uint32_t off, uint32_t lds_base, uint64_t lanes)
{
    const uint64_t sb = sgpr_base(base);
    asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 exec, %3\n\tglobal_load_lds_dword %1, %2\n\ts_mov_b64 exec, -1" :
                 : "s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(off), "s"(sb),
                   "s"(sgpr_base(reinterpret_cast<const void*>(lanes)))
                 : "memory");
}

// Permutation of the 16-byte chunks of staged row `row` (chunk ch sits at
// ch ^ swizzle): a staged tile is read both by rows (16 rows of one chunk per
// LDS phase) and transposed (four rows of four chunks), so 16 rows take 16
// different permutations and four consecutive ones differ in the chunk's
// upper bits.
template <int D>
__device__ inline int bwd_swz(int row)
{
    return D == 128 ? 4 * (row & 3) + ((row >> 2) & 3) : 4 * ((row >> 1) & 1) + ((row >> 2) & 3);
}

// Offsets of the operand reads of a staged 32-row tile: by rows, step t (row
// l % 32, chunk 2 t + l / 32) at row ^ 32 t; transposed, rows 16 s + 8 r +
// 4 (l / 32) .. +3 of d 32 dt + l % 32, at (tr[dt] ^ 32 r) + (16 s + 8 r) rows.
template <int D>
struct BwdOffsets {
    int row;
    int tr[D / 32];
    __device__ explicit BwdOffsets(int lane)
    {
        row = (lane & 31) * 2 * D + 16 * ((lane >> 5) ^ bwd_swz<D>(lane & 31));
        const int q = lane >> 4, i = lane & 15, r = 4 * (q >> 1) + (i >> 2);
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
            tr[dt] = r * 2 * D + 16 * ((4 * dt + 2 * (q & 1) + ((i & 3) >> 1)) ^ bwd_swz<D>(r)) + 8 * (i & 1);
    }
};

template <int D>
__device__ inline u32x4_t bwd_read_row(const unsigned char* tile, const BwdOffsets<D>& off, int t)
{
    return *reinterpret_cast<const u32x4_t*>(tile + (off.row ^ (32 * t)));
}

template <int D>
__device__ inline u32x4_t bwd_read_tr(const unsigned char* tile, const BwdOffsets<D>& off, int s, int dt)
{
    typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;
    const unsigned char* p = tile + 16 * s * 2 * D;
    const u32x2_t x0 = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(p + off.tr[dt])));
    const u32x2_t x1 = __builtin_bit_cast(
        u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(p + 8 * 2 * D + (off.tr[dt] ^ 32))));
    return u32x4_t{x0.x, x0.y, x1.x, x1.y};
}

// ---- 1: D_i = <dO_i, O_i> ----
template <int D>
__global__ __launch_bounds__(256) void bwd_drow_kernel(BwdArgs a)
{
    constexpr int PER = D / 16;  // elements per lane, 16 lanes per row
    const long rows = (long)a.E * a.N * a.H_q;
    const long i = (long)wg_id() * 16 + wi_id() / 16;
    const int l = wi_id() % 16;
    if (i >= rows) return;
    float s = 0.f;
    const uint16_t* o = a.out + i * D + PER * l;
    const uint16_t* d = a.dout + i * D + PER * l;
#pragma unroll
    for (int k = 0; k < PER; ++k)
        s = fmaf(__uint_as_float((uint32_t)o[k] << 16), __uint_as_float((uint32_t)d[k] << 16), s);
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) s += __shfl_xor(s, off);
    const bool live = a.event_lens[i / ((long)a.N * a.H_q)] > 0;
    if (l == 0) a.drow[i] = bwd_drow_word(s, live);
}

// ---- 2: dk, dv per 128 keys ----
template <int D>
__global__ __launch_bounds__(256) void bwd_dkdv_kernel(BwdArgs a)
{
    constexpr int ROWB = 2 * D, CH = D / 8, KS = D / 16, DT = D / 32;
    constexpr int NSTAGE = 4, TILE = 64 * ROWB, STAGE = 2 * TILE;  // Q rows, then dO rows
    constexpr int KPI = 1024 / ROWB, PPW = STAGE / 1024 / 4;       // rows per piece, pieces per wave
    __shared__ __attribute__((aligned(1024))) unsigned char lds[NSTAGE * STAGE];
    __shared__ __attribute__((aligned(16))) float rowv[NSTAGE][2][64];  // l2, D

    const int w = __builtin_amdgcn_readfirstlane(wi_id() >> 6);
    const int lane = wi_id() & 63, l32 = lane & 31, hi = lane >> 5;
    const int g = (int)__builtin_amdgcn_workgroup_id_y(), split = (int)__builtin_amdgcn_workgroup_id_z();
    const int UP = (a.Lmax + 127) / 128, UPS = (a.cap + 127) / 128;
    const int u = wg_id();
    const int L = min(max(a.prefix_len[0], 0), a.Lmax);
    const int NG = a.N * a.G;

    // keys [k0, kend) of the prefix or of stream own's cache, nvalid of them
    // holding rows; query rows [r_begin, r_end) see some of them
    const bool prefix = u < UP;
    const int own = prefix ? 0 : (u - UP) / UPS;
    const int k0 = 128 * (prefix ? u : (u - UP) % UPS);
    const int kend = min(k0 + 128, prefix ? a.Lmax : a.cap);
    const int nf = a.event_lens[own];
    const int nvalid = max(0, min(kend, prefix ? L : nf) - k0);
    int r_begin = prefix ? 0 : own * NG + min(k0, a.N) * a.G;
    const int r_end = prefix ? a.R : (own + 1) * NG;
    // the row splits cut the prefix's rows, or a pure causal sequence's
    const bool cut = prefix || a.Lmax == 0;
    if (!cut && split > 0) return;
    int nst = nvalid > 0 ? (r_end - r_begin + 63) / 64 : 0;
    if (cut && a.row_splits > 1) {
        const int per = (nst + a.row_splits - 1) / a.row_splits;
        r_begin += 64 * per * split;
        nst = max(0, min(per, nst - per * split));
    }
    nst = __builtin_amdgcn_readfirstlane(nst);
    // a key's rows start at rmin: own row t is seen by tokens j >= t
    const int rmin = prefix ? 0 : own * NG + (k0 + 32 * w + l32) * a.G;
    // stages whose rows see none of the wave's keys: left out, so that what
    // they hold (0 times an infinite dO is NaN) stays with the keys they see
    const int skip = prefix ? 0 : max(own * NG + (k0 + 32 * w) * a.G - r_begin, 0) / 64;

    // ---- DMA of one stage: waves 0, 1 Q rows, waves 2, 3 dO rows; waves 0, 2 also a half of lse, waves 1, 3 of D ----
    const bool w_is_d = w >= 2;
    const uint64_t qb = sgpr_base(a.q), db = sgpr_base(a.dout);
    const uint64_t src = w_is_d ? db : qb;
    const uint64_t lseb = sgpr_base(a.lse), drowb = sgpr_base(a.drow);
    const uint64_t rvb = (w & 1) == 0 ? lseb : drowb;
    const int rv0 = 32 * (w >> 1);  // first row value of the wave; lanes 0 .. 31 load
    const int row0 = (w & 1) * PPW * KPI + lane / CH;
    uint32_t choff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) choff[i] = 16u * ((lane % CH) ^ bwd_swz<D>(row0 + i * KPI));
    const float inv_g = 1.f / (float)a.G;
    const uint32_t lds0 = lds_u32(lds) + (w_is_d ? TILE : 0) + (w & 1) * PPW * 1024;
    auto issue_stage = [&](int st) __attribute__((always_inline)) {
        const uint64_t lanes = ring_lanes(st, nst);
        const int rb = r_begin + 64 * min(st, nst - 1);
        const int t0 = rb / a.G, h0 = rb - t0 * a.G;
        const uint64_t base = src + 2 * D * ((long)t0 * a.H_q + g * a.G);
        const uint32_t dst = lds0 + (st % NSTAGE) * STAGE;
#pragma unroll
        for (int i = 0; i < PPW; ++i) {
            // rows past the last re-read it (see row_values)
            const int n = h0 + min(row0 + i * KPI, r_end - 1 - rb);
            const int t = (int)(((float)n + 0.5f) * inv_g);  // n / G: n < G + 64
            const uint32_t off = (uint32_t)(t * a.H_q + n - t * a.G) * (2 * D) + choff[i & 3];
            dma_16B_m0(reinterpret_cast<const void*>(base), off, dst + 1024 * i, lanes);
        }
        const int n = h0 + min(rv0 + lane, r_end - 1 - rb);
        const int t = (int)(((float)n + 0.5f) * inv_g);
        dma_4B_m0(reinterpret_cast<const void*>(rvb + 4 * ((long)t0 * a.H_q + g * a.G)), 4 * (t * a.H_q + n - t * a.G),
                  lds_u32(rowv[st % NSTAGE][w & 1] + rv0), lanes & 0xffffffffull);
    };

    // The row values of a landed stage made ready, by wave 0, one barrier
    // before they are read: lse in base 2, infinite (so that p = 0) for rows
    // of ended streams and rows past the last, whose D becomes 0.
    auto row_values = [&](int st) __attribute__((always_inline)) {
        float* const v = rowv[st % NSTAGE][0] + lane;
        const float l = v[0], dr = v[64];
        const bool none = __float_as_uint(dr) == kEndedRow || r_begin + 64 * st + lane >= r_end;
        v[0] = none ? __builtin_inff() : l * kLog2eF;
        v[64] = none ? 0.f : dr;
    };

    // this wave's keys as B operands
    u32x4_t kB[KS], vB[KS];
    {
        const int key = min(k0 + 32 * w + l32, max(k0 + nvalid - 1, 0));  // keys past the last repeat it; not stored
        const long base = ((prefix ? (long)key : (long)own * a.cap + key) * a.H_kv + g) * D + 8 * hi;
        const uint64_t kb = prefix ? sgpr_base(a.kp) : sgpr_base(a.ke), vb = prefix ? sgpr_base(a.vp) : sgpr_base(a.ve);
#pragma unroll
        for (int t = 0; t < KS; ++t) {
            kB[t] = vB[t] = u32x4_t{0u, 0u, 0u, 0u};
            if (nvalid > 0) {
                kB[t] = *reinterpret_cast<const u32x4_t*>(kb + 2 * (base + 16 * t));
                vB[t] = *reinterpret_cast<const u32x4_t*>(vb + 2 * (base + 16 * t));
            }
        }
    }
    if (nst > 0) {
#pragma unroll
        for (int st = 0; st < NSTAGE - 1; ++st) issue_stage(st);
    }
    wait_vmcnt<0>();  // plain loads and DMA complete in no order relative to each other
#pragma unroll
    for (int t = 0; t < KS; ++t) asm volatile("" : "+a"(kB[t]), "+a"(vB[t]));
    bf32x16_t dk[DT], dv[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) dk[dt][i] = dv[dt][i] = 0.f;
    const BwdOffsets<D> off(lane);

    lds_barrier();  // every wave's pieces of the first stages have landed
    if (w == 0 && nst > 0) row_values(0);
    auto enter = [&](int st) __attribute__((always_inline)) {
        // stage st + 1 has landed too
        stage_barrier<PPW + 1>();
        issue_stage(st + 3);
        if (w == 0 && st + 1 < nst) row_values(st + 1);
    };
    int st = 0;
    for (; st < min(skip, nst); ++st) enter(st);
    for (; st < nst; ++st) {
        enter(st);
        const unsigned char* qt = lds + (st % NSTAGE) * STAGE;
        const unsigned char* dt_ = qt + TILE;
        const int lo0 = rmin - (r_begin + 64 * st) - 4 * hi;
        bf32x16_t s[2], dp[2];
        u32x4_t p[2][2], ds[2][2];
        auto scores = [&](int b) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 16; ++i) s[b][i] = dp[b][i] = 0.f;
#pragma unroll
            for (int t = 0; t < KS; ++t) {
                s[b] = branch_mfma(bwd_read_row<D>(qt + 32 * b * ROWB, off, t), kB[t], s[b]);
                dp[b] = branch_mfma(bwd_read_row<D>(dt_ + 32 * b * ROWB, off, t), vB[t], dp[b]);
            }
        };
        auto soft = [&](int b) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const f32x4_t l2 = *reinterpret_cast<const f32x4_t*>(&rowv[st % NSTAGE][0][32 * b + 8 * k + 4 * hi]);
                const f32x4_t dr = *reinterpret_cast<const f32x4_t*>(&rowv[st % NSTAGE][1][32 * b + 8 * k + 4 * hi]);
                float pe[4], de[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float x = fmaf(s[b][4 * k + j], a.c, -l2[j]);
                    pe[j] = fast_exp2(32 * b + 8 * k + j >= lo0 ? x : kNegInf);
                    de[j] = pe[j] * (dp[b][4 * k + j] - dr[j]);
                }
                p[b][k >> 1][2 * (k & 1)] = pack_bf16x2(pe[0], pe[1]);
                p[b][k >> 1][2 * (k & 1) + 1] = pack_bf16x2(pe[2], pe[3]);
                ds[b][k >> 1][2 * (k & 1)] = pack_bf16x2(de[0], de[1]);
                ds[b][k >> 1][2 * (k & 1) + 1] = pack_bf16x2(de[2], de[3]);
                if (k & 1) asm volatile("" : "+v"(p[b][k >> 1]), "+v"(ds[b][k >> 1]));  // computed in this phase
            }
        };
        auto grads = [&](int b) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    dv[dt] = branch_mfma(p[b][q], bwd_read_tr<D>(dt_ + 32 * b * ROWB, off, q, dt), dv[dt]);
                    dk[dt] = branch_mfma(ds[b][q], bwd_read_tr<D>(qt + 32 * b * ROWB, off, q, dt), dk[dt]);
                }
        };
        scores(0);
        __builtin_amdgcn_sched_barrier(0);
        scores(1);
        soft(0);
        __builtin_amdgcn_sched_barrier(0);
        grads(0);
        soft(1);
        __builtin_amdgcn_sched_barrier(0);
        grads(1);
    }
    wait_vmcnt<0>();  // no DMA into the LDS outlives the work-group

    // lane: d 32 dt + l % 32 of keys 32 w + 8 (i / 4) + 4 (l / 32) + i % 4; every key of the tile is written
    const bool later = cut && split > 0;
    float* const dkb = later ? a.part0 + (2 * split - 2) * a.part_elems : prefix ? a.dkp : a.dke;
    float* const dvb = later ? a.part0 + (2 * split - 1) * a.part_elems : prefix ? a.dvp : a.dve;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int kk = 32 * w + 8 * (i >> 2) + 4 * hi + (i & 3);
        if (k0 + kk >= kend) continue;
        const long base = ((prefix ? 0L : (long)own * a.cap) + k0 + kk) * a.H_kv * D + (long)g * D + l32;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            dkb[base + 32 * dt] = kk < nvalid ? a.tau * dk[dt][i] : 0.f;
            dvb[base + 32 * dt] = kk < nvalid ? dv[dt][i] : 0.f;
        }
    }
}

// ---- 3: dq per 256 rows ----
template <int D>
__global__ __launch_bounds__(256) void bwd_dq_kernel(BwdArgs a)
{
    constexpr int ROWB = 2 * D, CH = D / 8, KS = D / 16, DT = D / 32, NT = 2;
    constexpr int NSTAGE = 4, TILE = kUnit * ROWB, STAGE = 2 * TILE;  // K, then V
    constexpr int KPI = 1024 / ROWB, PPW = STAGE / 1024 / 4;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[NSTAGE * STAGE];

    const int w = __builtin_amdgcn_readfirstlane(wi_id() >> 6);
    const int lane = wi_id() & 63, l32 = lane & 31, hi = lane >> 5;
    const int g = (int)__builtin_amdgcn_workgroup_id_y(), split = (int)__builtin_amdgcn_workgroup_id_z();
    const int NG = a.N * a.G;
    const int row0 = 256 * wg_id(), nrows = min(256, a.R - row0);
    const int L = min(max(a.prefix_len[0], 0), a.Lmax), upre = (L + kUnit - 1) / kUnit;
    // the group's key sequence: the prefix units, then those of its rows'
    // streams, each up to the group's largest token of it; one stream's
    // units or, in turn, those of several
    const int f_lo = row0 / NG, f_hi = (row0 + nrows - 1) / NG;
    const int tok_last = ((row0 + nrows - 1) / a.G) % a.N;
    auto seen = [&](int f) __attribute__((always_inline)) {
        return min(max(a.event_lens[f], 0), f == f_hi ? tok_last + 1 : a.N);
    };
    int own = 0;
    for (int f = f_lo; f <= f_hi; ++f) own += (seen(f) + kUnit - 1) / kUnit;
    const int total = upre + own;
    const int u0 = min(split * a.unit_per_chunk, total);
    const int u1 = split == a.key_splits - 1 ? total : min(u0 + a.unit_per_chunk, total);
    const int nst = __builtin_amdgcn_readfirstlane(u1 - u0);
    // unit u, which is at or after the last one asked for through this cursor
    struct Cursor { int f, start; };
    auto unit = [&](Cursor& cu, int u) __attribute__((always_inline)) {
        int stream = -1, t0 = u * kUnit, n = L;
        if (u >= upre) {
            int nf = seen(cu.f);
            while (cu.f < f_hi && u - upre >= cu.start + (nf + kUnit - 1) / kUnit) {
                cu.start += (nf + kUnit - 1) / kUnit;
                nf = seen(++cu.f);
            }
            stream = cu.f;
            t0 = (u - upre - cu.start) * kUnit;
            n = nf;
        }
        const long row = stream < 0 ? (long)t0 : (long)stream * a.cap + t0;
        return UnitInfo{(row * a.H_kv + g) * D, min(kUnit, n - t0), stream, t0};
    };
    Cursor dma_at{f_lo, 0}, at{f_lo, 0};

    const bool w_is_v = w >= 2;
    const uint64_t kpb = sgpr_base(a.kp), vpb = sgpr_base(a.vp), keb = sgpr_base(a.ke), veb = sgpr_base(a.ve);
    const uint64_t pre = w_is_v ? vpb : kpb, evt_pre = (w_is_v ? veb : keb) - pre;
    const uint32_t strideB = (uint32_t)a.H_kv * ROWB;
    const int key0 = (w & 1) * PPW * KPI + lane / CH;
    uint32_t choff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) choff[i] = 16u * ((lane % CH) ^ bwd_swz<D>(key0 + i * KPI));
    const uint32_t lds0 = lds_u32(lds) + (w_is_v ? TILE : 0) + (w & 1) * PPW * 1024;
    auto issue_stage = [&](int st) __attribute__((always_inline)) {
        const uint64_t lanes = ring_lanes(st, nst);
        const UnitInfo ui = unit(dma_at, u0 + min(st, nst - 1));
        const void* base = reinterpret_cast<const void*>(pre + (ui.stream < 0 ? 0 : evt_pre) + 2 * ui.key_off);
#pragma unroll
        for (int i = 0; i < PPW; ++i)  // keys past the last valid one re-read it (they are masked)
            dma_16B_m0(base, (uint32_t)min(key0 + i * KPI, ui.nk - 1) * strideB + choff[i & 3],
                       lds0 + (st % NSTAGE) * STAGE + 1024 * i, lanes);
    };

    // this lane's rows: 32 nt + l % 32 of the wave's 64
    const bool active = 64 * w < nrows;
    int r_tok[NT], r_stream[NT];
    float l2[NT], dr[NT];
    u32x4_t qB[NT][KS], dB[NT][KS];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int r = row0 + min(64 * w + 32 * nt + l32, nrows - 1);  // rows past the last repeat it; not stored
        r_stream[nt] = r / NG;
        r_tok[nt] = (r / a.G) % a.N;
        const long row = bwd_qrow(a, g, r), qr = row * D + 8 * hi;
        const bool live = a.event_lens[r_stream[nt]] > 0;
        l2[nt] = live ? a.lse[row] * kLog2eF : __builtin_inff();
        dr[nt] = 0.f;
#pragma unroll
        for (int t = 0; t < KS; ++t) {
            qB[nt][t] = *reinterpret_cast<const u32x4_t*>(a.q + qr + 16 * t);
            dB[nt][t] = *reinterpret_cast<const u32x4_t*>(a.dout + qr + 16 * t);
        }
        // D_i: the lane holds half of the row's elements, the lane 32 on the others
        float sum = 0.f;
#pragma unroll
        for (int t = 0; t < KS; ++t) {
            const u32x4_t x = *reinterpret_cast<const u32x4_t*>(a.out + qr + 16 * t);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                sum = fmaf(__uint_as_float(x[k] << 16), __uint_as_float(dB[nt][t][k] << 16), sum);
                sum = fmaf(__uint_as_float(x[k] & 0xffff0000u), __uint_as_float(dB[nt][t][k] & 0xffff0000u), sum);
            }
        }
        sum += __shfl_xor(sum, 32);
        if (live) dr[nt] = sum;
        if (a.row_splits == 1 && split == 0 && hi == 0 && 64 * w + 32 * nt + l32 < nrows)
            a.drow[row] = bwd_drow_word(sum, live);  // for the dk, dv pass, which runs next
    }
    if (nst > 0) {
#pragma unroll
        for (int st = 0; st < NSTAGE - 1; ++st) issue_stage(st);
    }
    wait_vmcnt<0>();  // plain loads and DMA complete in no order relative to each other
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int t = 0; t < KS; ++t) asm volatile("" : "+a"(qB[nt][t]), "+a"(dB[nt][t]));
    bf32x16_t acc[NT][DT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[nt][dt][i] = 0.f;
    const BwdOffsets<D> off(lane);

    for (int st = 0; st < nst; ++st) {
        stage_barrier<2 * PPW>();
        issue_stage(st + 3);
        const UnitInfo ui = unit(at, u0 + st);
        int lim[NT];  // visible keys of the lane's rows
        bool any = false;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            lim[nt] = min(ui.nk, ui.stream < 0 ? kUnit : r_stream[nt] == ui.stream ? r_tok[nt] + 1 - ui.k0 : 0);
            any |= lim[nt] > 0;
        }
        if (!active || !__any(any)) continue;
        const unsigned char* kt = lds + (st % NSTAGE) * STAGE;
        const unsigned char* vt = kt + TILE;
#pragma unroll 1
        for (int kb = 0; kb < kUnit; kb += 32) {
            const unsigned char* kr = kt + kb * ROWB;
            const unsigned char* vr = vt + kb * ROWB;
            u32x4_t kf[KS], vf[KS], ds[NT][2];
            bf32x16_t s[NT], dp[NT];
#pragma unroll
            for (int t = 0; t < KS; ++t) {
                kf[t] = bwd_read_row<D>(kr, off, t);
                vf[t] = bwd_read_row<D>(vr, off, t);
            }
            auto scores = [&](int nt) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < 16; ++i) s[nt][i] = dp[nt][i] = 0.f;
#pragma unroll
                for (int t = 0; t < KS; ++t) {
                    s[nt] = branch_mfma(kf[t], qB[nt][t], s[nt]);
                    dp[nt] = branch_mfma(vf[t], dB[nt][t], dp[nt]);
                }
            };
            auto soft = [&](int nt) __attribute__((always_inline)) {
                const int lm = lim[nt] - kb - 4 * hi;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    float de[2];
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const int i = 2 * k + j;
                        const float x = fmaf(s[nt][i], a.c, -l2[nt]);
                        de[j] = fast_exp2(8 * (i >> 2) + (i & 3) < lm ? x : kNegInf) * (dp[nt][i] - dr[nt]);
                    }
                    ds[nt][k >> 2][k & 3] = pack_bf16x2(de[0], de[1]);
                    if ((k & 3) == 3) asm volatile("" : "+v"(ds[nt][k >> 2]));  // computed in this phase
                }
            };
            auto grads = [&](int nt) __attribute__((always_inline)) {
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt)
                        acc[nt][dt] = branch_mfma(bwd_read_tr<D>(kr, off, q, dt), ds[nt][q], acc[nt][dt]);
            };
            scores(0);
            __builtin_amdgcn_sched_barrier(0);
            scores(1);
            soft(0);
            __builtin_amdgcn_sched_barrier(0);
            grads(0);
            soft(1);
            __builtin_amdgcn_sched_barrier(0);
            grads(1);
        }
    }
    wait_vmcnt<0>();  // no DMA into the LDS outlives the work-group

    if (!active) return;
    // lane: row 32 nt + l % 32, d 32 dt + 8 (i / 4) + 4 (l / 32) + i % 4
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int r = 64 * w + 32 * nt + l32;
        if (r >= nrows) continue;
        float* const base = split == 0 ? a.dq
                            : split <= a.part_n ? a.part0 + (split - 1) * a.part_elems
                                                : a.part1 + (split - 1 - a.part_n) * a.part_elems;
        float* dst = base + bwd_qrow(a, g, row0 + r) * D + 4 * hi;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                *reinterpret_cast<f32x4_t*>(dst + 32 * dt + 8 * k) =
                    f32x4_t{a.tau * acc[nt][dt][4 * k], a.tau * acc[nt][dt][4 * k + 1], a.tau * acc[nt][dt][4 * k + 2],
                            a.tau * acc[nt][dt][4 * k + 3]};
    }
}

// ---- 4: out += its later splits, in order; n4 float4 per tensor ----
// y picks the tensor: out0, whose split k is float4 tensor (k - 1) step of
// part0 (past part_n of them, of part1), or out1, each one tensor further on.
__global__ __launch_bounds__(256) void bwd_sum_kernel(f32x4_t* out0, f32x4_t* out1, const f32x4_t* part0,
                                                      const f32x4_t* part1, long n4, int step, int part_n, int splits)
{
    const long i = (long)wg_id() * 256 + wi_id();
    if (i >= n4) return;
    const int y = (int)__builtin_amdgcn_workgroup_id_y();
    f32x4_t* const out = y > 0 ? out1 : out0;
    f32x4_t s = out[i];
    for (int k = 1; k < splits; ++k) {
        const f32x4_t* p = k <= part_n ? part0 + (long)(k - 1) * step * n4 : part1 + (long)(k - 1 - part_n) * step * n4;
        s += p[y * n4 + i];
    }
    out[i] = s;
}

}  // namespace pdec
