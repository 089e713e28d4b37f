// Prompt processing for gfx950: the forward over all P prompt rows at once.
//
// Paper, Section 3.1 "Parallel Decoding", step 1, and the first lines of
// Algorithm 1: before any drafting the LLM reads the prompt once, which fills
// the (k, v) cache and yields the first generated token.  With hundreds of
// rows the GEMMs are bound by the matrix cores, not by weight streaming, so
// they get a form of their own: every wave owns a 16 TN-feature x 64-row output
// tile, a weight fragment meets 4 row groups (each as hi and lo term) instead
// of one, and the eight waves of a block share their fragments through LDS.
//
// Shared with the verification step: the packed weights (MFMA-fragment order,
// weights as the A operand, activations as the B operand, so the fused
// epilogues find rotary and gate/up partners in lane ^ 32), the split-bf16
// activation operand, and the cache layout.
//
// Rows are indexed by page-aligned position: row m is absolute position
// (L & ~15) + m, where L is the cache length before the call, so a 16-row
// group is exactly one cache page and all 16 tokens of a page are written by
// one wave.  Rows in front of L (first group) or behind L + P (last group) are
// computed on zeros / leftovers and never stored.
//
// Activation operand of a GEMM with K = 32 * nks columns:
//   Xq[row group][k-step][hi|lo][lane = 16 * kg + (m & 15)][8]   bf16,
// lane holding columns 32 ks + 8 kg .. + 8 of row m: the B fragment of
// v_mfma_f32_16x16x32_bf16, loaded with one coalesced 1 KiB read.
#pragma once
#include <utility>

#include "anpd_fast.h"

namespace anpd {

constexpr int kPgThreads = 512;       // GEMM block: 8 waves, 4 (features) x 2 (rows); half of it in the narrow form
constexpr int kPfTM = 4;              // row groups per wave
constexpr int kPgSplit = 4;           // K splits of the residual GEMMs

struct PrefillArgs {
    const uint4 *Wp;      // packed weights [n_tiles][nks][64]
    const uint4 *Xq;      // activation operand [G][nks][2][64]
    int nks, n_tiles, G;
    int tile0, g0;        // first tile, first row group wanted (the last layer's rows in front of it feed nothing)
    int L, P;             // cache length before the call, prompt rows
    int S;                // K splits (1 except RESIDUAL)
    // RESIDUAL
    float *part;          // partial products fp32 [S][16 G][d]
    int d;
    // GATE_UP
    bf16_t *out;          // operand of the down projection
    int out_nks;
    // QKV
    bf16_t *qp;           // query operand [head][G][head_dim / 32][2][64][8]
    bf16_t *pool;
    const int32_t *page_table;
    const float2 *rope;
    int layer, n_layers, n_heads, head_dim;
    int n_kv_heads;
};

// Blocks are dealt to the 8 XCDs in turn, and each XCD has its own L2.  Give XCD x a contiguous
// range of the (weights, rows) order, so that the blocks sharing a weight range, and the row
// blocks they all stream in step, meet in one L2 instead of being fetched into several.
// (Without a branch: behind one, the compiler requests the other arguments only when the grid's size is there, a round trip later.  By rocprofv3,
// d 1536, QKV / O and down / gate/up of 16 rows 8.3 -> 8.15, 5.6 -> 5.25, 8.8 -> 8.55 us, of 32 10.5 -> 10.1, 6.3 -> 6.1, 10.9 -> 10.5.)
__device__ __forceinline__ int xcd_order(int block, int n_blocks)
{
    const int xcd = block % 8, rem = n_blocks % 8;
    return xcd * (n_blocks / 8) + (xcd < rem ? xcd : rem) + block / 8;
}

__host__ __device__ __forceinline__ size_t xq_offset(int nks, int m, int k, int lo)
{
    return ((((size_t)(m >> 4) * nks + (k >> 5)) * 2 + lo) * 64 + (size_t)((k >> 3) & 3) * 16 + (m & 15)) * 8 + (k & 7);
}

// two floats rounded to bf16 (nearest even) side by side, one instruction
__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 b16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){a, b}, b16x2));
}

// the rests of a and b behind their bf16 halves `hi`, rounded to bf16
__device__ __forceinline__ uint32_t pack_lo(float a, float b, uint32_t hi)
{
    return pack_bf16(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xffff0000u));
}

// four consecutive columns k .. k + 3 (k % 4 == 0) of row m, as hi and lo terms
__device__ __forceinline__ void xq_store4(bf16_t *xq, int nks, int m, int k, f32x4 v)
{
    const uint2 hi = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
    *reinterpret_cast<uint2 *>(xq + xq_offset(nks, m, k, 0)) = hi;
    *reinterpret_cast<uint2 *>(xq + xq_offset(nks, m, k, 1)) = make_uint2(pack_lo(v[0], v[1], hi.x), pack_lo(v[2], v[3], hi.y));
}

__device__ __forceinline__ f32x4 widen4(uint2 b)
{
    return (f32x4){__uint_as_float(b.x << 16), __uint_as_float(b.x & 0xffff0000u), __uint_as_float(b.y << 16),
                   __uint_as_float(b.y & 0xffff0000u)};
}

// ------------------------------------------------------------ RMSNorm rows
//
// Row m: first x += the kPgSplit partial products of the residual GEMM that ran
// before (in split order), then
// h = x * g / sqrt(mean(x^2) + eps), stored as the split operand of the GEMM
// that follows.  EMBED: the row is fetched from the embedding table instead
// (x[m] = E[token]).  Rows outside the prompt are stored as zeros.
// Every load of a row is in flight together (split after split, a row took five round trips to memory:
// with the numbering below, 512 rows of the 7B shape 16.9 -> 13.3 us, 3584 rows 110 -> 83).  NV: 1024-column pieces of a row (d <= 1024 NV).
// The rows of a group write 8-byte pieces of the same lines of the operand: blocks are dealt to the eight XCDs in
// turn, and a group's sixteen blocks are numbered to land on one, whose L2 puts the lines together.
// grid: 128 ceil((G - g0) / 8) blocks (one per row, from group g0 on) of 256 threads.
template <bool EMBED, int NV>
__global__ __launch_bounds__(256) void prefill_norm_kernel(const bf16_t *__restrict__ E, const int32_t *__restrict__ tok,
                                                            float *__restrict__ x, const float *__restrict__ part,
                                                            const bf16_t *__restrict__ gain, bf16_t *__restrict__ xq, int nks,
                                                            int d, int g0, int G, int L, int P, float inv_d, float eps)
{
    __shared__ float red[4];
    const int grp = g0 + (int)(blockIdx.x & 7) + 8 * (int)(blockIdx.x >> 7);
    if (grp >= G) return;
    const int m = 16 * grp + (int)((blockIdx.x >> 3) & 15), r = m - (L & 15);
    const bool valid = r >= 0 && r < P;
    const size_t rows = (size_t)G * 16;
    float *xr = x + (size_t)m * d;
    f32x4 v[NV];
    float ss = 0.f;
    if (valid) {
        // every load of the row is requested before the first one is used
        const bf16_t *er = EMBED ? E + (size_t)tok[r] * d : nullptr;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int k = 4 * threadIdx.x + 1024 * i;
            v[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
            if (k < d) v[i] = EMBED ? widen4(*reinterpret_cast<const uint2 *>(er + k)) : *reinterpret_cast<const f32x4 *>(xr + k);
        }
        if (!EMBED) {
            f32x4 p[kPgSplit][NV];
#pragma unroll
            for (int s = 0; s < kPgSplit; ++s)
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    const int k = 4 * threadIdx.x + 1024 * i;
                    p[s][i] = (f32x4){0.f, 0.f, 0.f, 0.f};
                    if (k < d) p[s][i] = *reinterpret_cast<const f32x4 *>(part + ((size_t)s * rows + m) * d + k);
                }
#pragma unroll
            for (int s = 0; s < kPgSplit; ++s)   // split order
#pragma unroll
                for (int i = 0; i < NV; ++i) v[i] += p[s][i];
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int k = 4 * threadIdx.x + 1024 * i;
            if (k < d) {
                *reinterpret_cast<f32x4 *>(xr + k) = v[i];
                ss = fmaf(v[i][3], v[i][3], fmaf(v[i][2], v[i][2], fmaf(v[i][1], v[i][1], fmaf(v[i][0], v[i][0], ss))));
            }
        }
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    const float rinv = 1.0f / sqrtf((red[0] + red[1] + red[2] + red[3]) * inv_d + eps);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int k = 4 * threadIdx.x + 1024 * i;
        if (k < d) {
            f32x4 h = {0.f, 0.f, 0.f, 0.f};
            if (valid) h = v[i] * rinv * widen4(*reinterpret_cast<const uint2 *>(gain + k));
            xq_store4(xq, nks, m, k, h);
        }
    }
}

// --------------------------------------------------------------- epilogues

__host__ __device__ __forceinline__ size_t qpf_offset(int head, int G, int head_dim, int m, int dim, int lo)
{
    const int nksq = head_dim >> 5;
    return (((((size_t)head * G + (m >> 4)) * nksq + (dim >> 5)) * 2 + lo) * 64 + (size_t)((dim >> 3) & 3) * 16 + (m & 15)) * 8 +
           (dim & 7);
}

// y: this lane's four outputs (features 4 kg .. 4 kg + 3 of weight tile `tile`) for row m.
// Every lane of the wave must call this: the fused forms exchange values with lane ^ 32.  (QKV: prefill_finish_qkv.)
template <int EPI>
__device__ __forceinline__ void prefill_epilogue(const PrefillArgs &a, int tile, int m, int kg, f32x4 y, bool valid, int sp)
{
    if (EPI == EPI_RESIDUAL) {
        if (valid) *reinterpret_cast<f32x4 *>(a.part + ((size_t)sp * a.G * 16 + m) * a.d + tile * 16 + 4 * kg) = y;
    } else if (EPI == EPI_GATE_UP) {
        // gate rows are in the lower half of the wave, the matching up rows in the upper half: two swaps give either half
        // both rows of two of the four features (each lane all four, with half of the lanes' work thrown away, and
        // the rows exchanged through LDS: see the kernel's comment)
        float q[2], up[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(y[i]), __float_as_uint(y[i + 2]), false, false);
            const float g = __uint_as_float(p[0]);
            q[i] = g / (1.0f + expf(-g));
            up[i] = __uint_as_float(p[1]);
        }
        if (valid) {
            const int k = tile * 8 + 4 * (kg & 1) + 2 * (kg >> 1);
            const uint32_t hi = pack_bf16(q[0] * up[0], q[1] * up[1]);
            *reinterpret_cast<uint32_t *>(a.out + xq_offset(a.out_nks, m, k, 0)) = hi;
            // (the product's rest in the fused form, by name: left to itself the compiler fuses or does not, by the code around
            // it, and the forms' bits must agree)
            *reinterpret_cast<uint32_t *>(a.out + xq_offset(a.out_nks, m, k, 1)) =
                pack_bf16(fmaf(q[0], up[0], -__uint_as_float(hi << 16)), fmaf(q[1], up[1], -__uint_as_float(hi & 0xffff0000u)));
        }
    }
}

// QKV: rotary embedding, query operand, cache write, for the row groups g0 .. g0 + TG - 1 of one weight tile.  What
// depends on the tile or on the group alone is worked out once for all of them, and every angle is requested before
// the first is used (one row group after the other, each with its own divisions, addresses and waits: 4400
// instructions per wave behind the loop at TN = 3, 1800 now).
// Tried: values exchanged between four lanes for stores of 8 bytes instead of four of 2 (no change).
// page: byte offsets of the groups' pages in the pool.
template <int TG>
__device__ __forceinline__ void prefill_finish_qkv(const PrefillArgs &a, int tile, int g0, const f32x4 (&y)[TG], const bool (&valid)[TG],
                                                   const size_t (&page)[TG])
{
    const int lane = threadIdx.x & 63, slot = lane & 15, kg = lane >> 4;
    const int tph = a.head_dim / 16, half = a.head_dim / 2, Tq = a.n_heads * tph, Tkv = a.n_kv_heads * tph;
    if (tile >= Tq + Tkv) {
        const int t = tile - Tq - Tkv, h = t / tph, j = t - h * tph;
        // (head block of the page, dimensions 16 j .. of it)
        char *dst = (char *)(a.pool + kvf_base(0, a.layer, a.n_layers, 1, h, a.n_kv_heads, a.head_dim) + vf_elem(slot, 16 * j + 4 * kg));
#pragma unroll
        for (int g = 0; g < TG; ++g) {
            if (!valid[g]) continue;
            bf16_t *d = (bf16_t *)(dst + page[g]);
#pragma unroll
            for (int i = 0; i < 4; ++i) d[4 * i] = (bf16_t)pack_bf16(y[g][i], 0.f);
        }
        return;
    }
    const bool is_q = tile < Tq;
    const int t = is_q ? tile : tile - Tq, h = t / tph, j = t - h * tph;
    const int i0 = 8 * j + 4 * (kg & 1), dim = i0 + (kg < 2 ? 0 : half);
    f32x4 cs[TG][2];   // (cos, sin) of pairs 0, 1 and 2, 3
    const float2 *rope = a.rope + (size_t)((a.L & ~15) + g0 * 16 + slot) * half + i0;
#pragma unroll
    for (int g = 0; g < TG; ++g) {
        cs[g][0] = cs[g][1] = (f32x4){1.f, 0.f, 1.f, 0.f};
        if (valid[g]) {
            const f32x4 *c = reinterpret_cast<const f32x4 *>(rope + (size_t)g * 16 * half);
            cs[g][0] = c[0];
            cs[g][1] = c[1];
        }
    }
    char *k_dst = (char *)(a.pool + kvf_base(0, a.layer, a.n_layers, 0, h, a.n_kv_heads, a.head_dim) + kf_elem(slot, dim));
    bf16_t *q_dst = a.qp + qpf_offset(h, a.G, a.head_dim, g0 * 16 + slot, dim, 0);
    const int q_group = (a.head_dim >> 5) * 1024;   // elements between row groups; 512: from hi to lo
#pragma unroll
    for (int g = 0; g < TG; ++g) {
        f32x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // the same output of lane ^ 32
            auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(y[g][i]), __float_as_uint(y[g][i]), false, false);
            const float other = __uint_as_float(kg < 2 ? p[1] : p[0]), c = cs[g][i >> 1][2 * (i & 1)], cross = other * cs[g][i >> 1][2 * (i & 1) + 1];
            o[i] = kg < 2 ? fmaf(y[g][i], c, -cross) : fmaf(y[g][i], c, cross);
        }
        if (!valid[g]) continue;
        const uint2 hi = make_uint2(pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3]));
        if (is_q) {
            *reinterpret_cast<uint2 *>(q_dst + g * q_group) = hi;
            *reinterpret_cast<uint2 *>(q_dst + g * q_group + 512) = make_uint2(pack_lo(o[0], o[1], hi.x), pack_lo(o[2], o[3], hi.y));
        } else {
            *reinterpret_cast<uint2 *>(k_dst + page[g]) = hi;
        }
    }
}

// The epilogues of one wave: tiles f0 .. f0 + TN - 1 (below tile_end), row groups g0 .. g0 + TG - 1 (below G).
template <int EPI, int TN, int TG>
__device__ __forceinline__ void prefill_finish(const PrefillArgs &a, int f0, int tile_end, int g0, const f32x4 (&acc)[TN][TG], int sp)
{
    const int lane = threadIdx.x & 63, kg = lane >> 4, r0 = a.L & 15;
    bool valid[TG];
    size_t page[TG];
#pragma unroll
    for (int g = 0; g < TG; ++g) {
        const int m = (g0 + g) * 16 + (lane & 15);
        valid[g] = g0 + g < a.G && m >= r0 && m < r0 + a.P;
        page[g] = 0;
        if (EPI == EPI_QKV && g0 + g < a.G)
            page[g] = kvf_base(a.page_table[(a.L >> 4) + g0 + g], 0, a.n_layers, 0, 0, a.n_kv_heads, a.head_dim) * sizeof(bf16_t);
    }
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        if (f0 + t >= tile_end) break;   // wave-uniform
        if (EPI == EPI_QKV) {
            prefill_finish_qkv<TG>(a, f0 + t, g0, acc[t], valid, page);
        } else {
#pragma unroll
            for (int g = 0; g < TG; ++g) prefill_epilogue<EPI>(a, f0 + t, (g0 + g) * 16 + (lane & 15), kg, acc[t][g], valid[g], sp);
        }
    }
}

// -------------------------------------------------------------------- GEMM
//
// Y^T[features][rows] = W X^T with hi and lo terms of X accumulated into the
// same tile.  Block = 4 x 2 waves (WF = 4), 64 TN features x 128 rows, each wave
// TN weight fragments x 4 row groups.  Per k-step the block needs 4 TN weight
// fragments and 16 activation fragments of 1 KiB; each wave requests its share
// of them straight into LDS (buffer loads with the LDS bit: lane i's 16 bytes
// land at base + 16 i, the fragment order itself; absent tiles, row groups and
// k-steps read zeros and fetch nothing) through a ring of k-steps, and every wave
// then reads its TN + 8 fragments per k-step from LDS.  A fragment thus crosses
// the L2 -> CU path once per block instead of once per wave that uses it.
//
// Three things take about the same time here - the matrix cores (8 TN MFMAs per wave and k-step), the LDS
// reads (TN + 8 fragments per wave) and the L2 -> CU traffic (4 TN + 16 fragments per block) - so they have to
// run side by side: a wave holds the fragments of k-step i in one set of registers while it reads those of k-step
// i + 1 into the other, one every few MFMAs, and the three k-steps behind that are on their way into LDS.  The
// requests for the fourth go out between the MFMAs as well: all at once behind the barrier they held up every wave
// until the queue had taken them (gate/up of 512 rows 141.5 -> 139.4 us, of 128 rows 87 -> 83).  One block barrier
// per k-step: it publishes the stage whose loads every wave has just waited for and frees the stage that every
// wave has just finished reading.
// (Figures here and in launch_prefill_gemm are of the kernel alone, repeated, before every load had its own place in the ring,
// which took 1 to 3 % off; between the others of a prompt, traced, gate/up took 153 us at 512 rows where it took 135.5 alone, 934 at
// 3584 where it took 921.)
// What is left (gate/up of 512 rows, one round of 232 blocks, 135.5 us): 0.93 us per k-step, of which the MFMAs
// alone would take 0.66 at the clock that the power limit leaves them (0.79 without the loads into LDS, 0.83
// without the reads; 0.79 with a third of the chip at work, and no faster without the reads: what they cost is
// power), and 16 us around the loop.  Of those the SwiGLU of the epilogue took 4 more while every lane computed four
// products and half the lanes threw them away (139.4 -> 135.5; gate/up of 3584 rows 983 -> 965).
// Tried: one barrier per two k-steps (no change at TN = 6, 5 % slower at TN = 2, whose loads have less time to land),
// 32x32x16 MFMAs (registers only, random operands: 10 % slower), blocks of four waves, two per compute unit, whose
// barriers fall at different times (half as much again to read per MFMA: gate/up of 3584 rows 1124 against 1002).
//
// RESIDUAL GEMMs (few output features) are split S ways along K so that the
// grid fills the chip; the S partial tiles go to `part` and are added to the
// residual stream, in split order, by the norm kernel that follows.  S is
// fixed by the matrix, never by the number of rows: a row's sums are formed
// in the same order whatever else is in the batch.
// grid: ceil((n_tiles - tile0) / (4 TN)) * S * ceil((G - g0) / 8) blocks; rows run fastest, so
// consecutive blocks share a weight range.
template <int OFF>
__device__ __forceinline__ u32x4_t lds_read16(uint32_t addr)
{
    u32x4_t v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
    return v;
}

// waits until at most N of this wave's loads are outstanding, then for the block
template <int N>
__device__ __forceinline__ void wait_loads_and_meet()
{
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(N) : "memory");
}

// WF: waves side by side along the features (2 along the rows).  Fragments per stage, loads per wave and stage, places per
// stage (every load has one, also those of nothing that make every wave's number even), stages of the ring, bytes of LDS
__host__ __device__ constexpr int pg_units(int TN, int WF) { return WF * TN + 16; }
__host__ __device__ constexpr int pg_loads(int TN, int WF) { return (pg_units(TN, WF) + 2 * WF - 1) / (2 * WF); }
__host__ __device__ constexpr int pg_places(int TN, int WF) { return pg_loads(TN, WF) * 2 * WF; }
__host__ __device__ constexpr int pg_stages(int WF) { return WF == 4 ? 4 : 3; }
__host__ __device__ constexpr size_t pg_lds_bytes(int TN, int WF) { return (size_t)pg_stages(WF) * pg_places(TN, WF) * 1024; }

// calls f with 0, 1, ... as compile-time constants
template <int... I, typename F>
__device__ __forceinline__ void index_each(std::integer_sequence<int, I...>, F f)
{
    f(std::integral_constant<int, I>{}...);
}

// one wave's fragments of a k-step
template <int TN>
struct PgFrags {
    u32x4_t w[TN], xh[kPfTM], xl[kPfTM];
};

// Block `block` of n_blocks that take the tiles [tile0, tile_end).
template <int EPI, int TN, int WF>
__device__ __forceinline__ void prefill_gemm_block(const PrefillArgs &a, int block, int n_blocks, int tile0, int tile_end)
{
    constexpr int kUnits = pg_units(TN, WF), kLoads = pg_loads(TN, WF), kPlaces = pg_places(TN, WF), kStages = pg_stages(WF);
    extern __shared__ uint4 ring[];   // [kStages][kPlaces][64]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wf = wave % WF, wr = wave / WF;
    const int n_br = (a.G - a.g0 + 7) / 8;
    int id = xcd_order(block, n_blocks);
    const int br = id % n_br;
    id /= n_br;
    const int sp = id % a.S, bt = id / a.S;
    const int F0 = tile0 + bt * WF * TN, G0 = a.g0 + br * 8;
    const int nks = a.nks;
    const int ks0 = (int)((long long)sp * nks / a.S), n_it = (int)((long long)(sp + 1) * nks / a.S) - ks0;

    // this wave's share of a stage: units kLoads * wave .. + kLoads - 1 (units 0 .. 4 TN - 1 weights, then row
    // groups x (hi, lo)); a unit past the end is an empty descriptor: every wave issues the same number of
    // loads per stage, which is what the waits below count
    __amdgpu_buffer_rsrc_t rs[kLoads];
    int uoff[kLoads], ustride[kLoads];
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
        const int u = kLoads * wave + j;
        if (u < WF * TN) {
            const int tile = F0 + u;
            const bool have = tile < tile_end;
            rs[j] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4 *>(a.Wp + ((size_t)(have ? tile : 0) * nks + ks0) * 64), 0,
                                                      have ? n_it * 1024 : 0, 0x00020000);
            uoff[j] = 0;
            ustride[j] = 1024;
        } else {
            // the descriptor ends with this row group's last k-step of the split
            const int v = u - WF * TN, g = G0 + (v >> 1);   // (row group, hi | lo)
            const bool have = u < kUnits && g < a.G;
            rs[j] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4 *>(a.Xq + ((size_t)(have ? g : 0) * nks + ks0) * 128), 0,
                                                      have ? n_it * 2048 : 0, 0x00020000);
            uoff[j] = (v & 1) * 1024;
            ustride[j] = 2048;
        }
    }
    // the stage that begins with place `stage` of the ring <- k-step `it` (past the end: zeros, nothing fetched)
    // (one place for all loads of nothing instead of one each had a choice per load and a product per stage in the loop, scalar
    // instructions that showed at short k-steps: TN = 2, QKV of 144 rows 59.3 -> 55.8 us, 13B 72.7 -> 69.4, O and down of 3584
    // rows, TN = 4, 382 -> 373)
    auto request_one = [&](int j, int it, int stage) __attribute__((always_inline)) {
        load_to_lds(rs[j], ring + (size_t)(stage + kLoads * wave + j) * 64, uoff[j] + it * ustride[j] + lane * 16);
    };
    auto request = [&](int it, int stage) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < kLoads; ++j) request_one(j, it, stage);
    };

    f32x4 acc[TN][kPfTM];
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int g = 0; g < kPfTM; ++g) acc[t][g] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)ring + (uint32_t)lane * 16;

    // The fragment reads are written as assembly: reads the compiler can see would make it wait for
    // every outstanding load into LDS first (it cannot tell the ring's stages apart).
    using Frags = PgFrags<TN>;
    // read i of a stage: weight fragments, then the row groups' hi terms, then their lo terms
    auto read_one = [&](auto index, Frags &f, uint32_t aw, uint32_t ax) __attribute__((always_inline)) {
        constexpr int i = decltype(index)::value;
        if constexpr (i < TN) f.w[i] = lds_read16<1024 * i>(aw);
        else if constexpr (i < TN + 4) f.xh[i - TN] = lds_read16<2048 * (i - TN)>(ax);
        else f.xl[i - TN - 4] = lds_read16<2048 * (i - TN - 4) + 1024>(ax);
    };
    auto wait_reads = [&](Frags &f) __attribute__((always_inline)) {
        // (the second statement carries the remaining registers through the same wait)
        asm volatile("s_waitcnt lgkmcnt(0)"
                     : "+v"(f.xh[0]), "+v"(f.xh[1]), "+v"(f.xh[2]), "+v"(f.xh[3]), "+v"(f.xl[0]), "+v"(f.xl[1]), "+v"(f.xl[2]), "+v"(f.xl[3]));
#pragma unroll
        for (int t = 0; t < TN; ++t) asm volatile("" : "+v"(f.w[t]));
    };
    // MFMA j of a k-step: every (weight, row group) pair's hi term, then every pair's lo term
    auto mma_one = [&](const Frags &f, int j) __attribute__((always_inline)) {
        const int t = (j % (4 * TN)) / 4, g = j % 4;
        acc[t][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f.w[t]),
                                                            __builtin_bit_cast(bf16x8, j < 4 * TN ? f.xh[g] : f.xl[g]), acc[t][g], 0, 0, 0);
    };
    // The reads of the next k-step's fragments from stage `stage`, one every few MFMAs of this one's, the last
    // some MFMAs before the end: issued in one go they would fill the LDS queue and hold up every wave's MFMAs
    // until they are through.
    auto interleave = [&](const Frags &cur, Frags &next, int stage, int ahead, int free_stage) __attribute__((always_inline)) {
        constexpr int NR = TN + 8, NM = 8 * TN, SPAN = NM * 85 / 100;
        const uint32_t sbase = lds_base + (uint32_t)stage * 1024;
        const uint32_t aw = sbase + (uint32_t)(TN * wf) * 1024, ax = sbase + (uint32_t)(WF * TN + 8 * wr) * 1024;
        auto part = [&](auto index) __attribute__((always_inline)) {
            constexpr int i = decltype(index)::value;
            read_one(index, next, aw, ax);
#pragma unroll
            for (int j = 0; j < kLoads; ++j)
                if (j * NR / kLoads == i) request_one(j, ahead, free_stage);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = i * SPAN / NR; j < (i + 1 == NR ? NM : (i + 1) * SPAN / NR); ++j) mma_one(cur, j);
            __builtin_amdgcn_sched_barrier(0);
        };
        index_each(std::make_integer_sequence<int, NR>{}, [&](auto... index) __attribute__((always_inline)) { (part(index), ...); });
    };
    // One k-step: `cur` holds its fragments.  This wave's loads of k-step it + 1 have landed when at most the
    // kStages - 2 younger stages are outstanding; after the barrier every wave's have, and every wave has its
    // fragments of k-step it in registers, so that slot is free for k-step it + kStages.
    int stage = 0;   // of k-step it: its first place
    auto step = [&](const Frags &cur, Frags &next, int it) __attribute__((always_inline)) {
        wait_loads_and_meet<(kStages - 2) * kLoads>();
        const int free_stage = stage;
        stage = stage == (kStages - 1) * kPlaces ? 0 : stage + kPlaces;
        interleave(cur, next, stage, it + kStages, free_stage);
        wait_reads(next);
    };
#pragma unroll
    for (int s = 0; s < kStages; ++s) request(s, s * kPlaces);
    Frags fa, fb;
    wait_loads_and_meet<(kStages - 1) * kLoads>();
    index_each(std::make_integer_sequence<int, TN + 8>{}, [&](auto... index) __attribute__((always_inline)) {
        (read_one(index, fa, lds_base + (uint32_t)(TN * wf) * 1024, lds_base + (uint32_t)(WF * TN + 8 * wr) * 1024), ...);
    });
    wait_reads(fa);
    for (int it = 0; it < n_it; it += 2) {   // (an odd n_it ends with a k-step of zeros)
        step(fa, fb, it);
        step(fb, fa, it + 1);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (the last requests, of nothing)

    const int f0 = F0 + TN * wf, g0 = G0 + 4 * wr;
    prefill_finish<EPI, TN, kPfTM>(a, f0, tile_end, g0, acc, sp);
}

template <int EPI, int TN>
__global__ __launch_bounds__(kPgThreads) void prefill_gemm_kernel(PrefillArgs a)
{
    prefill_gemm_block<EPI, TN, 4>(a, blockIdx.x, gridDim.x, a.tile0, a.n_tiles);
}
// half as wide, four waves
template <int EPI, int TN>
__global__ __launch_bounds__(256, 2) void prefill_narrow_kernel(PrefillArgs a)
{
    prefill_gemm_block<EPI, TN, 2>(a, blockIdx.x, gridDim.x, a.tile0, a.n_tiles);
}
// the tiles up to tiles_a in blocks of TA, n_a of them, the rest in blocks of TB
template <int EPI, int TA, int TB>
__global__ __launch_bounds__(kPgThreads) void prefill_mixed_kernel(PrefillArgs a, int n_a, int tiles_a)
{
    if ((int)blockIdx.x < n_a) prefill_gemm_block<EPI, TA, 4>(a, blockIdx.x, n_a, a.tile0, tiles_a);
    else prefill_gemm_block<EPI, TB, 4>(a, (int)blockIdx.x - n_a, (int)gridDim.x - n_a, tiles_a, a.n_tiles);
}

// ------------------------------------------------- GEMM, few rows
//
// Prompts (pieces) of a few row groups: the weights' bytes are what counts, and the form above, made for tiles of 128
// rows, keeps 24 to 72 KB of them in flight per compute unit, on a third of the chip.  Here a wave streams the one tile
// that it owns through a ring of 16 k-steps of registers against TG row groups, whose fragments two waves of their own
// bring through LDS, eight k-steps at a time, for all waves of the block: they wait for their own loads only, and the
// others' weights stay in flight (loads of a wave come back in the order they were requested).  The waves meet once
// per eight k-steps.  An element's sums are those of the form above: one chain over the k-steps, hi term, lo term.
// Bound by the weights and, from about 64 rows, by what the operand and the weights (read once per TG groups) take from
// L2: 7B shape, 32 / 64 rows, QKV 19.2 / 19.9 us (5.2 / 5.1 TB/s of weights; the form above 45), gate/up 28.4 / 30.9
// (48), down 17.0 / 19.0 (33).  The order of a k-step's requests is in the source: left to itself the compiler put
// the weight loads of eight k-steps together at their end, behind reads waited for one by one (QKV 21.3 / 24.0).
// Tried: four row groups per block (no faster at any size), one wave or four bringing the operand (the same).
constexpr int kFewChunk = 8, kFewBufs = 3;   // k-steps per buffer of the operand, buffers
__host__ __device__ constexpr int few_units(int TG) { return kFewChunk * 2 * TG; }   // fragments per buffer
__host__ __device__ constexpr size_t few_lds_bytes(int TG) { return (size_t)kFewBufs * few_units(TG) * 1024; }
constexpr int kFewDepth = 16;   // weight fragments in flight per wave
constexpr int kFewLoaders = 2;  // waves that bring the operand
constexpr int kFewWaves = 14;   // most waves with a tile
// blockDim: 64 x (tiles per block + kFewLoaders).  grid: ceil(n_tiles / tiles per block) * S * ceil(G / TG), rows fastest.
// ONCE: one block takes all row groups, so the weights are read once and marked non-temporal (weights from HBM, 16 / 32 rows:
// QKV 20.0 -> 19.2 us, 22.2 -> 20.6, gate/up 32.5 -> 30.5, 34.5 -> 33.1).
template <int EPI, int TG, bool ONCE>
__global__ __launch_bounds__((kFewWaves + kFewLoaders) * 64) void prefill_few_kernel(PrefillArgs a)
{
    constexpr int D = kFewDepth, DX = kFewChunk, NB = kFewBufs, UNITS = few_units(TG);
    extern __shared__ uint4 xs[];   // [NB][DX][TG][hi | lo][64]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n_waves = (int)(blockDim.x >> 6) - kFewLoaders;
    const int n_br = (a.G - a.g0 + TG - 1) / TG;
    int id = xcd_order((int)blockIdx.x, (int)gridDim.x);
    const int br = id % n_br;
    id /= n_br;
    const int sp = id % a.S, bt = id / a.S;
    const int G0 = a.g0 + br * TG, nks = a.nks;
    const int ks0 = (int)((long long)sp * nks / a.S), n_it = (int)((long long)(sp + 1) * nks / a.S) - ks0;
    const int n_chunks = (n_it + DX - 1) / DX;
    if (wave >= n_waves) {
        // a wave that brings the operand, DX / kFewLoaders k-steps of every chunk: chunk c + NB - 1 is requested when chunk c is ready
        const int k0 = (wave - n_waves) * (DX / kFewLoaders);
        auto load_x = [&](int c) __attribute__((always_inline)) {
            uint4 *dst = xs + (size_t)(c % NB) * UNITS * 64;
#pragma unroll
            for (int g = 0; g < TG; ++g) {
                const bool have = G0 + g < a.G;
                __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4 *>(a.Xq + ((size_t)(have ? G0 + g : 0) * nks + ks0) * 128), 0,
                                                                             have ? n_it * 2048 : 0, 0x00020000);
#pragma unroll
                for (int k = 0; k < DX / kFewLoaders; ++k)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        load_to_lds(r, dst + ((size_t)((k0 + k) * TG + g) * 2 + h) * 64, ((c * DX + k0 + k) * 2 + h) * 1024 + lane * 16);
            }
        };
        for (int c = 0; c < NB - 1; ++c) load_x(c);
        for (int c = 0; c < n_chunks; ++c) {
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NB - 2) * UNITS / kFewLoaders) : "memory");
            load_x(c + NB - 1);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        return;
    }
    const int tile = a.tile0 + bt * n_waves + wave;
    const bool have = tile < a.n_tiles;
    __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4 *>(a.Wp + ((size_t)(have ? tile : 0) * nks + ks0) * 64), 0,
                                                                  have ? n_it * 1024 : 0, 0x00020000);
    u32x4_t w[D];
    auto load_w = [&](int s, int i) __attribute__((always_inline)) { w[s] = __builtin_amdgcn_raw_buffer_load_b128(rw, lane * 16 + i * 1024, 0, ONCE ? kAuxStream : 0); };
#pragma unroll
    for (int s = 0; s < D; ++s) load_w(s, s);
    f32x4 acc[TG];
#pragma unroll
    for (int g = 0; g < TG; ++g) acc[g] = (f32x4){0.f, 0.f, 0.f, 0.f};
    u32x4_t xf[2][TG][2];
    int buf = 0;
    for (int c0 = 0; c0 < n_chunks; c0 += D / DX) {
#pragma unroll
        for (int h = 0; h < D / DX; ++h) {
            const int c = c0 + h;
            if (c >= n_chunks) break;   // (the same for the whole block)
            block_sync_lds();
            const u32x4_t *x = reinterpret_cast<const u32x4_t *>(xs) + (size_t)buf * UNITS * 64 + lane;
            buf = buf + 1 == NB ? 0 : buf + 1;
            auto read_x = [&](int k) __attribute__((always_inline)) {
#pragma unroll
                for (int g = 0; g < TG; ++g) {
                    xf[k & 1][g][0] = x[((k * TG + g) * 2) * 64];
                    xf[k & 1][g][1] = x[((k * TG + g) * 2 + 1) * 64];
                }
            };
            read_x(0);
#pragma unroll
            for (int k = 0; k < DX; ++k) {
                const int s = h * DX + k;
                if (k + 1 < DX) read_x(k + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int hl = 0; hl < 2; ++hl)
#pragma unroll
                    for (int g = 0; g < TG; ++g)
                        acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[s]), __builtin_bit_cast(bf16x8, xf[k & 1][g][hl]), acc[g], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                load_w(s, c * DX + k + D);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    prefill_finish<EPI, 1, TG>(a, tile, a.n_tiles, G0, reinterpret_cast<f32x4 (&)[1][TG]>(acc), sp);
}

// --------------------------------------------------------------- attention
//
// Causal attention of the prompt rows over the cache (which by now holds the
// prompt's own K and V).  Block = (head, two 16-row groups), four waves; wave w
// takes the page pairs w, w + 4, ... and both row groups against each, the waves' running (maximum, denominator,
// output) meet in LDS at the end.  A group is one cache page, so every earlier
// page is visible in full and only the group's own page needs the causal mask.  Per pair: S = K q^T (query as
// hi + lo B operands; scores land with keys in registers and rows across lanes), online softmax
// per row in the base-2 domain, P as hi + lo B operands straight from those registers, O += V^T P with the two pages'
// keys in one 32-key MFMA.  The next pair's K is requested when this pair's scores are done, its V when its
// output is.
// Why: with one wave per row group every group read all its pages (6.6 GB per layer from L2 at 3584 rows: 300 us at
// what L2 delivers), 16-key MFMAs did half the work of a 32-key one in the same time, the output was rescaled and a maximum
// exchanged per page, and a short prompt behind a long cache left the pages to a few waves one after the other.
// 7B shape, 512 / 3584 rows: 35 -> 21 / 489 -> 409 us per layer; 205 rows behind 777, 32 heads over 2 key / value heads: 63 -> 19.
// Then nothing covered a wave's exponentials at 3584 rows: with the query rows in registers a lane of head dim 128 held 238 and 80
// accumulators, one wave per SIMD (vector ALU 45 %, matrix cores 22 % busy).  The rows are the same for the block's four
// waves: read from LDS for every pair (QLDS), they leave 184 registers and two waves per SIMD: 512 / 3584 rows 19.5 -> 16.2 /
// 414 -> 284 us.  (Three waves, 168 registers, some of them in scratch memory: 23.5 / 443.)  Where the blocks are too few for
// that second wave the reads are all that is left of it, and the rows stay in registers: 128 rows, LDS / registers 7.9 / 6.7 us,
// 256 rows, 256 blocks, 9.8 / 9.0, 320 rows behind 1000, 320 blocks, 28 / 36.  At head dim 64 two blocks fit a compute unit with the
// rows in registers (188): 32 heads, 272 / 512 rows, 7.0 / 6.4, 10.3 / 9.9, 600 behind 1000, 608 blocks, 27.0 / 37.2.
// A row's sums depend on absolute page numbers only, not on how the prompt was cut.  (They are not, bit for bit, those of
// one wave going page by page with a maximum that always moves: one layer's output is 8e-6 apart, 2^-17 being what the
// weights' two bf16 terms keep, and equally far from the 64-bit result.)
// Scores of any size are right (see kHugeScore).  What is not finite: a key whose score is NaN has weight 0; V of keys on a row's own page that the row must not see is
// multiplied by 0, as in a step, V of later pages is not.
// grid: (n_heads, ceil((G - first) / 2)): row groups from `first` on; later groups (more pages) start first.
constexpr float kHugeScore = 0x1p29f;   // rounding a base-2 score of this size may move it by 2^5; below it by 2^4, weights stay under 2^(8 + 16)
template <int DH, bool QLDS>
__global__ __launch_bounds__(256, QLDS ? 2 : 1) void prefill_attn_kernel(const uint4 *__restrict__ qp, const bf16_t *__restrict__ pool,
                                                            const int32_t *__restrict__ page_table, int first, int G, int L, int P,
                                                            int layer, int n_layers, int n_heads, int n_kv_heads, float scale,
                                                            bf16_t *__restrict__ xq_att, int nks_d)
{
    constexpr int NKS = DH / 32, NDT = DH / 16, WAVES = 4;
    // the query rows while the pages go by, the waves' outputs behind them
    __shared__ union {
        uint4 q[2][NKS][2][64];   // [group][32 dims][hi | lo], the same for every wave
        float part[WAVES][2][NDT][64][4];
    } lds;
    __shared__ float wmax[WAVES][2][16], wden[WAVES][2][16];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), slot = lane & 15, kg = lane >> 4;
    const int head = blockIdx.x, kvh = head / (n_heads / n_kv_heads);
    const int g0 = first + 2 * ((int)gridDim.y - 1 - (int)blockIdx.y), n_grp = G - g0 < 2 ? G - g0 : 2;
    const int own0 = (L >> 4) + g0;                 // the first group's own page; the second group's is the next one
    const int last_page = own0 + n_grp - 1, last_pair = last_page >> 1;

    uint4 qf[2][NKS][2];   // (the query rows in registers)
    if (QLDS) {
        for (int i = wave; i < 2 * NKS * 2; i += WAVES) {
            const int x = i / (2 * NKS), r = i % (2 * NKS);
            (&lds.q[0][0][0][0])[i * 64 + lane] = qp[(((size_t)head * G + g0 + (x < n_grp ? x : 0)) * 2 * NKS + r) * 64 + lane];
        }
    } else {
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const uint4 *q = qp + ((size_t)head * G + g0 + (x < n_grp ? x : 0)) * NKS * 128;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
                for (int hl = 0; hl < 2; ++hl) qf[x][ks][hl] = q[(ks * 2 + hl) * 64 + lane];
        }
    }
    // page numbers of the wave's next 64 pairs, one pair per lane; a pair's second page, if it does not exist, is the
    // first one again (its keys get weight 0)
    int ida = 0, idb = 0;
    auto fetch_ids = [&](int k0) __attribute__((always_inline)) {
        const int pa = 2 * (wave + WAVES * (k0 + lane));
        ida = page_table[pa <= last_page ? pa : last_page];
        idb = page_table[pa + 1 <= last_page ? pa + 1 : last_page];
    };
    uint4 kf[2][NKS];
    uint2 vf[2][NDT];
    auto load_k = [&](int page, uint4 (&k)[NKS]) __attribute__((always_inline)) {
        const uint4 *kp = reinterpret_cast<const uint4 *>(pool + kvf_base(page, layer, n_layers, 0, kvh, n_kv_heads, DH));
#pragma unroll
        for (int i = 0; i < NKS; ++i) k[i] = kp[i * 64 + lane];
    };
    auto load_v = [&](int page, uint2 (&v)[NDT]) __attribute__((always_inline)) {
        const uint2 *vp = reinterpret_cast<const uint2 *>(pool + kvf_base(page, layer, n_layers, 1, kvh, n_kv_heads, DH));
#pragma unroll
        for (int i = 0; i < NDT; ++i) v[i] = vp[i * 64 + lane];
    };
    const float scale2 = scale * 1.44269504088896f;
    float m_run[2] = {kMasked, kMasked}, d_run[2] = {0.f, 0.f};
    f32x4 o[2][NDT];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) o[x][dt] = (f32x4){0.f, 0.f, 0.f, 0.f};

    const int n_pairs = last_pair >= wave ? (last_pair - wave) / WAVES + 1 : 0;   // this wave's
    if (n_pairs > 0) {
        fetch_ids(0);
        const int pa = __builtin_amdgcn_readlane(ida, 0), pb = __builtin_amdgcn_readlane(idb, 0);
        load_k(pa, kf[0]);
        load_k(pb, kf[1]);
        load_v(pa, vf[0]);
        load_v(pb, vf[1]);
    }
    if (QLDS) __syncthreads();
    if (n_pairs > 0) {
        for (int k = 0; k < n_pairs; ++k) {
            const int page0 = 2 * (wave + WAVES * k);
            // ---- scores of both groups: lane (slot, kg) has keys 4 kg + i of either page, row slot
            f32x4 sc[2][2];
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y) {
                    f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
                        for (int hl = 0; hl < 2; ++hl)
                            t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[y][ks]),
                                                                        __builtin_bit_cast(bf16x8, QLDS ? lds.q[x][ks][hl][lane] : qf[x][ks][hl]), t, 0, 0, 0);
                    sc[x][y] = t;
                }
            if (((k + 1) & 63) == 0) fetch_ids(k + 1);
            // (past the end: the last page, requested for nothing)
            const int na = __builtin_amdgcn_readlane(ida, (k + 1) & 63), nb = __builtin_amdgcn_readlane(idb, (k + 1) & 63);
            load_k(na, kf[0]);
            load_k(nb, kf[1]);
            // (the second group first: a page that it must not see, the first must not see either)
#pragma unroll
            for (int x = 1; x >= 0; --x) {
                const int own = own0 + x;
                if (x >= n_grp || page0 > own) continue;   // (whole wave) nothing of this pair is visible to the group
                float p[8], mx = kMasked;
                const bool all_seen = page0 + 1 < own;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int page = page0 + (j >> 2);
                    p[j] = sc[x][j >> 2][j & 3];
                    if (!all_seen) p[j] = page < own || (page == own && 4 * kg + (j & 3) <= slot) ? p[j] : kMasked;
                    mx = fmaxf(mx, p[j]);
                }
                // The row's reference follows its maximum only when that is more than 2^8 above it: the weights are
                // then at most 2^8, which costs no precision, and the output is rescaled a few times instead of
                // at every other pair.  (A row's own decision: its bits do not depend on the rows beside it.)
                mx = rows_max(mx) * scale2;
                const float m_new = mx > m_run[x] + 8.f ? mx : m_run[x], alpha = __builtin_amdgcn_exp2f(m_run[x] - m_new);
                m_run[x] = m_new;
                float den = 0.f;
                u32x4_t ph, pl;
                auto weights = [&](bool select, bool huge) __attribute__((always_inline)) {
                    den = 0.f;
                    auto weight = [&](float score) __attribute__((always_inline)) {
                        float t = fmaf(score, scale2, -m_new);
                        if (huge) {   // (opaque: the difference must not be fused with the product)
                            float scaled = score * scale2;
                            asm volatile("" : "+v"(scaled));
                            t = fabsf(m_new) >= kHugeScore ? scaled - m_new : t;
                        }
                        const float w = __builtin_amdgcn_exp2f(t);
                        return select && !(score > 0.5f * kMasked) ? 0.f : w;   // (a key that the row must not see)
                    };
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float a = weight(p[2 * j]), b = weight(p[2 * j + 1]);
                        den += a;
                        den += b;
                        ph[j] = pack_bf16(a, b);
                        pl[j] = pack_bf16(a - __uint_as_float(ph[j] << 16), b - __uint_as_float(ph[j] & 0xffff0000u));
                    }
                };
                weights(!all_seen, false);
                // Looked for behind the sums, in two comparisons: a key whose score is NaN has weight 0, as in a step; and
                // where the reference is huge, the fused product is not the product that it was rounded from: the
                // difference, up to 2^-24 of it, would be the largest key's exponent.
                if (__builtin_amdgcn_ballot_w64(den != den || fabsf(m_new) >= kHugeScore) != 0) weights(true, true);
                d_run[x] = fmaf(d_run[x], alpha, den);
                // (whole-wave branch; a factor of 1 changes nothing)
                if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0) {
#pragma unroll
                    for (int dt = 0; dt < NDT; ++dt) o[x][dt] = o[x][dt] * alpha;
                }
                // a page behind the group's own takes no part at all: 0 times an infinity in its V would be NaN
                if (page0 + 1 > own) {
#pragma unroll
                    for (int dt = 0; dt < NDT; ++dt) vf[1][dt] = make_uint2(0, 0);
                }
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt) {
                    const u32x4_t v = {vf[0][dt].x, vf[0][dt].y, vf[1][dt].x, vf[1][dt].y};
                    o[x][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v), __builtin_bit_cast(bf16x8, ph), o[x][dt], 0, 0, 0);
                    o[x][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v), __builtin_bit_cast(bf16x8, pl), o[x][dt], 0, 0, 0);
                }
            }
            load_v(na, vf[0]);
            load_v(nb, vf[1]);
        }
    }
    // ---- the waves meet: every wave scales to the row's maximum, the sums are formed in wave order
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const float d = rows_sum(d_run[x]);
        if (kg == 0) { wmax[wave][x][slot] = m_run[x]; wden[wave][x][slot] = d; }
    }
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        float bm = wmax[0][x][slot];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) bm = fmaxf(bm, wmax[w][x][slot]);
        const float f = __builtin_amdgcn_exp2f(m_run[x] - bm);
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) *reinterpret_cast<f32x4 *>(lds.part[wave][x][dt][lane]) = o[x][dt] * f;
    }
    __syncthreads();
    for (int u = wave; u < 2 * NDT; u += WAVES) {
        const int x = u / NDT, dt = u % NDT;
        if (x >= n_grp) break;
        float bm = wmax[0][x][slot], den = 0.f;
#pragma unroll
        for (int w = 1; w < WAVES; ++w) bm = fmaxf(bm, wmax[w][x][slot]);
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            den = fmaf(wden[w][x][slot], __builtin_amdgcn_exp2f(wmax[w][x][slot] - bm), den);
            v += *reinterpret_cast<const f32x4 *>(lds.part[w][x][dt][lane]);
        }
        const int m = (g0 + x) * 16 + slot, r = m - (L & 15);
        const bool valid = r >= 0 && r < P;
        const float inv = 1.0f / den;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = valid ? v[i] * inv : 0.f;
        xq_store4(xq_att, nks_d, m, head * DH + 16 * dt + 4 * kg, v);
    }
}

// ---------------------------------------------------- hand-over to the step
//
// The last prompt row is the only one whose logits are needed.  Adds the last
// down projection's partial products to it and leaves it where the step's
// LM-head GEMM expects its input (class-8 packed operand of x * gain in row 0,
// per-tile sums of squares); sets the cache length to just below the row, so
// that the step's own argmax kernel, run for one appended row, finishes the
// job.   grid: d / 16 blocks of one wave.
__global__ __launch_bounds__(64) void prefill_last_kernel(const float *__restrict__ x_row, const float *__restrict__ part_row,
                                                           int S, size_t part_stride, const bf16_t *__restrict__ gain,
                                                           bf16_t *__restrict__ xp, float *__restrict__ ssp,
                                                           int32_t *__restrict__ len_ptr, int len_before_row)
{
    const int lane = threadIdx.x, slot = lane & 15, kg = lane >> 4;
    const int tile = blockIdx.x, n = tile * 16 + 4 * kg;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (slot == 0) {
        v = *reinterpret_cast<const f32x4 *>(x_row + n);
        for (int s = 0; s < S; ++s) v += *reinterpret_cast<const f32x4 *>(part_row + (size_t)s * part_stride + n);
        xp_store4<false>(xp, 8, 0, n, v * widen4(*reinterpret_cast<const uint2 *>(gain + n)));
    }
    float s = fmaf(v[3], v[3], fmaf(v[2], v[2], fmaf(v[1], v[1], v[0] * v[0])));
    s += __shfl_xor(s, 16, kWave);
    s += __shfl_xor(s, 32, kWave);
    if (lane == 0) ssp[(size_t)tile * 32] = s;
    if (blockIdx.x == 0 && lane == 0) *len_ptr = len_before_row;
}

}  // namespace anpd
