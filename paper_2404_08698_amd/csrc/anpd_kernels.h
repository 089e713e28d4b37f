// HIP kernels of the ANPD verification step for gfx950 (MI355X, CDNA4).
//
// The step is one LLaMA-shaped forward over a window of M = k+1 rows (the last
// accepted token plus k drafts; paper Section 3.1, "Parallel Decoding", step 2)
// against a paged KV cache, ending in greedy argmax per row and the
// longest-matching-prefix acceptance of Algorithm 1.
//
// Every kernel computes a window row from that row's own data in an order
// that does not depend on M, so the result for a position is bit-identical
// whether it was verified in a 1-row or a 32-row window.  That is what makes
// ANPD on this path reproduce greedy decoding token for token.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace anpd {

typedef uint16_t bf16_t;  // bfloat16 storage
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kWave = 64;
constexpr int kAttnSplit = 64;        // keys per attention split (fixed: part of the numerics)
constexpr float kMasked = -1.0e30f;   // score of a key a row must not see

// ---------------------------------------------------------------- scalars

__device__ __forceinline__ float bf16_to_f32(bf16_t b) { return __uint_as_float((uint32_t)b << 16); }

// round to nearest, ties to even (finite inputs)
__device__ __forceinline__ bf16_t f32_to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

__device__ __forceinline__ float load_f32(const float *p, size_t i) { return p[i]; }
__device__ __forceinline__ float load_f32(const bf16_t *p, size_t i) { return bf16_to_f32(p[i]); }
__device__ __forceinline__ void store_kv(float *p, size_t i, float v) { p[i] = v; }
__device__ __forceinline__ void store_kv(bf16_t *p, size_t i, float v) { p[i] = f32_to_bf16(v); }

// eight consecutive elements, widened to float
__device__ __forceinline__ void load8(const float *p, float (&o)[8])
{
    float4 a = *reinterpret_cast<const float4 *>(p);
    float4 b = *reinterpret_cast<const float4 *>(p + 4);
    o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
    o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
}
__device__ __forceinline__ void load8(const bf16_t *p, float (&o)[8])
{
    uint4 r = *reinterpret_cast<const uint4 *>(p);
    o[0] = __uint_as_float(r.x << 16); o[1] = __uint_as_float(r.x & 0xffff0000u);
    o[2] = __uint_as_float(r.y << 16); o[3] = __uint_as_float(r.y & 0xffff0000u);
    o[4] = __uint_as_float(r.z << 16); o[5] = __uint_as_float(r.z & 0xffff0000u);
    o[6] = __uint_as_float(r.w << 16); o[7] = __uint_as_float(r.w & 0xffff0000u);
}

// Device-coherent accesses (relaxed, agent scope): the store is written through and the load is
// served from the coherence point, so blocks on different XCDs can hand small results to each
// other through a counter without cache-wide write-back / invalidate fences.
template <typename T>
__device__ __forceinline__ void st_agent(T *p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ __forceinline__ T ld_agent(const T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// The same at system scope, for words in pinned host memory.
template <typename T>
__device__ __forceinline__ void st_system(T *p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }
template <typename T>
__device__ __forceinline__ T ld_system(const T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }

// Accessors for data that one block writes and another block reads.  COH = false: ordinary
// accesses, for kernels whose producers ran in an earlier launch.  COH = true: device-coherent
// accesses (see st_agent / ld_agent), for the persistent kernel where producer and consumer run in
// the same launch on different XCDs.  Wider items are moved as 8-byte pieces.
template <bool COH>
__device__ __forceinline__ float ldc(const float *p) { return COH ? ld_agent(p) : *p; }
template <bool COH>
__device__ __forceinline__ void stc(float *p, float v)
{
    if (COH) st_agent(p, v);
    else *p = v;
}
template <bool COH>
__device__ __forceinline__ uint2 ldc8(const uint2 *p)
{
    if (!COH) return *p;
    unsigned long long v = ld_agent(reinterpret_cast<const unsigned long long *>(p));
    return make_uint2((uint32_t)v, (uint32_t)(v >> 32));
}
template <bool COH>
__device__ __forceinline__ void stc8(void *p, uint2 v)
{
    if (COH) st_agent(reinterpret_cast<unsigned long long *>(p), (unsigned long long)v.x | ((unsigned long long)v.y << 32));
    else *reinterpret_cast<uint2 *>(p) = v;
}
template <bool COH>
__device__ __forceinline__ uint4 ldc16(const uint4 *p)
{
    if (!COH) return *p;
    uint2 lo = ldc8<true>(reinterpret_cast<const uint2 *>(p)), hi = ldc8<true>(reinterpret_cast<const uint2 *>(p) + 1);
    return make_uint4(lo.x, lo.y, hi.x, hi.y);
}
template <bool COH>
__device__ __forceinline__ void stc16(float *p, f32x4 v)
{
    if (COH) {
        stc8<true>(p, make_uint2(__float_as_uint(v[0]), __float_as_uint(v[1])));
        stc8<true>(p + 2, make_uint2(__float_as_uint(v[2]), __float_as_uint(v[3])));
    } else {
        *reinterpret_cast<f32x4 *>(p) = v;
    }
}
// 2-byte store; the coherent form is the same instruction with the write-through bits set
template <bool COH>
__device__ __forceinline__ void stc2(bf16_t *p, bf16_t v)
{
    if (COH) asm volatile("global_store_short %0, %1, off sc0 sc1" ::"v"(p), "v"((uint32_t)v) : "memory");
    else *p = v;
}

// Indexed loads from a buffer whose base pointer is the same for the whole wave.  The coherent
// form uses buffer instructions with the sc0 sc1 bits, which the compiler can keep in flight
// together (atomic loads are issued one at a time); the plain form is an ordinary load.
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
constexpr int kAuxCoherent = 17;  // sc0 | sc1
// Weights are read once per step and never again before 13 GB of other weights have gone by: loads
// marked non-temporal stream them past the caches instead of displacing what is re-read (activations,
// the cache pages).  Measured on the weight access pattern alone: 7.1 TB/s against 6.4 TB/s unmarked.
constexpr int kAuxStream = 2;     // nt
__device__ __forceinline__ uint4 ld_stream(const uint4 *p)
{
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    u4 v = __builtin_nontemporal_load(reinterpret_cast<const u4 *>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint2 ld_stream(const uint2 *p)
{
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    u2 v = __builtin_nontemporal_load(reinterpret_cast<const u2 *>(p));
    return make_uint2(v.x, v.y);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t wave_buffer(const void *base)
{
    // (said explicitly to be the same in every lane: a base that was computed on the vector ALU - an index
    // from an integer division, say - would otherwise make every load a loop over the distinct descriptors)
    const unsigned long long a = (unsigned long long)base;
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)a);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(a >> 32));
    return __builtin_amdgcn_make_buffer_rsrc((void *)(((unsigned long long)hi << 32) | lo), 0, 0x7fffffff, 0x00020000);
}
template <bool COH>
__device__ __forceinline__ uint4 ld16_at(const uint4 *base, uint32_t idx)
{
    if (!COH) return base[idx];
    u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(wave_buffer(base), (int)(idx * 16u), 0, kAuxCoherent);
    return make_uint4(v.x, v.y, v.z, v.w);
}
// 16 bytes that a block of the same launch on the same XCD has stored: past the vector cache, from the L2 that the two share
constexpr int kAuxNear = 16;  // sc1
__device__ __forceinline__ u32x4_t ld16_near(const void *base, uint32_t byte)
{
    return __builtin_amdgcn_raw_buffer_load_b128(wave_buffer(base), (int)byte, 0, kAuxNear);
}
template <bool COH>
__device__ __forceinline__ uint2 ld8_at(const uint2 *base, uint32_t idx)
{
    if (!COH) return base[idx];
    u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(wave_buffer(base), (int)(idx * 8u), 0, kAuxCoherent);
    return make_uint2(v.x, v.y);
}
template <bool COH>
__device__ __forceinline__ float ldf_at(const float *base, uint32_t idx)
{
    if (!COH) return base[idx];
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(wave_buffer(base), (int)(idx * 4u), 0, kAuxCoherent));
}

// threadIdx.x as a value the optimiser treats as new at every call.  In the persistent kernel,
// lane-dependent offsets derived from the plain threadIdx.x are loop invariant over the layers: they
// get computed once up front, by the dozen, and then live in scratch memory.
__device__ __forceinline__ int fresh_tid()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// Block barrier that orders LDS traffic only.  __syncthreads() also waits for every outstanding
// global load of the wave, which would drain the weight prefetch at each tile boundary.
__device__ __forceinline__ void block_sync_lds() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Wait until this wave's outstanding global stores have been acknowledged.
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Value of lane + 8 / lane - 8 within each row of 16 lanes, as a DPP move on the vector ALU
// (no trip through the LDS crossbar).  Lanes whose source falls outside the row read 0.
__device__ __forceinline__ float row_down8(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x108, 0xF, 0xF, true));
}
__device__ __forceinline__ float row_up8(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x118, 0xF, 0xF, true));
}

// Maximum / sum over the four lanes l, l ^ 16, l ^ 32, l ^ 48 (one lane of each row of 16), the same value in
// all four: two row swaps on the vector ALU (v_permlane16_swap exchanges the odd rows of its first operand
// with the even rows of its second, v_permlane32_swap the upper half with the lower half), no trip through
// LDS.  The sum adds in the order of the xor-16, xor-32 butterfly.
__device__ __forceinline__ float rows_max(float v)
{
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float rows_sum(float v)
{
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}
// Window class: how many 16-row MFMA slots a window of M rows occupies (8 = half a tile).
__host__ __device__ __forceinline__ int window_class(int M) { return M <= 8 ? 8 : (M <= 16 ? 16 : 32); }

// The MFMA GEMMs take their activation operand as two bf16 terms, v ~= hi + lo
// (hi = bf16(v), lo = bf16(v - hi)), which keeps ~16 mantissa bits of the fp32
// activation, laid out in MFMA B-fragment order Xp[k-step][frag][lane][8]:
// lane = 16 * kg + slot holds columns 32 * ks + 8 * kg .. + 8 of the row in `slot`.
//   class 8:  one fragment; slot m = hi of row m, slot m + 8 = lo of row m;
//   class 16: fragments (hi, lo) of rows 0..15;
//   class 32: fragments (hi, lo) of rows 0..15, then (hi, lo) of rows 16..31;
//   packed_class(nf), nf >= 2: nf fragments in the class-8 arrangement, fragment f holding rows 8 f .. 8 f + 7
//   (slot m % 8 = hi, slot m % 8 + 8 = lo): the one-kernel step's form for windows of more than 8 rows.
// Returns the bf16-element offset of (row m, column k, hi|lo).
__host__ __device__ constexpr int packed_class(int nf) { return nf == 1 ? 8 : 1000 + nf; }
__host__ __device__ __forceinline__ size_t xp_offset(int cls, int m, int k, int lo)
{
    const int ks = k >> 5, kg = (k >> 3) & 3, j = k & 7;
    int nt, frag, slot;
    if (cls == 8) { nt = 1; frag = 0; slot = m + 8 * lo; }
    else if (cls >= 1000) { nt = cls - 1000; frag = m >> 3; slot = (m & 7) + 8 * lo; }
    else { nt = cls >> 3; frag = 2 * (m >> 4) + lo; slot = m & 15; }
    return ((((size_t)ks * nt + frag) * 64) + (size_t)kg * 16 + slot) * 8 + j;
}

// A step's tokens, passed to the kernels by value: nothing is uploaded before a step.
constexpr int kMaxRows = 32;   // ANPD_MAX_WINDOW
struct StepTokens {
    int32_t t[kMaxRows];
};

// Puts what a step needs in device memory - a draft tree, the sequences of a batch - there from the kernel's arguments.
// (Copies from pinned memory, two for a batch, are launches of their own, and longer ones.)   grid: 1 block
constexpr int kUploadWords = 32 + 32 * 8;
struct UploadWords {
    uint32_t w[kUploadWords];
};
__global__ __launch_bounds__(kUploadWords) void upload_kernel(uint32_t *__restrict__ dst, UploadWords words, int n)
{
    if ((int)threadIdx.x < n) dst[threadIdx.x] = words.w[threadIdx.x];
}

// Page layout of the generic path: [page][layer][k|v][head][token in page][head_dim].
__device__ __forceinline__ size_t kv_offset(int page, int layer, int n_layers, int kv, int head, int n_heads,
                                            int tok_in_page, int page_tokens, int head_dim)
{
    return ((((size_t)page * n_layers + layer) * 2 + kv) * n_heads + head) * ((size_t)page_tokens * head_dim) +
           (size_t)tok_in_page * head_dim;
}

// ------------------------------------------------------------------ embed

// x[r][:] = E[token[r]][:]   grid: rows (at most kMaxRows)
template <typename WT>
__global__ __launch_bounds__(256) void embed_kernel(const WT *__restrict__ E, StepTokens tok, float *__restrict__ x, int d)
{
    int r = blockIdx.x;
    const WT *src = E + (size_t)tok.t[r] * d;
    for (int i = threadIdx.x; i < d; i += blockDim.x) x[(size_t)r * d + i] = load_f32(src, (size_t)i);
}

// ------------------------------------------------ GEMM (fp32 matrix cores)
//
// Y[M][N] = X[M][K] * W[N][K]^T with exact fp32 products on v_mfma_f32_16x16x4_f32, weights (fp32 or bf16)
// row-major as the caller gave them.  Block = 8 waves on 16 output features (two times 16 where the epilogue
// pairs them) x 16 or 32 rows; wave w takes the 128-byte chunks w, w + 8, ... of a weight row (32 columns of fp32, 64
// of bf16), lane (r, kg) holding 32 bytes of weight row r and the same columns of window row r, i.e. an MFMA
// contracts one column of each of four lanes.  A wave's loads of two or three chunks are in flight together.  The partial tiles meet in LDS and are
// added in pairs.  An element's sums do not depend on the other rows, on M or on the block's row count.
//
// At the shapes this path is made for (d 256, FFN 688) every kernel is a chain of latencies, so the step is cut
// into as few launches as the grid-wide dependencies allow: RMSNorm is folded in (x * gain goes into the product,
// the block sums x^2 of its rows beside it, 1 / rms scales the result), and so are rotary embedding and cache
// write, residual add and SwiGLU.  One layer is five launches where one per operation took eleven, and a launch
// takes 3-4 us instead of 11 (dot products with a butterfly over the lanes per output: 40 us at 32 rows, which
// it took eight at a time).  The first QKV of a step looks its rows up in the embedding table as well.
enum { GEN_PLAIN = 0, GEN_QKV = 1, GEN_RESIDUAL = 2, GEN_GATE_UP = 3, GEN_LOGITS = 4 };
__host__ __device__ constexpr bool gen_norm(int mode) { return mode == GEN_QKV || mode == GEN_GATE_UP || mode == GEN_LOGITS; }
__host__ __device__ constexpr bool gen_pairs(int mode) { return mode == GEN_QKV || mode == GEN_GATE_UP; }

struct GenArgs {
    const float *X;       // [M][K]
    int M, K;
    const void *W0, *W1, *W2;   // PLAIN, LOGITS, RESIDUAL: W0; GATE_UP: gate, up; QKV: wq, wk, wv
    const void *gain;     // QKV, GATE_UP, LOGITS: the RMSNorm of X that is folded in
    float eps;
    float *Y;             // PLAIN, LOGITS: output; QKV: rotated q; RESIDUAL: updated in place; GATE_UP: silu(gate) * up
    int ldy;
    // QKV
    const float2 *rope;
    void *pool;
    const int32_t *page_table, *len_ptr;
    const int32_t *depth; // draft tree: a row's rotary position is length + depth (nullable)
    int layer, n_layers, n_heads, n_kv_heads, head_dim, page_tokens;
    // first QKV of a step
    const void *embed;    // [vocab][K]: X is the window's rows of it
    float *x;             // [M][K], which they are written to
};

// eight weights as they lie in memory
template <typename WT>
struct Raw8;
template <>
struct Raw8<float> {
    float4 a, b;
    __device__ __forceinline__ void clear() { a = b = make_float4(0.f, 0.f, 0.f, 0.f); }
    __device__ __forceinline__ void load(const float *p) { a = *reinterpret_cast<const float4 *>(p); b = *reinterpret_cast<const float4 *>(p + 4); }
    __device__ __forceinline__ float at(int j) const { const float4 &v = j < 4 ? a : b; return (j & 3) == 0 ? v.x : ((j & 3) == 1 ? v.y : ((j & 3) == 2 ? v.z : v.w)); }
};
template <>
struct Raw8<bf16_t> {
    uint4 a;
    __device__ __forceinline__ void clear() { a = make_uint4(0, 0, 0, 0); }
    __device__ __forceinline__ void load(const bf16_t *p) { a = *reinterpret_cast<const uint4 *>(p); }
    __device__ __forceinline__ float at(int j) const
    {
        const uint32_t v = (j >> 1) == 0 ? a.x : ((j >> 1) == 1 ? a.y : ((j >> 1) == 2 ? a.z : a.w));
        return __uint_as_float(j & 1 ? v & 0xffff0000u : v << 16);
    }
};

// FEW: forms for a few rows of bf16 weights and blocks for several rounds of the chip, one chunk in flight per wave and
// three or four blocks per compute unit instead of several chunks and two.  FEW_ROWS_LDS keeps the window's rows in LDS: read
// from memory they are two thirds of a wave's loads, and return behind the weights.  See launch_gen_few.  (O and down, of
// one or two blocks per compute unit, take the rows in LDS only and keep their chunks.)
// Chunks in flight otherwise: what the blocks of a compute unit have registers for.  (One more in the bf16 LM head and
// QKV spills 21 and 32 registers: LM head of the 7B, 13B and ChatGLM3 shapes, 1 row, 129 -> 75, 162 -> 92, 247 -> 141 us;
// two layers' QKV 82 -> 74, 103 -> 92, 50 -> 48.)   An element's sums are the same in all forms.
// grid: (features / 16, or pairs of 16; ceil(M / (16 RT)))
enum { FEW_NO = 0, FEW_ROWS = 1, FEW_ROWS_LDS = 2 };
struct GenAttnArgs {
    const float *q;
    int q_stride;
    const void *pool;
    const int32_t *page_table, *len_ptr;
    int M, layer, n_layers, n_heads, n_kv_heads, page_tokens, row0, part_rows, max_splits, head_dim;
    float scale;
    float *part;
    uint32_t *counter;
    float *att;
    const uint32_t *row_mask;   // draft tree: nullable
};
// Block (bx, by) of such a grid.  tok: the first QKV of a step, whose rows are looked up in the embedding table (null otherwise).
// ONE: what the block reads of X comes from blocks of the same launch on the same XCD (read past the vector cache, from
// their L2); the first weights are requested, then `wait` says that X is there.  Every wave calls it once.  ONE_U: chunks in flight then.
// SPLITS > 0 (with ONE): X is attention's output, merged here from the partial results of up to that many splits.
template <int MODE, int RT>
struct GenShared {
    float red[8][gen_pairs(MODE) ? 2 : 1][RT][64][4];
    float ssq[8][RT][16];
};
// Columns k .. k + 7 of attention's output of row `row`: the splits' partial results, which blocks of the same launch on the same XCD have
// stored, merged in increasing order, as attn_gen_block does.
template <int SPLITS>
__device__ __forceinline__ void gen_merge8(const GenAttnArgs &a, int len, int row, int k, f32x4 &lo, f32x4 &hi)
{
    const int dh = a.head_dim, head = k / dh, e = k - head * dh, ns = (len + row) / kAttnSplit + 1;
    const uint32_t slot0 = (uint32_t)(head * a.max_splits) * (uint32_t)a.part_rows + (uint32_t)(row - a.row0), stride = (uint32_t)a.part_rows;
    const float *ps = a.part + (size_t)a.n_heads * a.max_splits * a.part_rows * dh;
    f32x4 v0[SPLITS], v1[SPLITS];
    u32x2_t st[SPLITS];
#pragma unroll
    for (int s = 0; s < SPLITS; ++s) {
        const uint32_t at = slot0 + (uint32_t)(s < ns ? s : 0) * stride;
        v0[s] = __builtin_bit_cast(f32x4, ld16_near(a.part, (at * (uint32_t)dh + (uint32_t)e) * 4u));
        v1[s] = __builtin_bit_cast(f32x4, ld16_near(a.part, (at * (uint32_t)dh + (uint32_t)e + 4u) * 4u));
        st[s] = __builtin_amdgcn_raw_buffer_load_b64(wave_buffer(ps), (int)(at * 8u), 0, kAuxNear);
    }
    float g = kMasked;
#pragma unroll
    for (int s = 0; s < SPLITS; ++s) g = fmaxf(g, __uint_as_float(st[s][0]));   // (a split beyond the last is the first again)
    float dn = 0.f;
    lo = hi = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < SPLITS; ++s) {
        if (s >= ns) continue;
        const float wgt = expf(__uint_as_float(st[s][0]) - g);
        dn = fmaf(wgt, __uint_as_float(st[s][1]), dn);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            lo[i] = fmaf(wgt, v0[s][i], lo[i]);
            hi[i] = fmaf(wgt, v1[s][i], hi[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) { lo[i] /= dn; hi[i] /= dn; }
}
struct NoWait {
    __device__ __forceinline__ void operator()() const {}
    __device__ __forceinline__ void publish() const {}   // called by every wave before the block meets again
};
template <typename WT, int MODE, int RT, int FEW, bool FIRST, bool ONE = false, int ONE_U = 1, int SPLITS = 0, typename Wait = NoWait>
__device__ __forceinline__ void gemm_gen_block(const GenArgs &a, const int32_t *tok, int bx, int by, GenShared<MODE, RT> &sh, const Wait &wait = Wait(),
                                               const GenAttnArgs *parts = nullptr)
{
    constexpr int NW = gen_pairs(MODE) ? 2 : 1, S = sizeof(WT) == 2 ? 2 : 1, WAVES = 8,
                  U = ONE ? ONE_U : (FEW && MODE != GEN_RESIDUAL) || (S == 2 && RT == 1 && MODE == GEN_QKV) ? 1 : (S == 2 && (NW == 2 || RT == 2 || MODE == GEN_LOGITS) ? 2 : 3);
    static_assert(FEW == FEW_NO || RT == 1, "one row tile");
    extern __shared__ float x_lds[];   // FEW_ROWS_LDS: [M][K]
    constexpr bool NORM = gen_norm(MODE);
    auto &red = sh.red;
    auto &ssq = sh.ssq;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = lane & 15, kg = lane >> 4;
    const int K = a.K, m0 = by * 16 * RT;

    // the weight rows of this block's tiles
    const WT *w[NW];
    int sect = 0, head = 0, i0 = 0;   // QKV: q | k | v, its head, the pair's first dimension
    if (MODE == GEN_QKV) {
        const int half = a.head_dim / 2, per_head = half / 16;
        head = bx / per_head;
        i0 = 16 * (bx - head * per_head);
        sect = head < a.n_heads ? 0 : (head < a.n_heads + a.n_kv_heads ? 1 : 2);
        head -= sect == 0 ? 0 : (sect == 1 ? a.n_heads : a.n_heads + a.n_kv_heads);
        const void *wq = a.W0, *wk = a.W1, *wv = a.W2;   // (values: a choice among the arguments' places would put them all into scratch memory)
        const WT *W = (const WT *)(sect == 0 ? wq : (sect == 1 ? wk : wv)) + (size_t)(head * a.head_dim + i0 + r) * K;
        w[0] = W;
        w[NW - 1] = W + (size_t)half * K;
    } else {
        w[0] = (const WT *)a.W0 + (size_t)(bx * 16 + r) * K;
        if (NW == 2) w[NW - 1] = (const WT *)a.W1 + (size_t)(bx * 16 + r) * K;
    }
    const WT *gain = (const WT *)a.gain;
    const WT *row[RT];   // FIRST: the embedding of row m0 + 16 t + r
#pragma unroll
    for (int t = 0; t < RT; ++t) row[t] = FIRST && m0 + 16 * t + r < a.M ? (const WT *)a.embed + (size_t)tok[m0 + 16 * t + r] * K : nullptr;
    // QKV: what the epilogue of the finishing waves needs besides the sums, requested first: position -> page, angles
    int pos = 0, page = 0;
    float2 cs[4];
    if (MODE == GEN_QKV && wave < RT && m0 + 16 * wave + r < a.M) {
        const int m = m0 + 16 * wave + r, len = *a.len_ptr;
        pos = len + m;   // the row's cache slot
        if (sect > 0) page = a.page_table[pos / a.page_tokens];
        if (sect < 2) {
            const float2 *c = a.rope + (size_t)(a.depth ? len + a.depth[m] : pos) * (a.head_dim / 2) + i0 + 4 * kg;
#pragma unroll
            for (int q = 0; q < 4; ++q) cs[q] = c[q];
        }
    }

    // several chains of sums side by side: shorter chains round less (the result is as close to the 64-bit one as
    // the dot products' was) and do not wait for one another
    constexpr int NA = NW == 2 ? 4 : 8;
    f32x4 acc[NA][NW][RT];
    float ss[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        ss[t] = 0.f;
#pragma unroll
        for (int n = 0; n < NW; ++n)
#pragma unroll
            for (int q = 0; q < NA; ++q) acc[q][n][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    if (FEW == FEW_ROWS_LDS) {
        for (int i = 4 * (int)threadIdx.x; i < a.M * K; i += 4 * 512) *reinterpret_cast<float4 *>(x_lds + i) = *reinterpret_cast<const float4 *>(a.X + i);
        __syncthreads();
    }
    f32x4 old = {0.f, 0.f, 0.f, 0.f};   // (ONE, RESIDUAL)
    const int len = SPLITS > 0 ? *parts->len_ptr : 0;
    for (int c0 = wave; c0 * 32 * S < K || (ONE && c0 == wave); c0 += WAVES * U) {
        Raw8<WT> wv[U][S][NW];
        Raw8<WT> gv[U][S];
        float xv[U][S][RT][8];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int k = (c0 + u * WAVES) * 32 * S + 8 * (S * kg + s);
#pragma unroll
                for (int n = 0; n < NW; ++n) wv[u][s][n].clear();
                gv[u][s].clear();
#pragma unroll
                for (int i = 0; i < 8; ++i)
#pragma unroll
                    for (int t = 0; t < RT; ++t) xv[u][s][t][i] = 0.f;
                if (k < K) {
#pragma unroll
                    for (int n = 0; n < NW; ++n) wv[u][s][n].load(w[n] + k);
#pragma unroll
                    for (int t = 0; t < RT; ++t)
                        if (m0 + 16 * t + r < a.M) {
                            if (FIRST) load8(row[t] + k, xv[u][s][t]);
                            else if (!ONE) load8((FEW == FEW_ROWS_LDS ? x_lds : a.X) + (size_t)(m0 + 16 * t + r) * K + k, xv[u][s][t]);
                        }
                    if (NORM) gv[u][s].load(gain + k);
                }
            }
        if constexpr (ONE) {
            if (c0 == wave) {
                wait();
                const int t = wave, m = m0 + 16 * t + r;
                if (MODE == GEN_RESIDUAL && t < RT && m < a.M)
                    old = __builtin_bit_cast(f32x4, ld16_near(a.Y, (uint32_t)(m * a.ldy + bx * 16 + 4 * kg) * 4u));
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    const int k = (c0 + u * WAVES) * 32 * S + 8 * (S * kg + s);
#pragma unroll
                    for (int t = 0; t < RT; ++t)
                        if (!FIRST && k < K && m0 + 16 * t + r < a.M) {
                            f32x4 lo, hi;
                            if constexpr (SPLITS > 0) {
                                gen_merge8<SPLITS>(*parts, len, m0 + 16 * t + r, k, lo, hi);
                            } else {
                                const uint32_t at = ((uint32_t)(m0 + 16 * t + r) * (uint32_t)K + (uint32_t)k) * 4u;
                                lo = __builtin_bit_cast(f32x4, ld16_near(a.X, at));
                                hi = __builtin_bit_cast(f32x4, ld16_near(a.X, at + 16u));
                            }
#pragma unroll
                            for (int i = 0; i < 4; ++i) { xv[u][s][t][i] = lo[i]; xv[u][s][t][4 + i] = hi[i]; }
                        }
                }
        }
        if (FIRST && bx == 0) {   // the first block leaves the rows where the residual stream begins
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    const int k = (c0 + u * WAVES) * 32 * S + 8 * (S * kg + s);
#pragma unroll
                    for (int t = 0; t < RT; ++t)
                        if (k < K && m0 + 16 * t + r < a.M) {
                            f32x4 *x = reinterpret_cast<f32x4 *>(a.x + (size_t)(m0 + 16 * t + r) * K + k);
                            x[0] = (f32x4){xv[u][s][t][0], xv[u][s][t][1], xv[u][s][t][2], xv[u][s][t][3]};
                            x[1] = (f32x4){xv[u][s][t][4], xv[u][s][t][5], xv[u][s][t][6], xv[u][s][t][7]};
                        }
                }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
#pragma unroll
                    for (int t = 0; t < RT; ++t) {
                        float x = xv[u][s][t][j];
                        if (NORM) {
                            ss[t] = fmaf(x, x, ss[t]);
                            x *= gv[u][s].at(j);
                        }
#pragma unroll
                        for (int n = 0; n < NW; ++n)
                            acc[j % NA][n][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[u][s][n].at(j), x, acc[j % NA][n][t], 0, 0, 0);
                    }
                }
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        ss[t] = rows_sum(ss[t]);
        if (kg == 0) ssq[wave][t][r] = ss[t];
#pragma unroll
        for (int n = 0; n < NW; ++n) {
            f32x4 s = (acc[0][n][t] + acc[1][n][t]) + (acc[2][n][t] + acc[3][n][t]);
            if (NA == 8) s += (acc[NA - 4][n][t] + acc[NA - 3][n][t]) + (acc[NA - 2][n][t] + acc[NA - 1][n][t]);
            *reinterpret_cast<f32x4 *>(red[wave][n][t][lane]) = s;
        }
    }
    // (the one launch: the item's flag stands for the rows that every wave has stored above; the waves that set it wait for their own stores
    // only.  By now a wave's loads have long returned: only the first block waits at all)
    if (ONE && FIRST) wait_stores();
    wait.publish();
    __syncthreads();
    if (wave >= RT) return;
    // wave t finishes row tile t: lane (m, kg) has features 4 kg .. 4 kg + 3 of row m0 + 16 t + m
    const int t = wave, m = m0 + 16 * t + r;
    f32x4 y[NW];
#pragma unroll
    for (int n = 0; n < NW; ++n) {
        f32x4 p[WAVES];
#pragma unroll
        for (int v = 0; v < WAVES; ++v) p[v] = *reinterpret_cast<const f32x4 *>(red[v][n][t][lane]);
        y[n] = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
    }
    if (NORM) {
        float q[WAVES];
#pragma unroll
        for (int v = 0; v < WAVES; ++v) q[v] = ssq[v][t][r];
        const float tot = ((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7]));
        const float rinv = 1.0f / sqrtf(tot / (float)K + a.eps);
#pragma unroll
        for (int n = 0; n < NW; ++n) y[n] = y[n] * rinv;
    }
    if (m >= a.M) return;
    const int f = bx * 16 + 4 * kg;   // (all but QKV)
    if (MODE == GEN_PLAIN || MODE == GEN_LOGITS) {
        // (the caller's buffer need not be aligned for wide stores)
#pragma unroll
        for (int i = 0; i < 4; ++i) a.Y[(size_t)m * a.ldy + f + i] = y[0][i];
    } else if (MODE == GEN_RESIDUAL) {
        f32x4 *x = reinterpret_cast<f32x4 *>(a.Y + (size_t)m * a.ldy + f);
        *x = (ONE ? old : *x) + y[0];
    } else if (MODE == GEN_GATE_UP) {
        f32x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = y[0][i] / (1.0f + expf(-y[0][i])) * y[NW - 1][i];
        *reinterpret_cast<f32x4 *>(a.Y + (size_t)m * a.ldy + f) = o;
    } else {
        const int half = a.head_dim / 2, i = i0 + 4 * kg;
        f32x4 lo = y[0], hi = y[NW - 1];
        if (sect < 2) {   // rotate the pairs (i, i + head_dim / 2) by the row's position
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                lo[q] = y[0][q] * cs[q].x - y[NW - 1][q] * cs[q].y;
                hi[q] = y[NW - 1][q] * cs[q].x + y[0][q] * cs[q].y;
            }
        }
        if (sect == 0) {
            float *q = a.Y + (size_t)m * a.ldy + head * a.head_dim + i;
            *reinterpret_cast<f32x4 *>(q) = lo;
            *reinterpret_cast<f32x4 *>(q + half) = hi;
        } else {
            const size_t o = kv_offset(page, a.layer, a.n_layers, sect - 1, head, a.n_kv_heads, pos % a.page_tokens, a.page_tokens, a.head_dim) + i;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                store_kv((WT *)a.pool, o + q, lo[q]);
                store_kv((WT *)a.pool, o + half + q, hi[q]);
            }
        }
    }
}

template <typename WT, int MODE, int RT, int FEW = FEW_NO>
__global__ __launch_bounds__(512, FEW && MODE != GEN_RESIDUAL ? (gen_norm(MODE) ? 6 : 8) : (sizeof(WT) == 2 && RT == 1 ? 4 : 2)) void gemm_gen_kernel(GenArgs a)
{
    __shared__ GenShared<MODE, RT> sh;
    gemm_gen_block<WT, MODE, RT, FEW, false>(a, nullptr, blockIdx.x, blockIdx.y, sh);
}
// The first QKV of a step: its rows come from the embedding table, without a launch in front of it that copies them.  A step of
// a small model is a chain of launches of 3-4 us: 67.7 -> 65.5 us of kernels (traced) and one launch less at d 256, two layers,
// fp32, 5 rows, where the step as a whole gains no more than its runs differ, 3 to 9 % of some 86 us.  Prompts keep the launch: their
// pieces have up to 256 rows, whose tokens do not fit a kernel's arguments.
template <typename WT, int RT>
__global__ __launch_bounds__(512, sizeof(WT) == 2 && RT == 1 ? 4 : 2) void gemm_gen_first_kernel(GenArgs a, StepTokens tok)
{
    __shared__ GenShared<GEN_QKV, RT> sh;
    gemm_gen_block<WT, GEN_QKV, RT, FEW_NO, true>(a, tok.t, blockIdx.x, blockIdx.y, sh);
}

// ------------------------------------------------------------- attention
//
// Window-causal attention of the M query rows over the paged cache.  Keys are
// cut into fixed splits of kAttnSplit absolute positions; block (head, split, 16-row group), one wave per 16
// keys, computes for each row the split's score maximum, sum of exponentials and unnormalised weighted V sum on
// the fp32 matrix cores; the last block of a (head, row group) merges the splits of its rows in increasing
// order.  Row r sees keys 0..len + r; keys it must not see get
// weight exactly 0 and, where their V is not finite, take no part at all, so a row's numbers do not depend on M or on the
// rows behind it.
// A long window is gone through in launches of at most part_rows rows, of which this one takes those from row0 on.
// part: outputs [head][split][part_rows][DH], then (maximum, denominator) [head][split][part_rows][2].
// counter: [row group][head], a 256-byte line each, zero between calls.
// grid: (n_heads, n_splits, row groups), 4 waves.
template <int DH>
struct GenAttnShared {
    float red[kAttnSplit / 16][DH / 16][64][4];
    float wmax[kAttnSplit / 16][16], wden[kAttnSplit / 16][16];
    bool last;
};
// Block (head, split, group).  ONE: as in gemm_gen_block, eight waves, of which four have keys; those of earlier steps are requested
// before `wait`.
// merge: by the last block; else the partial results are what it leaves.
template <typename KT, int DH, bool ONE = false, typename Wait = NoWait>
__device__ __forceinline__ void attn_gen_block(const GenAttnArgs &a, int head, int split, int group, GenAttnShared<DH> &sh, const Wait &wait = Wait(), bool merge = true)
{
    constexpr int NC = DH / 16, WAVES = kAttnSplit / 16;
    auto &red = sh.red;
    auto &wmax = sh.wmax;
    auto &wden = sh.wden;
    const KT *pool = (const KT *)a.pool;
    const int32_t *page_table = a.page_table;
    const uint32_t *row_mask = a.row_mask;
    const int M = a.M, layer = a.layer, n_layers = a.n_layers, n_heads = a.n_heads, n_kv_heads = a.n_kv_heads, page_tokens = a.page_tokens;
    const int row0 = a.row0, m0 = row0 + 16 * group;
    const int kvh = head / (n_heads / n_kv_heads);   // the key / value head this query head reads
    const int L = *a.len_ptr;
    const int n_splits = (L + (m0 + 16 < M ? m0 + 16 : M) + kAttnSplit - 1) / kAttnSplit;
    if (split >= n_splits) {  // no row of the group sees a key of this split
        wait();
        wait.publish();
        return;
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = lane & 15, kg = lane >> 4;
    const int key0 = split * kAttnSplit + 16 * wave, m = m0 + r;

    // every load of the wave goes out together: lane (r, kg) takes columns 16 c + 4 kg .. + 4 of key key0 + r and of
    // query row m0 + r, and dimensions 16 c + r of the values of keys key0 + 4 kg .. + 4
    float kf[NC][4], qf[NC][4], vf[NC][4];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) { kf[c][i] = 0.f; qf[c][i] = 0.f; vf[c][i] = 0.f; }
    // the wave's keys' pages (behind the last key, the last key's), then keys lo .. hi - 1
    // (All five are waited for here, in front of the branches around the loads of keys and values: for a value loaded in one branch and used in
    // another the compiler waits for every load in between.  By rocprofv3, 5 rows: d 1024 at 600 positions 11.1 -> 8.9 us, eight layers of d 256 at
    // 2000 14.1 -> 13.2; 17 rows, d 384 with heads of 128 at 600, 16.3 -> 14.6; 128 rows, d 256 9.2 -> 7.8.)
    auto page_of = [&](int key) __attribute__((always_inline)) { return page_table[(key < L + M ? key : L + M - 1) / page_tokens]; };
    int page_k = page_of(key0 + r), page_v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) page_v[i] = page_of(key0 + 4 * kg + i);
    asm volatile("" : "+v"(page_k), "+v"(page_v[0]), "+v"(page_v[1]), "+v"(page_v[2]), "+v"(page_v[3]));
    // (ONE: the window's own, which other blocks of the launch have stored, past the vector cache, as all that crosses blocks)
    static_assert(!ONE || sizeof(KT) == 4, "ONE: fp32 caches");
    auto load_kv = [&](int lo, int hi, auto own) __attribute__((always_inline)) {
        constexpr bool past = ONE && decltype(own)::value;
        if (key0 + r >= lo && key0 + r < hi) {
            const KT *kr = pool + kv_offset(page_k, layer, n_layers, 0, kvh, n_kv_heads, (key0 + r) % page_tokens, page_tokens, DH) + 4 * kg;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                if (past) {
                    const uint4 v = ldc16<true>(reinterpret_cast<const uint4 *>(kr + 16 * c));
                    kf[c][0] = __uint_as_float(v.x); kf[c][1] = __uint_as_float(v.y); kf[c][2] = __uint_as_float(v.z); kf[c][3] = __uint_as_float(v.w);
                    continue;
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) kf[c][i] = load_f32(kr, (size_t)(16 * c + i));
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int key = key0 + 4 * kg + i;
            if (key >= lo && key < hi) {
                const KT *vr = pool + kv_offset(page_v[i], layer, n_layers, 1, kvh, n_kv_heads, key % page_tokens, page_tokens, DH) + r;
#pragma unroll
                for (int c = 0; c < NC; ++c) vf[c][i] = past ? ldc<true>(reinterpret_cast<const float *>(vr) + 16 * c) : load_f32(vr, (size_t)(16 * c));
            }
        }
    };
    const bool mine = !ONE || wave < WAVES;   // (a block of the one launch has more waves than this needs)
    if (ONE) {
        if (mine) load_kv(0, L, std::false_type());
        wait();
    }
    if (mine && m < M) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const size_t at = (size_t)m * a.q_stride + head * DH + 4 * kg + 16 * c;
            f32x4 v;
            if (ONE) v = __builtin_bit_cast(f32x4, ld16_near(a.q, (uint32_t)at * 4u));
            else v = *reinterpret_cast<const f32x4 *>(a.q + at);
#pragma unroll
            for (int i = 0; i < 4; ++i) qf[c][i] = v[i];
        }
    }
    if (mine) load_kv(ONE ? L : 0, L + M, std::true_type());
    wait.publish();
    // ---- scores: lane (r, kg) has keys key0 + 4 kg + i of row m
    // (eight chains, as in the GEMM)
    f32x4 sq[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        sq[j] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = j & 1; c < NC; c += 2) sq[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][j >> 1], qf[c][j >> 1], sq[j], 0, 0, 0);
    }
    const f32x4 s = ((sq[0] + sq[1]) + (sq[2] + sq[3])) + ((sq[4] + sq[5]) + (sq[6] + sq[7]));
    const uint32_t vis = row_mask && m < M ? row_mask[m] : 0u;
    // whether row `row`, whose mask is `mask`, sees key `key`
    auto sees = [&](int row, uint32_t mask, int key) __attribute__((always_inline)) {
        return row_mask ? key < L || (key - L < 32 && ((mask >> (key - L)) & 1u)) : key <= L + row;
    };
    float p[4], mx = kMasked;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        p[i] = m < M && sees(m, vis, key0 + 4 * kg + i) ? s[i] * a.scale : kMasked;
        mx = fmaxf(mx, p[i]);
    }
    mx = rows_max(mx);
    if (mine && kg == 0) wmax[wave][r] = mx;
    __syncthreads();
    float bm = wmax[0][r], den = 0.f;
#pragma unroll
    for (int v = 1; v < WAVES; ++v) bm = fmaxf(bm, wmax[v][r]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        p[i] = p[i] > 0.5f * kMasked ? expf(p[i] - bm) : 0.f;
        den += p[i];
    }
    den = rows_sum(den);
    if (mine && kg == 0) wden[wave][r] = den;
    // ---- weighted V: lane (r, kg) has dimensions 16 c + 4 kg .. + 4 of row m
    // A weight of 0 does not keep out what is not finite.  Where a key that some row must not see has such a V, the rows
    // are taken one at a time, each over the keys that it sees.
    bool apart = false;
    if (key0 + 15 > L + (row_mask ? 0 : m0)) {
        float z[2] = {0.f, 0.f};   // not finite if a value is not (or a product of two is beyond fp32: no harm)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            z[0] = fmaf(vf[c][0], vf[c][1], z[0]);
            z[1] = fmaf(vf[c][2], vf[c][3], z[1]);
        }
        apart = __builtin_amdgcn_ballot_w64(!(fabsf(z[0]) + fabsf(z[1]) < INFINITY)) != 0;
    }
    auto weigh = [&](int c, const bool *seen) __attribute__((always_inline)) {
        f32x4 o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(!seen || seen[i] ? vf[c][i] : 0.f, p[i], (f32x4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        return (o[0] + o[1]) + (o[2] + o[3]);
    };
    if (!mine) {
    } else if (!apart) {
#pragma unroll
        for (int c = 0; c < NC; ++c) *reinterpret_cast<f32x4 *>(red[wave][c][lane]) = weigh(c, nullptr);
    } else {
        for (int q = 0; q < 16; ++q) {
            const uint32_t vis_q = (uint32_t)__builtin_amdgcn_readlane((int)vis, q);   // (lane q has row m0 + q)
            bool seen[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) seen[i] = sees(m0 + q, vis_q, key0 + 4 * kg + i);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const f32x4 o = weigh(c, seen);
                if (r == q) *reinterpret_cast<f32x4 *>(red[wave][c][lane]) = o;
            }
        }
    }
    __syncthreads();
    const size_t slot0 = ((size_t)head * a.max_splits) * a.part_rows, stride = (size_t)a.part_rows;   // rows of (head, split 0); rows per split
    float *po = a.part, *ps = a.part + (size_t)n_heads * a.max_splits * a.part_rows * DH;
    for (int c = wave; c < NC; c += ONE ? 2 * WAVES : WAVES) {
        f32x4 o = *reinterpret_cast<const f32x4 *>(red[0][c][lane]);
#pragma unroll
        for (int v = 1; v < WAVES; ++v) o += *reinterpret_cast<const f32x4 *>(red[v][c][lane]);
        if (m < M) stc16<!ONE>(po + (slot0 + split * stride + (m - row0)) * DH + 16 * c + 4 * kg, o);
    }
    if (wave == 0 && kg == 0 && m < M) {
        float d = wden[0][r];
#pragma unroll
        for (int v = 1; v < WAVES; ++v) d += wden[v][r];
        stc8<!ONE>(ps + (slot0 + split * stride + (m - row0)) * 2, make_uint2(__float_as_uint(bm), __float_as_uint(d)));
    }
    if (ONE && !merge) return;
    // ---- the last block of this head and row group merges the splits
    wait_stores();
    __syncthreads();
    uint32_t *ctr = a.counter + ((size_t)group * n_heads + head) * 64;
    if (threadIdx.x == 0)
        sh.last = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == (uint32_t)n_splits;
    __syncthreads();
    if (!sh.last) return;
    if (threadIdx.x == 0) st_agent(ctr, 0u);
    constexpr int SB = 8, DQ = DH / 4;
    for (int idx = threadIdx.x; idx < 16 * DQ; idx += ONE ? 512 : 256) {
        const int row = m0 + idx / DQ, e4 = idx % DQ;
        if (row >= M) continue;
        const int ns = (L + row) / kAttnSplit + 1;   // splits that hold keys this row may see
        const uint4 *o4 = reinterpret_cast<const uint4 *>(po);
        const uint2 *s2 = reinterpret_cast<const uint2 *>(ps);
        float g = kMasked;
        for (int s0 = 0; s0 < ns; s0 += SB) {
            float mv[SB];
#pragma unroll
            for (int j = 0; j < SB; ++j) mv[j] = __uint_as_float(ld8_at<true>(s2 + slot0, (uint32_t)((s0 + j < ns ? s0 + j : s0) * stride + (row - row0))).x);
#pragma unroll
            for (int j = 0; j < SB; ++j) g = fmaxf(g, mv[j]);
        }
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
        float dn = 0.f;
        for (int s0 = 0; s0 < ns; s0 += SB) {
            uint4 ov[SB];
            uint2 st[SB];
#pragma unroll
            for (int j = 0; j < SB; ++j) {
                const uint32_t at = (uint32_t)((s0 + j < ns ? s0 + j : s0) * stride + (row - row0));
                ov[j] = ld16_at<true>(o4 + slot0 * DQ, at * DQ + e4);
                st[j] = ld8_at<true>(s2 + slot0, at);
            }
#pragma unroll
            for (int j = 0; j < SB; ++j) {
                if (s0 + j >= ns) continue;
                const float wgt = expf(__uint_as_float(st[j].x) - g);
                dn = fmaf(wgt, __uint_as_float(st[j].y), dn);
                o[0] = fmaf(wgt, __uint_as_float(ov[j].x), o[0]);
                o[1] = fmaf(wgt, __uint_as_float(ov[j].y), o[1]);
                o[2] = fmaf(wgt, __uint_as_float(ov[j].z), o[2]);
                o[3] = fmaf(wgt, __uint_as_float(ov[j].w), o[3]);
            }
        }
        o[0] /= dn; o[1] /= dn; o[2] /= dn; o[3] /= dn;
        *reinterpret_cast<f32x4 *>(a.att + (size_t)row * n_heads * DH + head * DH + 4 * e4) = o;
    }
}
template <typename KT, int DH>
__global__ __launch_bounds__(256) void attn_kernel(GenAttnArgs a)
{
    __shared__ GenAttnShared<DH> sh;
    attn_gen_block<KT, DH>(a, blockIdx.x, blockIdx.y, blockIdx.z, sh);
}

// Appends n rows to the cache's length: a window of a prompt of which only the cache entries are wanted.
__global__ void advance_length_kernel(int32_t *__restrict__ len_ptr, int n)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *len_ptr += n;
}

// ------------------------------------------- argmax + acceptance + commit
//
// Block r finds argmax(logits[r]) (lowest index among equal maxima; a NaN is none); the last block to finish decides what is accepted,
// advances the cache length and writes the result.  KIND:
//   chain: Algorithm 1's rule: a = longest prefix with window[i + 1] == pred[i], next = pred[a], length += before + 1 + a
//     (rejected rows are simply left beyond the length and overwritten later; before: rows of the same prompt piece
//     in front of the first).  mode 1 accepts every row.
//   tree: row r > 0 is accepted iff its parent is and window[r] equals the prediction made at the parent; the deepest
//     accepted row wins (lowest index among equally deep); result[34 + j] = the row at depth j of the accepted path.
//   batch: the chain's rule inside every sequence's own rows, each sequence's length advanced.
// result: [0] = a, [1] = next, [2..2+M) = pred; host_result, host_batch (accepted, next of every sequence): in pinned host
// memory, so that no copy follows.
// One row is one block's loads: 16 bytes per thread and eight of them in flight (one value per thread and load took 14.6 us
// for 17 rows at a vocabulary of 32000 and 24.3 for one at 65024; 7.7 and 8.7 now), and the last block's rules are one
// lane per row or sequence (a launch of its own for a batch or a tree took 9 and 4.5 us more).   grid: M blocks of 1024.
enum { ACCEPT_CHAIN = 0, ACCEPT_TREE = 1, ACCEPT_BATCH = 2 };
// One sequence of a batched step: its cache and the window rows it owns (consecutive rows of the joint window).
struct SeqRef {
    bf16_t *pool;
    const int32_t *page_table;
    int32_t *len_ptr;
    int32_t row0, n_rows;
};
struct AcceptArgs {
    int32_t *result, *host_result, *len_ptr;
    uint32_t *counter;
    int before;                       // chain
    const int32_t *parent, *depth;    // tree
    const SeqRef *seqs;               // batch
    int n_seq;
    int32_t *host_batch;
    uint32_t *launches, *host_launches;   // the one launch of a small model: completed ones, here and in pinned host memory
};
struct AcceptShared {
    float bv[16];
    int bi[16];
    bool last;
};
// window: the rows' tokens.  Returns whether this block applied the rules.
// ONE: the logits come from blocks of the same launch on the same XCD (as in gemm_gen_block).  The caller's buffer may share its first and
// last line with something that was read before they were written, weights say, which this block's vector cache may still hold.
template <int KIND, int THREADS, bool ONE = false>
__device__ __forceinline__ bool argmax_accept_block(const float *__restrict__ logits, int V, int M, const int32_t *window, int mode, const AcceptArgs &a,
                                                    int r, AcceptShared &sh)
{
    auto &bv = sh.bv;
    auto &bi = sh.bi;
    auto &last = sh.last;
    const f32x4 *row = reinterpret_cast<const f32x4 *>(logits + (size_t)r * V);   // (V is a multiple of 16, logits are 16-byte aligned)
    float best = -INFINITY;
    int besti = 0x7fffffff;
    constexpr int U = 8;
    for (int i0 = threadIdx.x; i0 < V / 4; i0 += THREADS * U) {
        f32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + THREADS * u < V / 4) v[u] = ONE ? __builtin_bit_cast(f32x4, ld16_near(row, (uint32_t)(i0 + THREADS * u) * 16u)) : row[i0 + THREADS * u];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i0 + THREADS * u >= V / 4) break;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (v[u][j] > best) { best = v[u][j]; besti = 4 * (i0 + THREADS * u) + j; }   // (never a NaN)
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        float ov = __shfl_xor(best, off, kWave);
        int oi = __shfl_xor(besti, off, kWave);
        if (ov > best || (ov == best && oi < besti)) { best = ov; besti = oi; }
    }
    if ((threadIdx.x & 63) == 0) { bv[threadIdx.x >> 6] = best; bi[threadIdx.x >> 6] = besti; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < THREADS / 64; ++w)
            if (bv[w] > best || (bv[w] == best && bi[w] < besti)) { best = bv[w]; besti = bi[w]; }
        if (besti == 0x7fffffff) besti = 0;   // nothing above -infinity
        st_agent(a.result + 2 + r, (int32_t)besti);
        wait_stores();
        last = __hip_atomic_fetch_add(a.counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)(M - 1);
        st_system(a.host_result + 2 + r, (int32_t)besti);   // (after the counter: its way to the host is long)
    }
    __syncthreads();
    if (!last) return false;
    if (threadIdx.x >= 64) return true;
    const int lane = threadIdx.x;
    const int32_t pred = ld_agent(a.result + 2 + (lane < M ? lane : 0));
    if (KIND == ACCEPT_CHAIN || KIND == ACCEPT_BATCH) {
        // bit m: the token of row m + 1 is not the prediction made at row m
        const unsigned long long wrong = __builtin_amdgcn_ballot_w64(lane + 1 < M && window[lane + 1 < M ? lane + 1 : 0] != pred);
        constexpr bool seq = KIND == ACCEPT_BATCH;
        const bool mine = lane < (seq ? a.n_seq : 1);
        const int r0 = seq && mine ? a.seqs[lane].row0 : 0, n = seq ? (mine ? a.seqs[lane].n_rows : 1) : M;
        const unsigned long long end = 1ull << (n - 1);   // the last row's prediction has no token to match
        const int acc = mode == 0 ? __builtin_ctzll((wrong >> r0) | end) : n - 1;
        const int32_t next = __shfl(pred, r0 + acc, kWave);
        if (mine && seq) {
            st_system(a.host_batch + 2 * lane, (int32_t)acc);
            st_system(a.host_batch + 2 * lane + 1, next);
            *a.seqs[lane].len_ptr += 1 + acc;
        } else if (mine) {
            a.result[0] = acc;
            a.result[1] = next;
            st_system(a.host_result, (int32_t)acc);
            st_system(a.host_result + 1, next);
            *a.len_ptr += a.before + 1 + acc;
        }
    } else {
        const int p = lane > 0 && lane < M ? a.parent[lane] : 0, depth = lane < M ? a.depth[lane] : 0;
        // whether this row's token is the prediction made at its parent
        const int32_t at_parent = __shfl(pred, p, kWave);
        const unsigned long long right = __builtin_amdgcn_ballot_w64(lane > 0 && lane < M && window[lane < M ? lane : 0] == at_parent);
        unsigned long long ok = 1ull;
        int best_row = 0, best_depth = 0;
        for (int q = 1; q < M; ++q) {
            const int parent = __builtin_amdgcn_readlane(p, q), d = __builtin_amdgcn_readlane(depth, q);
            if (((ok >> parent) & 1ull) && ((right >> q) & 1ull)) {
                ok |= 1ull << q;
                if (d > best_depth) { best_row = q; best_depth = d; }
            }
        }
        const int32_t next = __builtin_amdgcn_readlane(pred, best_row);
        for (int q = best_row, j = best_depth; j >= 0; --j) {
            if (lane == 0) {
                a.result[34 + j] = q;
                st_system(a.host_result + 34 + j, (int32_t)q);
            }
            q = __builtin_amdgcn_readlane(p, q);
        }
        if (lane == 0) {
            a.result[0] = best_depth;
            a.result[1] = next;
            st_system(a.host_result, (int32_t)best_depth);
            st_system(a.host_result + 1, next);
            *a.len_ptr += 1 + best_depth;
        }
    }
    if (lane == 0) st_agent(a.counter, 0u);
    return true;
}
template <int KIND>
__global__ __launch_bounds__(1024) void argmax_accept_kernel(const float *__restrict__ logits, int V, int M, StepTokens window,
                                                              int mode, AcceptArgs a)
{
    __shared__ AcceptShared sh;
    argmax_accept_block<KIND, 1024>(logits, V, M, window.t, mode, a, blockIdx.x, sh);
}

// Generic-layout counterpart of kvf_compact_kernel.   grid: n_layers * 2 * n_heads blocks.
template <typename KT>
__global__ __launch_bounds__(128) void kv_compact_kernel(KT *__restrict__ pool, const int32_t *__restrict__ page_table,
                                                          const int32_t *__restrict__ result, int L, int n_layers, int n_heads,
                                                          int head_dim, int page_tokens)
{
    const int head = blockIdx.x % n_heads, kv = (blockIdx.x / n_heads) & 1, layer = blockIdx.x / (2 * n_heads);
    const int a = result[0];
    const int32_t *path = result + 34;
    for (int j = 1; j <= a; ++j) {
        const int src = L + path[j], dst = L + j;
        if (src != dst && (int)threadIdx.x < head_dim) {
            const size_t so = kv_offset(page_table[src / page_tokens], layer, n_layers, kv, head, n_heads, src % page_tokens,
                                        page_tokens, head_dim);
            const size_t dofs = kv_offset(page_table[dst / page_tokens], layer, n_layers, kv, head, n_heads, dst % page_tokens,
                                          page_tokens, head_dim);
            pool[dofs + threadIdx.x] = pool[so + threadIdx.x];
        }
        __syncthreads();
    }
}

// ----------------------------------------------------- cache import/export

// Copies n positions of one layer between fp32 [n][d] arrays and the cache.
template <typename KT, bool TO_CACHE>
__global__ __launch_bounds__(256) void kv_copy_kernel(KT *__restrict__ pool, const int32_t *__restrict__ page_table,
                                                       float *__restrict__ k, float *__restrict__ v, int pos0, int layer,
                                                       int n_layers, int n_heads, int head_dim, int page_tokens)
{
    const int r = blockIdx.x, pos = pos0 + r, d = n_heads * head_dim;
    const int page = page_table[pos / page_tokens], tip = pos % page_tokens;
    for (int e = threadIdx.x; e < d; e += 256) {
        int hd = e / head_dim, i = e - hd * head_dim;
        size_t ko = kv_offset(page, layer, n_layers, 0, hd, n_heads, tip, page_tokens, head_dim) + i;
        size_t vo = kv_offset(page, layer, n_layers, 1, hd, n_heads, tip, page_tokens, head_dim) + i;
        if (TO_CACHE) {
            store_kv(pool, ko, k[(size_t)r * d + e]);
            store_kv(pool, vo, v[(size_t)r * d + e]);
        } else {
            k[(size_t)r * d + e] = load_f32(pool, ko);
            v[(size_t)r * d + e] = load_f32(pool, vo);
        }
    }
}

}  // namespace anpd
