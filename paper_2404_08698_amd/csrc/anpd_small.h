// A step of a small fp32 model as ONE launch that runs on one XCD.
//
// As separate launches such a step is a chain of 12 kernels of 4 to 8 us (two layers, d 256): each a start, a few round
// trips to memory, an end that the next one waits for.  Nothing in it needs more than a few dozen blocks, and blocks of one
// XCD share an L2: what one stores (an ordinary store, acknowledged by that L2) the other reads 0.4 us later, where blocks of
// different XCDs, which meet at the memory side, take 1.1 (measured with one word and its data, going back and forth).
//
// The blocks that happen to run on the chosen XCD hand out the step's work items (the blocks of the separate kernels, same
// code, same bits) by a counter, phase after phase; the others leave at once.  An item requests its weights, waits until
// the phase before is complete, reads its activations, and sets its flag (a word of its own: counted by atomics on one word per
// phase, the last of 16 to 43 items was seen 1.6 us after its stores).  Progress does not depend on which blocks run, or how many:
// items are handed out in order, an item waits for earlier ones only, and those are held by blocks that run.  If no block at
// all runs on that XCD, nothing is done, which the host sees by the count of completed launches.
// Two layers, d 256, 5 rows at 128 positions: 84.5 -> 65.8 us per call, 48 of them in the kernel: 12 phases of 2.3 to 6.3 us, each the hand-over
// (0.2 to 0.6) and an item's own work behind it (1.5 to 2.6: reading the activations, O merging attention's splits meanwhile, products, exchange in LDS,
// epilogue), that twice in gate/up and the LM head, which have more items than there are blocks.  Tried: two blocks per compute unit (the same; 128 registers, 15 in scratch
// memory), the next item drawn at this one's start (held while this one waits: 76 us).
#pragma once
#include "anpd_kernels.h"

namespace anpd {

struct GenLayer {
    const void *attn_norm, *wq, *wk, *wv, *wo, *ffn_norm, *w_gate, *w_up, *w_down;
};
constexpr int kSmallBlocks = 256;   // one per compute unit, if every XCD gets its eighth
constexpr int kSmallMerge = 4;      // splits of the keys up to which O's items merge attention's partial results themselves

struct SmallArgs {
    GenArgs gen;                // what all products share
    GenAttnArgs attn;
    AcceptArgs accept;
    const GenLayer *layers;
    const void *final_norm, *lm_head;
    float *x, *act, *logits;    // (q and att: attn)
    int d, ffn, vocab, M, splits;
    int out0, n_out;            // rows whose logits are wanted
    int tree, mode;
    uint32_t *ticket, *other;   // items handed out, 0 when the launch begins; the next launch's, which this one leaves at 0
    uint32_t *flags;            // [phase][stride]: `launch` when the item's results are there
    int stride;
    uint32_t launch;
    int xcd;
    int32_t *error;             // pinned host memory
    int32_t spin_limit;
    StepTokens tok;
};

__device__ __forceinline__ int this_xcd()
{
    uint32_t id;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID, 0, 4)" : "=s"(id));
    return (int)id;
}
// Where the blocks of such a grid run: count[0 .. 15] of every XCD.
__global__ __launch_bounds__(512) void xcd_census_kernel(uint32_t *__restrict__ count)
{
    if (threadIdx.x == 0) atomicAdd(count + this_xcd(), 1u);
}

typedef const SmallArgs __attribute__((address_space(4))) *SmallArgsK;   // the kernel's arguments where they lie

// (field by field: copied as a whole, the arguments would lie in scratch memory)
__device__ __forceinline__ GenArgs small_gemm(SmallArgsK g, const float *X, int K, int M, const void *W0, const void *W1, const void *W2, const void *gain, float *Y, int ldy,
                                              int layer)
{
    GenArgs a;
    a.X = X; a.M = M; a.K = K;
    a.W0 = W0; a.W1 = W1; a.W2 = W2; a.gain = gain;
    a.eps = g->gen.eps;
    a.Y = Y; a.ldy = ldy;
    a.rope = g->gen.rope; a.pool = g->gen.pool; a.page_table = g->gen.page_table; a.len_ptr = g->gen.len_ptr; a.depth = g->gen.depth;
    a.layer = layer; a.n_layers = g->gen.n_layers; a.n_heads = g->gen.n_heads; a.n_kv_heads = g->gen.n_kv_heads;
    a.head_dim = g->gen.head_dim; a.page_tokens = g->gen.page_tokens;
    a.embed = g->gen.embed; a.x = g->gen.x;
    return a;
}

template <int DH, int RT>
union SmallShared {
    GenShared<GEN_QKV, RT> pair;
    GenShared<GEN_RESIDUAL, RT> one;
    GenAttnShared<DH> attn;
    AcceptShared accept;
};

// What an item's block code calls: operator() when its weights are requested, publish() before the block meets for the last time.
template <typename W, typename P>
struct SmallWait {
    const W &w;
    const P &p;
    __device__ __forceinline__ void operator()() const { w(); }
    __device__ __forceinline__ void publish() const { p(); }
};

// RT: row tiles (windows of up to 16 rows, 32).
template <int DH, int RT>
__global__ __launch_bounds__(512, 2) void small_step_kernel(SmallArgs /* read where they lie */)
{
    const SmallArgsK g = (SmallArgsK)__builtin_amdgcn_kernarg_segment_ptr();
    if (this_xcd() != g->xcd) return;
    __shared__ SmallShared<DH, RT> sh;
    __shared__ int handed[2];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_layers = g->attn.n_layers, M = g->M, d = g->d, ffn = g->ffn;
    const int n_qkv = (g->gen.n_heads + 2 * g->gen.n_kv_heads) * (g->gen.head_dim / 32), n_att = g->gen.n_heads * g->splits * RT, n_d = d / 16, n_ffn = ffn / 16;
    const int per_layer = n_qkv + n_att + 2 * n_d + n_ffn, body = n_layers * per_layer, n_lm = g->vocab / 16, total = body + n_lm + g->n_out;
    const bool merged = g->splits <= kSmallMerge;
    auto draw = [&]() __attribute__((always_inline)) {   // (lane 0's)
        int t = 0;
        if (lane == 0) t = (int)__hip_atomic_fetch_add(g->ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return t;
    };
    if (wave == 7) {
        const int t = draw();
        if (lane == 0) handed[1] = t;
    }
    block_sync_lds();
    int item = __builtin_amdgcn_readfirstlane(handed[1]), turn = 0;
    if (item == 0 && threadIdx.x == 0) *g->other = 0u;   // (the launch that counted there is over)
    bool failed = false;
    while (item < total) {
        // ---- which item: the i-th of phase p of layer l (p = 5: LM head, 6: argmax), and how many items there were in the phase before
        int l = 0, p, i = item, before;
        if (item < body) {
            l = item / per_layer;
            i -= l * per_layer;
            if (i < n_qkv) { p = 0; before = l > 0 ? n_d : 0; }
            else if ((i -= n_qkv) < n_att) { p = 1; before = n_qkv; }
            else if ((i -= n_att) < n_d) { p = 2; before = n_att; }
            else if ((i -= n_d) < n_ffn) { p = 3; before = n_d; }
            else { i -= n_ffn; p = 4; before = n_ffn; }
        } else {
            l = n_layers;
            i -= body;
            p = i < n_lm ? 5 : 6;
            before = p == 5 ? n_d : n_lm;
            if (p == 6) i -= n_lm;
        }
        const int phase = p == 6 ? 5 * n_layers + 1 : 5 * l + (p == 5 ? 0 : p);
        if (p != 2) before *= RT;   // (a flag per row tile, attention's items are of one)
        const uint32_t launch = g->launch;
        int t = 0;
        auto wait_body = [&]() __attribute__((always_inline)) {
            if (wave == 7) {
                const uint32_t *f = g->flags + (size_t)(phase > 0 ? phase - 1 : 0) * g->stride;
                int spins = 0;
                for (int i0 = 0; i0 < before && !failed;) {
                    const uint32_t v = __builtin_amdgcn_raw_buffer_load_b32(wave_buffer(f), (i0 + lane) * 4, 0, kAuxNear);
                    asm volatile("" ::: "memory");
                    if (__builtin_amdgcn_ballot_w64(i0 + lane >= before || v == launch) == ~0ull) {
                        i0 += 64;
                        continue;
                    }
                    ++spins;
                    if ((spins & 4095) == 0 && ld_system(g->error) != 0) failed = true;
                    if (spins / 8 > g->spin_limit) {   // (a poll takes a tenth of a microsecond)
                        if (lane == 0) st_system(g->error, 1);
                        failed = true;
                    }
                }
            }
            block_sync_lds();
            if (wave == 7) t = draw();   // (drawn earlier it would be held, not worked on, while this item waits)
        };
        auto publish_body = [&]() __attribute__((always_inline)) {
            if (wave == 7 && lane == 0) handed[turn] = t;
        };
        SmallWait<decltype(wait_body), decltype(publish_body)> wait = {wait_body, publish_body};
        typedef const GenLayer __attribute__((address_space(4))) *GenLayerK;
        const GenLayerK w = (GenLayerK)g->layers + (l < n_layers ? l : 0);   // (not written while the kernel runs)
        auto done = [&](int n_flags, int flag) __attribute__((always_inline)) {   // waves 0 .. n_flags - 1 have finished the item
            if (flag >= n_flags) return;
            wait_stores();
            if (lane == 0) g->flags[(size_t)phase * g->stride + i * n_flags + flag] = launch;
        };
        if (p == 0) {
            const GenArgs a = small_gemm(g, g->x, d, M, w->wq, w->wk, w->wv, w->attn_norm, const_cast<float *>(g->attn.q), d, l);
            if (l == 0) gemm_gen_block<float, GEN_QKV, RT, FEW_NO, true, true>(a, (const int32_t *)g->tok.t, i, 0, sh.pair, wait);
            else gemm_gen_block<float, GEN_QKV, RT, FEW_NO, false, true>(a, nullptr, i, 0, sh.pair, wait);
            done(RT, wave);
        } else if (p == 1 || p == 2) {
            const GenAttnArgs at = {g->attn.q, g->attn.q_stride, g->attn.pool, g->attn.page_table, g->attn.len_ptr, M, l, n_layers, g->attn.n_heads,
                                    g->attn.n_kv_heads, g->attn.page_tokens, 0, g->attn.part_rows, g->attn.max_splits, DH, g->attn.scale, g->attn.part,
                                    g->attn.counter, g->attn.att, g->attn.row_mask};
            if (p == 1) {
                const int head = i % at.n_heads, rest = i / at.n_heads;
                attn_gen_block<float, DH, true>(at, head, rest % g->splits, rest / g->splits, sh.attn, wait, !merged);
                wait_stores();
                block_sync_lds();
                done(1, wave);
            } else {
                const GenArgs a = small_gemm(g, at.att, d, M, w->wo, nullptr, nullptr, nullptr, g->x, d, l);
                if (merged) gemm_gen_block<float, GEN_RESIDUAL, RT, FEW_NO, false, true, 1, kSmallMerge>(a, nullptr, i, 0, sh.one, wait, &at);
                else gemm_gen_block<float, GEN_RESIDUAL, RT, FEW_NO, false, true, 1>(a, nullptr, i, 0, sh.one, wait);
                done(RT, wave);
            }
        } else if (p == 4) {
            const GenArgs a = small_gemm(g, g->act, ffn, M, w->w_down, nullptr, nullptr, nullptr, g->x, d, l);
            gemm_gen_block<float, GEN_RESIDUAL, RT, FEW_NO, false, true, 3>(a, nullptr, i, 0, sh.one, wait);
            done(RT, wave);
        } else if (p == 3) {
            const GenArgs a = small_gemm(g, g->x, d, M, w->w_gate, w->w_up, nullptr, w->ffn_norm, g->act, ffn, l);
            gemm_gen_block<float, GEN_GATE_UP, RT, FEW_NO, false, true>(a, nullptr, i, 0, reinterpret_cast<GenShared<GEN_GATE_UP, RT> &>(sh), wait);
            done(RT, wave);
        } else if (p == 5) {
            const GenArgs a = small_gemm(g, g->x + (size_t)g->out0 * d, d, g->n_out, g->lm_head, nullptr, nullptr, g->final_norm, g->logits, g->vocab, 0);
            gemm_gen_block<float, GEN_LOGITS, RT, FEW_NO, false, true>(a, nullptr, i, 0, reinterpret_cast<GenShared<GEN_LOGITS, RT> &>(sh), wait);
            done(RT, wave);
        } else {
            wait();
            wait.publish();
            const AcceptArgs ac = {g->accept.result, g->accept.host_result, g->accept.len_ptr, g->accept.counter, g->accept.before, g->accept.parent, g->accept.depth,
                                   nullptr, 0, nullptr, g->accept.launches, g->accept.host_launches};
            const int32_t *tok = (const int32_t *)g->tok.t + g->out0;
            const bool rules = g->tree ? argmax_accept_block<ACCEPT_TREE, 512, true>(g->logits, g->vocab, g->n_out, tok, g->mode, ac, i, sh.accept)
                                       : argmax_accept_block<ACCEPT_CHAIN, 512, true>(g->logits, g->vocab, g->n_out, tok, g->mode, ac, i, sh.accept);
            if (rules && g->tree) {
                // the accepted path's keys and values to consecutive slots (kv_compact_kernel's rule)
                wait_stores();
                block_sync_lds();
                const int acc = ld_agent(ac.result), len = ld_agent(ac.len_ptr) - 1 - acc, hkv = g->attn.n_kv_heads, pt = g->attn.page_tokens;
                for (int j = 1; j <= acc; ++j) {
                    const int src = len + ld_agent(ac.result + 34 + j), dst = len + j;
                    if (src == dst) continue;
                    float *pool = (float *)g->gen.pool;
                    const int from = g->attn.page_table[src / pt], to = g->attn.page_table[dst / pt];
                    for (int e = threadIdx.x; e < n_layers * 2 * hkv * DH; e += 512) {
                        const int b = e / DH, head = b % hkv, kv = (b / hkv) & 1, layer = b / (2 * hkv);
                        pool[kv_offset(to, layer, n_layers, kv, head, hkv, dst % pt, pt, DH) + e % DH] =
                            ldc<true>(pool + kv_offset(from, layer, n_layers, kv, head, hkv, src % pt, pt, DH) + e % DH);
                    }
                }
            }
            if (rules && threadIdx.x == 0) {
                const uint32_t n = *ac.launches + 1u;
                *ac.launches = n;
                st_system(ac.host_launches, n);
            }
            block_sync_lds();   // (sh.accept)
        }
        item = __builtin_amdgcn_readfirstlane(handed[turn]);   // (the block has met since)
        turn ^= 1;
    }
}

}  // namespace anpd
