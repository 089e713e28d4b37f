// Device half of the C ABI: model / cache objects and the verification step.
//
// One step (paper, Section 3.1 "Parallel Decoding" step 2; Algorithm 1) is a
// fixed sequence of kernel launches on the caller's stream.  The window's
// tokens go to the kernels by value; cache length and page table, and the
// description of a draft tree or of a batch, are read from device memory (a
// kernel that takes them by value writes them there, unless the step is one
// kernel, which takes them by value itself).  The kernels write (accepted, next, predictions)
// into pinned host memory, and the logits where the caller wants them.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "anpd_common.h"
#include "anpd_kernels.h"
#include "anpd_fast.h"
#include "anpd_mega.h"
#include "anpd_prefill.h"
#include "anpd_small.h"

using namespace anpd;

#define HIP_TRY(expr)                                                                             \
    do {                                                                                          \
        hipError_t e_ = (expr);                                                                   \
        if (e_ != hipSuccess) return fail(ANPD_E_HIP, "%s: %s", #expr, hipGetErrorString(e_));    \
    } while (0)

namespace {

size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

int kv_heads_of(const anpd_model_cfg &c) { return c.n_kv_heads > 0 ? c.n_kv_heads : c.n_heads; }
int kv_dim_of(const anpd_model_cfg &c) { return kv_heads_of(c) * c.head_dim; }

// Work items of a phase beyond the first 32, which is what an XCD's compute units hold at a time, in rounds of 32.
int small_rounds(int items) { return (items + 31) / 32 - 1; }
// Whether a window of so many rows and splits of the keys goes through a model as one launch on one XCD (anpd_small.h): as long as a
// layer's phases take no round besides the five that they are (one more up to d 384, 320 beyond 16 rows, where a round is short) and the LM
// head no more than one per layer.
// us of a step with the truncation in front of it, separate launches -> one; 5 rows at 128 positions, 2 layers, vocabulary 1024 unless said:
// d 256, FFN 688 97 -> 82, at 450 (one extra round) 97 -> 86, 32 rows 120 -> 108, 8 layers 255 -> 197, with vocabulary 4608 (eight more for
// the LM head) 260 -> 220.  d 320, FFN 1024 (one) 103 -> 97, 32 rows 131 -> 128.  d 384, FFN 512 (one) 99 -> 93; 8 layers, vocabulary
// 4608, 16 / 17 / 32 rows at 8 positions 287 -> 275, 341 -> 342, 354 -> 365.  d 448, FFN 512, one key / value head (none) 100 -> 90, seven
// (one) 101 -> 99, 17 rows at 8 positions 121 -> 124.  d 512, FFN 512, two key / value heads (none) 100 -> 94, eight (one) 101 -> 104, 32 rows
// at 8 positions 125 -> 138.  Two rounds: d 256, 17 rows at 500 122 -> 130; more for the LM head: vocabulary 32000 117 -> 237.
bool small_step(const anpd_model_cfg &c, int rows, int splits)
{
    const int rt = rows > 16 ? 2 : 1;
    const int extra = small_rounds((c.n_heads + 2 * (c.n_kv_heads > 0 ? c.n_kv_heads : c.n_heads)) * (c.head_dim / 32)) + small_rounds(c.n_heads * splits * rt) +
                      2 * small_rounds(c.d_model / 16) + small_rounds(c.d_ffn / 16);
    return rows <= kMaxRows && splits <= 8 && extra <= (c.d_model <= (rt == 1 ? 384 : 320) ? 1 : 0) && small_rounds(c.vocab / 16) <= c.n_layers;
}
bool small_model(const anpd_model_cfg &c) { return c.dtype == ANPD_F32 && c.gemm_path == ANPD_GEMM_AUTO && small_step(c, 1, 1); }

constexpr int kSmallLine = 64;   // words
// most items of a phase that such a step may have
size_t small_items(const anpd_model_cfg &c)
{
    const size_t qkv = (size_t)(c.n_heads + 2 * kv_heads_of(c)) * (size_t)(c.head_dim / 32), lm = (size_t)c.vocab / 16, ffn = (size_t)c.d_ffn / 16;
    size_t most = 256;
    for (size_t n : {qkv, lm, ffn, (size_t)c.d_model / 16}) most = 2 * n > most ? 2 * n : most;
    return (most + 63) / 64 * 64;
}

struct Layout {  // byte offsets into the model workspace
    size_t rope_tab, tree, batch, result, counter, gen_ctr, x, qkv, att, a, logits, part;
    // fast path: packed operands, partial sums of squares, packed weights
    size_t xp_d, xp_att, xp_f, ssp_a, ssp_b, split_part, qp, head_ctr, layer_tab, amax, row_ctr, bar, wp_lm, total;
    size_t xp_layers, xp_stride;   // the one-kernel step's operands (bytes; stride between the layers' sets in bf16 elements: 0, one set)
    std::vector<size_t> wp_qkv, wp_o, wp_gu, wp_down;
    int max_splits;
    size_t small_ctr, small_layers;   // the one launch of a small model: two item counters, a word for completed launches, the items' flags; its layers' pointers
    int small_stride;   // flags per phase
    int gen_rows, gen_part_rows;   // generic path: most rows that go through a layer together, and of those through attention
};

// Models on the caller's weights take a prompt in pieces of up to this many rows (a step's kernels, more of their blocks).
constexpr int kGenPieceRows = 256;
constexpr size_t kGenPartBytes = (size_t)16 << 20;   // attention's partial results of a piece, where that is more than a window's

bool wants_mfma(const anpd_model_cfg *c)
{
    return c->gemm_path == ANPD_GEMM_MFMA || c->gemm_path == ANPD_GEMM_MFMA_LAUNCHES ||
           (c->gemm_path == ANPD_GEMM_AUTO && c->dtype == ANPD_BF16);
}

size_t packed_bytes(size_t n_tiles, int K) { return n_tiles * (size_t)((K + 31) / 32) * 1024; }

bool wants_mfma(const anpd_model_cfg *c);

bool cfg_ok(const anpd_model_cfg *c, const char **why)
{
#define REQ(cond, msg) if (!(cond)) { *why = msg; return false; }
    REQ(c, "cfg is NULL");
    REQ(c->n_layers >= 1 && c->d_model >= 8 && c->n_heads >= 1 && c->d_ffn >= 8 && c->vocab >= 1, "non-positive dimension");
    REQ(c->n_heads * c->head_dim == c->d_model, "d_model must equal n_heads * head_dim");
    REQ(c->n_kv_heads >= 0 && (c->n_kv_heads == 0 || c->n_heads % c->n_kv_heads == 0), "n_kv_heads must be 0 or divide n_heads");
    REQ(c->head_dim == 64 || c->head_dim == 128, "head_dim must be 64 or 128");
    REQ(c->d_model % 16 == 0 && c->d_ffn % 16 == 0 && c->vocab % 16 == 0, "d_model, d_ffn and vocab must be multiples of 16");
    REQ(c->dtype == ANPD_F32 || c->dtype == ANPD_BF16, "dtype must be ANPD_F32 or ANPD_BF16");
    REQ(c->page_tokens >= 8 && c->page_tokens <= 256 && (c->page_tokens & (c->page_tokens - 1)) == 0, "page_tokens must be a power of two in 8..256");
    REQ(c->max_window >= 1 && c->max_window <= ANPD_MAX_WINDOW, "max_window must be in 1..ANPD_MAX_WINDOW");
    REQ(c->max_positions >= 1 && c->max_positions <= (1 << 20), "max_positions must be in 1..2^20");
    REQ(c->gemm_path == ANPD_GEMM_AUTO || c->gemm_path == ANPD_GEMM_DOT || c->gemm_path == ANPD_GEMM_MFMA ||
            c->gemm_path == ANPD_GEMM_MFMA_LAUNCHES, "unknown gemm_path");
    REQ(!((c->gemm_path == ANPD_GEMM_MFMA || c->gemm_path == ANPD_GEMM_MFMA_LAUNCHES) && c->dtype != ANPD_BF16),
        "the MFMA path needs bf16 weights");
    REQ(c->rms_eps > 0.f && c->rope_base > 1.f, "rms_eps / rope_base out of range");
    REQ(!(wants_mfma(c) && c->page_tokens != 16), "the MFMA path needs page_tokens == 16");
#undef REQ
    return true;
}

Layout make_layout(const anpd_model_cfg *c)
{
    Layout L;
    const size_t MW = (size_t)c->max_window, d = (size_t)c->d_model, F = (size_t)c->d_ffn, V = (size_t)c->vocab;
    const size_t kvd = (size_t)kv_dim_of(*c);
    L.max_splits = (c->max_positions + kAttnSplit - 1) / kAttnSplit + 1;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes); return at; };
    L.rope_tab = take((size_t)c->max_positions * (c->head_dim / 2) * sizeof(float2));
    L.tree = take(3 * ANPD_MAX_WINDOW * sizeof(int32_t));                 // draft tree: parent, depth, visibility mask
    L.batch = take(ANPD_MAX_WINDOW * sizeof(int32_t) + ANPD_MAX_WINDOW * sizeof(SeqRef));   // batched step: sequence of every row, sequences
    // accepted, next, predictions, accepted path of a tree
    L.result = take((2 + ANPD_MAX_WINDOW + ANPD_MAX_WINDOW + 1) * sizeof(int32_t));
    L.counter = take(sizeof(uint32_t));
    // (the matrix-core path has a workspace of the caller's for prompts)
    L.gen_rows = L.gen_part_rows = (int)MW;
    const size_t part_row = (size_t)c->n_heads * L.max_splits * (c->head_dim + 2) * 4;
    if (!wants_mfma(c)) {
        const int longest = c->max_positions < kGenPieceRows ? c->max_positions : kGenPieceRows;
        if (longest > L.gen_rows) L.gen_rows = longest;
        const int rows = (int)(kGenPartBytes / part_row / 16 * 16);
        if (rows > L.gen_part_rows) L.gen_part_rows = rows < L.gen_rows ? rows : L.gen_rows;
        // (more than one launch of attention: each begins with a row group)
        if (L.gen_part_rows < L.gen_rows && L.gen_part_rows % 16 != 0) L.gen_rows = L.gen_part_rows;
    }
    const size_t GR = (size_t)L.gen_rows;
    L.gen_ctr = take((size_t)c->n_heads * ((L.gen_part_rows + 15) / 16) * 64 * sizeof(uint32_t));
    L.small_ctr = L.small_layers = 0;
    L.small_stride = 0;
    if (small_model(*c)) {
        // (counters: a line each)
        L.small_stride = (int)small_items(*c);
        L.small_ctr = take((3 * kSmallLine + (size_t)(5 * c->n_layers + 1) * L.small_stride) * sizeof(uint32_t));
        L.small_layers = take((size_t)c->n_layers * sizeof(GenLayer));
    }
    L.x = take(GR * d * 4);
    L.qkv = take(GR * d * 4);
    L.att = take(GR * d * 4);
    L.a = take(GR * F * 4);
    L.logits = take(MW * V * 4);
    L.part = take(part_row * (wants_mfma(c) ? 32 : L.gen_part_rows));
    L.xp_d = L.xp_att = L.xp_f = L.ssp_a = L.ssp_b = L.split_part = L.qp = L.head_ctr = L.wp_lm = 0;
    L.layer_tab = L.amax = L.row_ctr = L.bar = 0;
    L.xp_layers = L.xp_stride = 0;
    if (wants_mfma(c)) {
        L.xp_d = take(((d + 31) / 32) * 4 * 1024);
        L.xp_att = take(((d + 31) / 32) * 4 * 1024);
        L.xp_f = take(((F + 31) / 32) * 4 * 1024);
        // one set of the four operands for all layers (a set per layer, 48 MB at the 7B shape, cost 0.6 % of the
        // step at 640 cached positions and 1.6 % at 2048: lines that come round once per step are cold when
        // they are written)
        L.xp_stride = 0;
        L.xp_layers = take((3 * x_operand_elems((int)d) + x_operand_elems((int)F)) * sizeof(bf16_t));
        L.ssp_a = take((d / 16) * 32 * 4);
        L.ssp_b = take((d / 16) * 32 * 4);
        if (c->max_window > 16) L.split_part = take((d / 16) * 8 * 4 * 1024);   // partial tiles of the split O / down projections
        L.qp = take((size_t)c->n_heads * 4 * (c->head_dim / 32) * 1024);
        L.head_ctr = take((size_t)c->n_heads * ANPD_MAX_WINDOW * kCounterStride * sizeof(uint32_t));   // [group of rows or sequence][head]
        L.layer_tab = take((size_t)c->n_layers * sizeof(LayerW));
        L.amax = take((V / 16) * 32 * sizeof(unsigned long long));
        L.row_ctr = take(sizeof(uint32_t));
        L.bar = take(kBarStride * 9 * sizeof(uint32_t) + (size_t)c->n_heads * kCounterStride * sizeof(uint32_t));   // barrier words, then per-head QKV counters
        L.wp_lm = take(packed_bytes(V / 16, (int)d));
        for (int l = 0; l < c->n_layers; ++l) {
            L.wp_qkv.push_back(take(packed_bytes((d + 2 * kvd) / 16, (int)d)));
            L.wp_o.push_back(take(packed_bytes(d / 16, (int)d)));
            L.wp_gu.push_back(take(packed_bytes(F / 8, (int)d)));
            L.wp_down.push_back(take(packed_bytes(d / 16, (int)F)));
        }
    }
    L.total = o;
    return L;
}

struct PrefillLayout {  // byte offsets into the caller's prefill workspace
    size_t tok, x, part, xq, xq_att, xq_f, qp, total;
};

// Sized for the worst alignment of the first row inside its cache page.
PrefillLayout make_prefill_layout(const anpd_model_cfg &c, int n_tokens)
{
    PrefillLayout L;
    const size_t G = ((size_t)n_tokens + 30) / 16, d = (size_t)c.d_model, F = (size_t)c.d_ffn;
    const size_t nks_d = (d + 31) / 32, nks_f = (F + 31) / 32;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes); return at; };
    L.tok = take((size_t)n_tokens * sizeof(int32_t));
    L.x = take(G * 16 * d * sizeof(float));
    L.part = take((size_t)kPgSplit * G * 16 * d * sizeof(float));
    L.xq = take(G * nks_d * 2048);
    L.xq_att = take(G * nks_d * 2048);
    L.xq_f = take(G * nks_f * 2048);
    L.qp = take((size_t)c.n_heads * G * (size_t)(c.head_dim / 32) * 2048);
    L.total = o;
    return L;
}

}  // namespace

struct anpd_model {
    anpd_model_cfg cfg;
    Layout lay;
    char *ws;
    bool mfma;
    int n_cu, device;
    bool mega;            // the one-kernel step is available
    bool mega_tree;       // ... and so is its draft-tree form
    bool mega_batch;      // ... and its several-sequences form
    bool mega_rows16;     // ... and its form for windows of 9 to 16 rows
    int mega_kc;          // k-steps per wave per work item of the one-kernel step (8: d_model <= 4096, 10: <= 5120)
    long long *trace;     // optional device buffer for barrier timestamps
    int mega_grid;
    bool plain_launch;    // launch the one-kernel step without the cooperative-launch API (profiling aid)
    int32_t spin_limit;   // polls before a grid-barrier wait gives up
    uint32_t bar_epoch;
    int xcd;               // where the one launch of a small model runs (-1: it is not used)
    uint32_t small_launches, small_launch;   // those that have to be completed by now; number of the last one, which its flags are set to
    uint32_t ready_epoch;  // QKV phases run by the one-kernel step so far
    const void *embed, *final_norm, *lm_head;
    std::vector<const void *> attn_norm, wq, wk, wv, wo, ffn_norm, w_gate, w_up, w_down;
    int32_t *pin;  // pinned host staging: [0..32) window, [32..99) result and accepted path, [100] error flag of the
                   // persistent kernel, [128..224) draft tree (parent, depth, mask), [256..320) results of a batch,
                   // [384..416) sequence of every row of a batch, [512..768) its sequences (SeqRef)
    int32_t *pin_dev;  // the same memory as the device addresses it
    // optional per-kernel timing with events on the launch stream
    bool prof;
    std::vector<hipEvent_t> ev;
    std::vector<int> ev_cat;
    int ev_used;
    double prof_ms[ANPD_PROF_NCAT];
    int64_t prof_launches[ANPD_PROF_NCAT];
    int64_t prof_steps;
};

struct anpd_kv {
    const anpd_model *m;
    char *pool;
    int32_t n_pages, max_tokens, len;
    size_t page_bytes;
    std::vector<int32_t> table;      // logical -> physical, -1 = none
    std::vector<int32_t> dev_table;  // what the device copy currently holds
    std::vector<int32_t> free_list;  // physical pages, handed out from the back
    int32_t *d_table, *d_len;
    int32_t *pin;                    // pinned staging: [0] length, [1..] table
    bool table_dirty;
};

namespace {

size_t page_bytes_of(const anpd_model_cfg &c)
{
    return (size_t)c.n_layers * 2 * kv_dim_of(c) * c.page_tokens * (c.dtype == ANPD_BF16 ? 2 : 4);
}

// ---- GEMM dispatch -----------------------------------------------------------

// fp32 matrix cores on the caller's row-major weights; n_blocks: output features / 16, or pairs of 16.
template <typename WT, int MODE>
int32_t launch_gen(const GenArgs &a, int n_blocks, hipStream_t st)
{
    // more than 16 rows: two row tiles per block, so that the weights are read once
    if (a.M > 16) hipLaunchKernelGGL((gemm_gen_kernel<WT, MODE, 2>), dim3((unsigned)n_blocks, (unsigned)((a.M + 31) / 32)), dim3(512), 0, st, a);
    else hipLaunchKernelGGL((gemm_gen_kernel<WT, MODE, 1>), dim3((unsigned)n_blocks), dim3(512), 0, st, a);
    HIP_TRY(hipGetLastError());
    return ANPD_OK;
}

// The same for what pays with a few rows: anpd_linear, LM head, O and down.  bf16, a few rows and blocks enough: many blocks
// side by side beat many loads per wave, whose last round of blocks is nearly empty; up to two rows (48 KB: LDS for two
// or three blocks) are kept in LDS.  us, otherwise -> as chosen: 22016 x 4096, 1 / 2 / 3 / 4 rows 52.0 -> 42.4, 51.7 -> 44.2,
// 52.9 -> 48.8, 55.2 -> 52.8 (8 rows 61.2 -> 62.6: not chosen); 27648 x 5120 75.4 -> 58.3, 77.9 -> 64.2, 80.8 -> 75.9, 83.3 -> 80.7;
// 8192 x 4096, two blocks per compute unit, 1 row 18.9 -> 18.2 (4096 x 4096, one block: 11.7 either way); 16384 x 1024
// 13.2 -> 9.3; LM head of the 7B, 13B and ChatGLM3 shapes, 1 row 75 -> 66, 92 -> 80, 141 -> 121, 4 rows 80 -> 76, 101 -> 99, 152 -> 143
// (the gate / up pairs lose by it: 7B, 1 row, 53 -> 62).  O and down: rows in LDS where more than one block per compute
// unit reads them: 13B, 1 row, O 27.0 -> 25.4, down 54.9 -> 50.3 (7B, one block per compute unit, O 15.8 -> 16.8: not chosen).
template <typename WT, int MODE>
int32_t launch_gen_few(const GenArgs &a, int n_blocks, int n_cu, hipStream_t st)
{
    if constexpr (sizeof(WT) == 2) {
        constexpr bool res = MODE == GEN_RESIDUAL;
        const dim3 grid((unsigned)n_blocks), block(512);
        // (55 KB and the 8.5 KB in which the sums meet: within the 64 KB that need no attribute)
        if (a.M <= 2 && a.M * a.K <= (res ? 14080 : 12288) && (res ? n_blocks > n_cu : n_blocks >= 2 * n_cu)) {
            hipLaunchKernelGGL((gemm_gen_kernel<WT, MODE, 1, FEW_ROWS_LDS>), grid, block, (size_t)a.M * a.K * sizeof(float), st, a);
            HIP_TRY(hipGetLastError());
            return ANPD_OK;
        }
        if constexpr (!res) {
            if (a.M <= 4 && n_blocks >= 3 * n_cu) {
                hipLaunchKernelGGL((gemm_gen_kernel<WT, MODE, 1, FEW_ROWS>), grid, block, 0, st, a);
                HIP_TRY(hipGetLastError());
                return ANPD_OK;
            }
        }
    }
    return launch_gen<WT, MODE>(a, n_blocks, st);
}

// ---- fast path: packed MFMA GEMMs ---------------------------------------------

// A kernel of the fast path whose LDS may be more than the 64 KB that need no attribute (attr_set: per kernel)
template <typename K>
int32_t launch_lds(K kernel, bool &attr_set, int blocks, int threads, size_t lds, const FastArgs &a, hipStream_t st)
{
    if (lds > 65536 && !attr_set) {
        HIP_TRY(hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        attr_set = true;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3((unsigned)threads), lds, st, a);
    HIP_TRY(hipGetLastError());
    return ANPD_OK;
}
template <int T, int D, int EPI>
int32_t launch_wide(const FastArgs &a, int blocks, hipStream_t st)
{
    static bool attr_set = false;
    return launch_lds(gemm_wide_kernel<T, D, EPI>, attr_set, blocks, kFastThreads, (size_t)4 * kFastWaves * 4 * 256 * sizeof(float), a, st);
}
// waves: most tiles per block.  Up to four, the tiles are dealt evenly over all compute units: with blocks of as many tiles as go in,
// up to half of the compute units had none (257 tiles in 129 blocks).  From five on 9 in 10 have one all the same, the
// stream of weights is as fast, and fewer blocks read the operand.  9 / 17 rows, K 4096 / 11008, full blocks -> even, us:
// 257 tiles 13.2 -> 12.3 / 15.7 -> 15.2, 30.0 -> 28.2 / 36.3 -> 34.5; 700 18.1 -> 17.4 / 20.1 -> 20.0, 42.0 -> 40.4 / 49.6 -> 47.8;
// 960 24.3 -> 22.6 / 28.6 -> 24.9, 54.9 -> 54.9 / 61.5 -> 61.8; 1376 30.6 -> 31.7 / 33.2 -> 32.8, 77.1 -> 77.3 / 83.1 -> 81.7,
// and as gate/up of a 17-row step 35.4 -> 36.1.
template <int NT, int WAVES, int EPI>
int32_t launch_tile(const FastArgs &a, int waves, int n_cu, hipStream_t st)
{
    static bool attr_set = false;
    const int blocks = waves > 4 ? (a.n_tiles + waves - 1) / waves : (a.n_tiles < n_cu ? a.n_tiles : n_cu);
    return launch_lds(gemm_tile_kernel<NT, WAVES, EPI>, attr_set, blocks, (waves + 1) * 64, tile_lds_bytes(NT), a, st);
}

template <int EPI>
int32_t launch_fast(FastArgs &a, int n_cu, bool force_stream, hipStream_t st)
{
    const int kpw = (a.nks + kFastWaves - 1) / kFastWaves;
    if (a.cls == 8 && kpw <= 20 && !force_stream) {
        dim3 grid((unsigned)(a.n_tiles < n_cu ? a.n_tiles : n_cu)), block(kFastWaves * 64);
        if (kpw <= 2) hipLaunchKernelGGL((gemm_xs_kernel<2, EPI>), grid, block, 0, st, a);
        else if (kpw <= 4) hipLaunchKernelGGL((gemm_xs_kernel<4, EPI>), grid, block, 0, st, a);
        else if (kpw <= 8) hipLaunchKernelGGL((gemm_xs_kernel<8, EPI>), grid, block, 0, st, a);
        else if (kpw <= 16) hipLaunchKernelGGL((gemm_xs_kernel<16, EPI>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((gemm_xs_kernel<20, EPI>), grid, block, 0, st, a);
    } else if (a.cls == 8 || (a.cls == 16 && a.n_tiles <= n_cu)) {
        // one block per tile; several blocks share a compute unit.  Also the faster form for 9..16 rows when there is only
        // one tile per compute unit (4096 x 11008, 12 rows: 27.4 us, a tile per wave 31.2).
        dim3 grid((unsigned)a.n_tiles), block(kFastWaves * 64);
        const int nt = a.cls / 8;
        size_t smem = (size_t)kFastWaves * nt * 256 * sizeof(float);
        if (nt == 1) hipLaunchKernelGGL((gemm_stream_kernel<1, EPI>), grid, block, smem, st, a);
        else hipLaunchKernelGGL((gemm_stream_kernel<2, EPI>), grid, block, smem, st, a);
    } else {
        // windows of 9..32 rows: a tile per wave where one round of blocks takes them all; else (LM heads) blocks of a
        // contiguous range of tiles, in as few passes over the operand as the accumulators allow.
        // (17..32 rows, at most a tile per compute unit: eight waves of a block on it took, traced, 512 features of K 4096 /
        // 11008 / 13824 15.1 / 30.9 / 36.0 us; one wave with 16 k-steps in flight 13.6 / 30.1 / 37.6, with 32 13.0 / 28.6 / 35.9;
        // 4096 features 16.4 / 34.4 / 40.3, 14.7 / 33.2 / 40.9, 14.7 / 32.3 / 39.6.  K that does not fill the longer ring has
        // nothing of it: K = 256 5.5 -> 5.9, K = 1024 5.3 -> 5.2.)
        const int per_block = (a.n_tiles + n_cu - 1) / n_cu;
        if (per_block == 1 && a.cls == 32 && a.nks >= tile_depth(4, 1)) return launch_tile<4, 1, EPI>(a, 1, n_cu, st);
        if (per_block <= kTileWaves) return a.cls == 32 ? launch_tile<4, kTileWaves, EPI>(a, per_block, n_cu, st) : launch_tile<2, kTileWaves, EPI>(a, per_block, n_cu, st);
        if (a.cls == 16) {
            static bool attr_set = false;
            return launch_lds(gemm_group_kernel<2, 8, EPI>, attr_set, n_cu, kFastThreads, (size_t)8 * kFastWaves * 2 * 256 * sizeof(float), a, st);
        }
        const int passes = (per_block + 7) / 8, per_pass = (per_block + passes - 1) / passes;
        return per_pass <= 6 ? launch_wide<6, 3, EPI>(a, n_cu, st) : launch_wide<8, 2, EPI>(a, n_cu, st);
    }
    HIP_TRY(hipGetLastError());
    return ANPD_OK;
}

// O and down projections.  17..32 rows with at most two tiles per compute unit: split by k-step class (see
// gemm_split_kernel), 8 classes x n_cu / 8 groups of 8 to 16 tiles each.  Fewer tiles than one per compute unit
// (small models) stay with one launch, which is all they are.
int32_t launch_residual(FastArgs &a, int n_cu, float *part, hipStream_t st)
{
    const int groups = n_cu / 8, waves = groups > 0 ? (a.n_tiles + groups - 1) / groups : 0;
    if (a.cls != 32 || waves < kFastWaves || waves > kSplitMaxWaves) return launch_fast<EPI_RESIDUAL>(a, n_cu, false, st);
    static bool attr_set = false;
    if (!attr_set) {
        HIP_TRY(hipFuncSetAttribute((const void *)gemm_split_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSplitLds));
        attr_set = true;
    }
    hipLaunchKernelGGL(gemm_split_kernel, dim3((unsigned)((a.n_tiles + waves - 1) / waves * 8)), dim3((unsigned)(waves * 64)), kSplitLds, st, a, part);
    hipLaunchKernelGGL(split_merge_kernel, dim3((unsigned)a.n_tiles, (unsigned)((a.M + 15) / 16)), dim3(64), 0, st, a,
                       (const float *)part);
    HIP_TRY(hipGetLastError());
    return ANPD_OK;
}

// the operand of anpd_linear (window class cls)
void launch_split(const float *X, bf16_t *xp, int M, int K, int cls, hipStream_t st)
{
    const int nks = (K + 31) / 32;
    hipLaunchKernelGGL(split_packed_kernel, dim3((unsigned)((4 * nks + 255) / 256), (unsigned)cls), dim3(256), 0, st, X, xp, M, K, nks, cls);
}

int32_t launch_pack(const void *s0, const void *s1, const void *s2, void *dst, int mode, int n_tiles, int K, int d,
                    int head_dim, int kvd, hipStream_t st)
{
    const int nks = (K + 31) / 32;
    size_t total = (size_t)n_tiles * nks * 64;
    hipLaunchKernelGGL(pack_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, (const bf16_t *)s0,
                       (const bf16_t *)s1, (const bf16_t *)s2, (uint4 *)dst, mode, n_tiles, K, nks, d, head_dim, kvd);
    HIP_TRY(hipGetLastError());
    return ANPD_OK;
}

// ---- cache pages ---------------------------------------------------------------

// Make sure logical pages covering positions [0, upto) exist; refresh the device table if needed.
int32_t ensure_pages(anpd_kv *kv, int32_t upto, hipStream_t st)
{
    const int pt = kv->m->cfg.page_tokens;
    const int need = (upto + pt - 1) / pt;
    for (int lp = 0; lp < need; ++lp) {
        if (kv->table[(size_t)lp] >= 0) continue;
        if (kv->free_list.empty()) return fail(ANPD_E_CAPACITY, "KV pool has no free page");
        kv->table[(size_t)lp] = kv->free_list.back();
        kv->free_list.pop_back();
        if (kv->table[(size_t)lp] != kv->dev_table[(size_t)lp]) kv->table_dirty = true;
    }
    if (kv->table_dirty) {
        // the staging buffer is free: every call that uses it synchronises before returning
        for (size_t i = 0; i < kv->table.size(); ++i) {
            if (kv->table[i] >= 0) kv->dev_table[i] = kv->table[i];
            kv->pin[1 + i] = kv->dev_table[i] < 0 ? 0 : kv->dev_table[i];
        }
        HIP_TRY(hipMemcpyAsync(kv->d_table, kv->pin + 1, kv->table.size() * sizeof(int32_t), hipMemcpyHostToDevice, st));
        kv->table_dirty = false;
    }
    return ANPD_OK;
}

// Return pages wholly beyond `len` to the free list.
void release_pages(anpd_kv *kv, int32_t len)
{
    const int pt = kv->m->cfg.page_tokens;
    const int keep = (len + pt - 1) / pt;
    for (int lp = (int)kv->table.size() - 1; lp >= keep; --lp) {
        if (kv->table[(size_t)lp] >= 0) {
            kv->free_list.push_back(kv->table[(size_t)lp]);
            kv->table[(size_t)lp] = -1;
        }
    }
}

// Timing mark: an event after the launches of category `cat` (-1 = start of the step).
inline void mark(anpd_model *m, int cat, hipStream_t st)
{
    if (!m->prof) return;
    if (m->ev_used == (int)m->ev.size()) {
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) return;
        m->ev.push_back(e);
        m->ev_cat.push_back(cat);
    }
    m->ev_cat[(size_t)m->ev_used] = cat;
    (void)hipEventRecord(m->ev[(size_t)m->ev_used], st);
    m->ev_used += 1;
}

// After the stream has been synchronised: add the intervals between this call's marks to the sums.
void collect_marks(anpd_model *m)
{
    if (!m->prof) return;
    for (int i = 1; i < m->ev_used; ++i) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, m->ev[(size_t)i - 1], m->ev[(size_t)i]) == hipSuccess) {
            m->prof_ms[m->ev_cat[(size_t)i]] += (double)ms;
            m->prof_launches[m->ev_cat[(size_t)i]] += 1;
        }
    }
    m->prof_steps += 1;
}

StepTokens step_tokens(const int32_t *window, int n)
{
    StepTokens t;
    for (int i = 0; i < ANPD_MAX_WINDOW; ++i) t.t[i] = i < n ? window[i] : 0;
    return t;
}

// Where a step's LM head writes its n logits: straight into the caller's buffer when that is memory of this device that
// takes 16-byte stores and holds them all, else into the workspace, from where they are copied (a buffer of another
// GPU, say; one that is too short makes the copy fail, where stores would go past its end).
float *logits_target(const anpd_model *m, float *out_logits, size_t n)
{
    float *own = (float *)(m->ws + m->lay.logits);
    if (!out_logits || ((uintptr_t)out_logits & 15) != 0) return own;
    hipPointerAttribute_t at;
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipPointerGetAttributes(&at, out_logits) != hipSuccess || hipMemGetAddressRange(&base, &size, (hipDeviceptr_t)out_logits) != hipSuccess) {
        (void)hipGetLastError();
        return own;
    }
    const bool fits = (char *)out_logits + n * sizeof(float) <= (char *)base + size;
    return at.type == hipMemoryTypeDevice && at.device == m->device && fits ? out_logits : own;
}

// The caller's buffer for n logits (null: none), and where the LM head writes them: looked up when its launch is due, by when
// the device is at work on the launches in front of it (two queries of the runtime, some 2 us).
struct LogitsTo {
    float *out;
    size_t n;
    float *at;
    float *find(const anpd_model *m) { return at = logits_target(m, out, n); }
    bool elsewhere() const { return out && out != at; }
};

// What the last kernel of a step writes, and where.
AcceptArgs accept_args(anpd_model *m, int32_t *len_ptr)
{
    AcceptArgs a;
    std::memset(&a, 0, sizeof(a));
    a.result = (int32_t *)(m->ws + m->lay.result);
    a.host_result = m->pin_dev + 32;
    a.host_batch = m->pin_dev + 256;
    a.len_ptr = len_ptr;
    a.counter = (uint32_t *)(m->ws + m->lay.counter);
    return a;
}
void launch_accept(int kind, const float *logits, int V, int M, const StepTokens &tok, int mode, const AcceptArgs &a, hipStream_t st)
{
#define ANPD_ACCEPT(K_) hipLaunchKernelGGL((argmax_accept_kernel<K_>), dim3((unsigned)M), dim3(1024), 0, st, logits, V, M, tok, mode, a)
    if (kind == ACCEPT_TREE) ANPD_ACCEPT(ACCEPT_TREE);
    else if (kind == ACCEPT_BATCH) ANPD_ACCEPT(ACCEPT_BATCH);
    else ANPD_ACCEPT(ACCEPT_CHAIN);
#undef ANPD_ACCEPT
}

// The generic forward: per layer QKV (+ norm, RoPE, cache write) -> attention (+ merge) -> O (+ residual) -> gate/up
// (+ norm, SwiGLU) -> down (+ residual); then LM head (+ norm) -> argmax / accept.
// tree: the window is a draft tree whose parent / depth / mask arrays are in the workspace.
// piece: the rows are M tokens of a prompt (up to Layout::gen_rows), of which only the cache entries are wanted
// (PIECE_CACHE) or, besides them, logits and prediction of the last row (PIECE_LAST).
enum Piece { PIECE_NONE, PIECE_CACHE, PIECE_LAST };
template <typename KT>
int32_t run_step_generic(anpd_model *m, anpd_kv *kv, const int32_t *tokens, int M, int mode, LogitsTo &logits_to, hipStream_t st,
                         bool tree = false, Piece piece = PIECE_NONE)
{
    const anpd_model_cfg &c = m->cfg;
    const Layout &L = m->lay;
    char *ws = m->ws;
    const int d = c.d_model, F = c.d_ffn, V = c.vocab, H = c.n_heads, dh = c.head_dim;
    const int Hkv = kv_heads_of(c);
    float *x = (float *)(ws + L.x), *q = (float *)(ws + L.qkv), *att = (float *)(ws + L.att);
    float *act = (float *)(ws + L.a), *part = (float *)(ws + L.part);
    uint32_t *attn_ctr = (uint32_t *)(ws + L.gen_ctr);
    int32_t *result = (int32_t *)(ws + L.result);
    KT *pool = (KT *)kv->pool;
    const float scale = 1.0f / sqrtf((float)dh);
    const int32_t *t_parent = (const int32_t *)(ws + L.tree), *t_depth = tree ? t_parent + ANPD_MAX_WINDOW : nullptr;
    const uint32_t *t_mask = tree ? (const uint32_t *)(t_parent + 2 * ANPD_MAX_WINDOW) : nullptr;
    int32_t rc;

    GenArgs base;
    std::memset(&base, 0, sizeof(base));
    base.M = M;
    base.eps = c.rms_eps;
    base.rope = (const float2 *)(ws + L.rope_tab);
    base.pool = kv->pool;
    base.page_table = kv->d_table;
    base.len_ptr = kv->d_len;
    base.depth = t_depth;
    base.n_layers = c.n_layers;
    base.n_heads = H;
    base.n_kv_heads = Hkv;
    base.head_dim = dh;
    base.page_tokens = c.page_tokens;
    auto gemm = [&](const float *X, int K, const void *W, const void *gain, float *Y, int ldy) {
        GenArgs g = base;
        g.X = X;
        g.K = K;
        g.W0 = W;
        g.gain = gain;
        g.Y = Y;
        g.ldy = ldy;
        return g;
    };

    m->ev_used = 0;
    mark(m, -1, st);
    // (the tokens by value, as many per launch as its arguments take; a step's first QKV looks its rows up itself, in 16-byte loads that an
    // embedding table at an odd address does not get)
    const bool embed_in_qkv = piece == PIECE_NONE && ((uintptr_t)m->embed & 15) == 0;
    for (int i = 0; i < M && !embed_in_qkv; i += kMaxRows) {
        const int n = M - i < kMaxRows ? M - i : kMaxRows;
        hipLaunchKernelGGL((embed_kernel<KT>), dim3(n), dim3(256), 0, st, (const KT *)m->embed, step_tokens(tokens + i, n), x + (size_t)i * d, d);
    }
    mark(m, ANPD_PROF_OTHER, st);
    for (int l = 0; l < c.n_layers; ++l) {
        const bool last = piece != PIECE_NONE && l + 1 == c.n_layers;
        {
            GenArgs g = gemm(x, d, m->wq[l], m->attn_norm[l], q, d);
            g.W1 = m->wk[l];
            g.W2 = m->wv[l];
            g.layer = l;
            const int blocks = (H + 2 * Hkv) * (dh / 32);
            if (l == 0 && embed_in_qkv) {
                g.embed = m->embed;
                g.x = x;
                const StepTokens tok = step_tokens(tokens, M);
                if (M > 16) hipLaunchKernelGGL((gemm_gen_first_kernel<KT, 2>), dim3((unsigned)blocks), dim3(512), 0, st, g, tok);
                else hipLaunchKernelGGL((gemm_gen_first_kernel<KT, 1>), dim3((unsigned)blocks), dim3(512), 0, st, g, tok);
                HIP_TRY(hipGetLastError());
            } else if ((rc = launch_gen<KT, GEN_QKV>(g, blocks, st)) != ANPD_OK) {
                return rc;
            }
        }
        mark(m, ANPD_PROF_GEMM_QKV, st);
        // (a piece of a prompt: behind the last layer's keys and values only the row whose logits are wanted goes on, with its row group)
        if (last && piece == PIECE_CACHE) break;
        const int first = last ? (M - 1) / 16 * 16 : 0;
        base.M = M - first;
        for (int row0 = first; row0 < M; row0 += L.gen_part_rows) {
            const int end = M - row0 < L.gen_part_rows ? M : row0 + L.gen_part_rows;
            const dim3 grid((unsigned)H, (unsigned)((kv->len + end + kAttnSplit - 1) / kAttnSplit), (unsigned)((end - row0 + 15) / 16));
            const GenAttnArgs ga = {q, d, kv->pool, kv->d_table, kv->d_len, end, l, c.n_layers, H, Hkv, c.page_tokens, row0, L.gen_part_rows,
                                    L.max_splits, dh, scale, part, attn_ctr, att, t_mask};
#define ANPD_ATTN_G(DH_) hipLaunchKernelGGL((attn_kernel<KT, DH_>), grid, dim3(256), 0, st, ga)
            if (dh == 128) ANPD_ATTN_G(128);
            else ANPD_ATTN_G(64);
#undef ANPD_ATTN_G
        }
        mark(m, ANPD_PROF_ATTN, st);
        if ((rc = launch_gen_few<KT, GEN_RESIDUAL>(gemm(att + (size_t)first * d, d, m->wo[l], nullptr, x + (size_t)first * d, d), d / 16, m->n_cu, st)) != ANPD_OK) return rc;
        mark(m, ANPD_PROF_GEMM_O, st);
        {
            GenArgs g = gemm(x + (size_t)first * d, d, m->w_gate[l], m->ffn_norm[l], act + (size_t)first * F, F);
            g.W1 = m->w_up[l];
            if ((rc = launch_gen<KT, GEN_GATE_UP>(g, F / 16, st)) != ANPD_OK) return rc;
        }
        mark(m, ANPD_PROF_GEMM_GATE_UP, st);
        if ((rc = launch_gen_few<KT, GEN_RESIDUAL>(gemm(act + (size_t)first * F, F, m->w_down[l], nullptr, x + (size_t)first * d, d), d / 16, m->n_cu, st)) != ANPD_OK) return rc;
        mark(m, ANPD_PROF_GEMM_DOWN, st);
    }
    if (piece == PIECE_CACHE) {
        hipLaunchKernelGGL(advance_length_kernel, dim3(1), dim3(64), 0, st, kv->d_len, M);
        mark(m, ANPD_PROF_OTHER, st);
        HIP_TRY(hipGetLastError());
        return ANPD_OK;
    }
    const int before = piece == PIECE_LAST ? M - 1 : 0;   // rows in front of the first whose logits are wanted
    base.M = M - before;
    HIP_TRY(hipGetLastError());   // (of the launches so far: the lookup clears it)
    float *logits = logits_to.find(m);
    if ((rc = launch_gen_few<KT, GEN_LOGITS>(gemm(x + (size_t)before * d, d, m->lm_head, m->final_norm, logits, V), V / 16, m->n_cu, st)) != ANPD_OK) return rc;
    mark(m, ANPD_PROF_GEMM_LM_HEAD, st);
    AcceptArgs ac = accept_args(m, kv->d_len);
    ac.before = before;
    ac.parent = t_parent;
    ac.depth = t_depth;
    launch_accept(tree ? ACCEPT_TREE : ACCEPT_CHAIN, logits, V, M - before, step_tokens(tokens + before, M - before), mode, ac, st);
    if (tree)
        hipLaunchKernelGGL((kv_compact_kernel<KT>), dim3((unsigned)(c.n_layers * 2 * Hkv)), dim3(128), 0, st, pool, kv->d_table,
                           (const int32_t *)result, kv->len, c.n_layers, Hkv, dh, c.page_tokens);
    mark(m, ANPD_PROF_OTHER, st);
    HIP_TRY(hipGetLastError());
    return ANPD_OK;
}

// The same step or piece as one launch, if the model is small (anpd_small.h) and the call allows it; *ran says whether.
int32_t run_step_small(anpd_model *m, anpd_kv *kv, const int32_t *tokens, int M, int mode, LogitsTo &logits_to, hipStream_t st, bool tree, Piece piece,
                       bool *ran)
{
    const anpd_model_cfg &c = m->cfg;
    const Layout &L = m->lay;
    *ran = false;
    const int splits = (kv->len + M + kAttnSplit - 1) / kAttnSplit, rt = M > 16 ? 2 : 1;
    if (m->xcd < 0 || !small_step(c, M, splits) || M > L.gen_part_rows || piece == PIECE_CACHE || ((uintptr_t)m->embed & 15) != 0) return ANPD_OK;
    // (errors of launches in front, or left behind by someone else, are reported with nothing launched: the lookup of the logits' buffer
    // would clear them, and behind the launch they would be taken for its own)
    HIP_TRY(hipGetLastError());
    char *ws = m->ws;
    const int d = c.d_model, F = c.d_ffn, V = c.vocab, H = c.n_heads, Hkv = kv_heads_of(c);
    SmallArgs g;
    std::memset(&g, 0, sizeof(g));
    g.gen.eps = c.rms_eps;
    g.gen.rope = (const float2 *)(ws + L.rope_tab);
    g.gen.pool = kv->pool;
    g.gen.page_table = kv->d_table;
    g.gen.len_ptr = kv->d_len;
    int32_t *t_parent = (int32_t *)(ws + L.tree);
    g.gen.depth = tree ? t_parent + ANPD_MAX_WINDOW : nullptr;
    g.gen.n_layers = c.n_layers;
    g.gen.n_heads = H;
    g.gen.n_kv_heads = Hkv;
    g.gen.head_dim = c.head_dim;
    g.gen.page_tokens = c.page_tokens;
    g.gen.embed = m->embed;
    g.gen.x = g.x = (float *)(ws + L.x);
    g.attn = {(float *)(ws + L.qkv), d, kv->pool, kv->d_table, kv->d_len, M, 0, c.n_layers, H, Hkv, c.page_tokens, 0, L.gen_part_rows, L.max_splits,
              c.head_dim, 1.0f / sqrtf((float)c.head_dim), (float *)(ws + L.part), (uint32_t *)(ws + L.gen_ctr), (float *)(ws + L.att),
              tree ? (const uint32_t *)(t_parent + 2 * ANPD_MAX_WINDOW) : nullptr};
    g.act = (float *)(ws + L.a);
    g.logits = logits_to.find(m);
    g.layers = (const GenLayer *)(ws + L.small_layers);
    g.final_norm = m->final_norm;
    g.lm_head = m->lm_head;
    g.d = d;
    g.ffn = F;
    g.vocab = V;
    g.M = M;
    g.splits = splits;
    g.out0 = piece == PIECE_LAST ? M - 1 : 0;
    g.n_out = M - g.out0;
    g.tree = tree;
    g.mode = mode;
    uint32_t *words = (uint32_t *)(ws + L.small_ctr);
    const uint32_t launch = m->small_launch + 1 ? m->small_launch + 1 : 1;   // (never 0, which is what the flags begin with)
    g.ticket = words + (m->small_launches & 1) * kSmallLine;
    g.other = words + (1 - (m->small_launches & 1)) * kSmallLine;
    g.flags = words + 3 * kSmallLine;
    g.stride = L.small_stride;
    g.launch = launch;
    g.xcd = m->xcd;
    g.error = m->pin_dev + 100;
    g.spin_limit = m->spin_limit;
    g.accept = accept_args(m, kv->d_len);
    g.accept.before = g.out0;
    g.accept.parent = t_parent;
    g.accept.depth = t_parent + ANPD_MAX_WINDOW;
    g.accept.launches = words + 2 * kSmallLine;
    g.accept.host_launches = (uint32_t *)m->pin_dev + 102;
    g.tok = step_tokens(tokens, M);
    m->ev_used = 0;
    mark(m, -1, st);
    const void *kernel = c.head_dim == 128 ? (rt == 2 ? (const void *)small_step_kernel<128, 2> : (const void *)small_step_kernel<128, 1>)
                                           : (rt == 2 ? (const void *)small_step_kernel<64, 2> : (const void *)small_step_kernel<64, 1>);
    void *args[] = {&g};
    const hipError_t e = hipLaunchKernel(kernel, dim3(kSmallBlocks), dim3(512), args, 0, st);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(ANPD_E_HIP, "the one launch of a small model's step: %s", hipGetErrorString(e));
    }
    // (whatever is said later: it runs, and counts itself)
    m->small_launch = launch;
    m->small_launches += 1;
    mark(m, ANPD_PROF_STEP, st);
    *ran = true;
    return ANPD_OK;
}

// A step or a piece of a model on the caller's weights.
int32_t run_step_weights(anpd_model *m, anpd_kv *kv, const int32_t *tokens, int M, int mode, LogitsTo &logits, hipStream_t st, bool tree = false,
                         Piece piece = PIECE_NONE)
{
    if (m->cfg.dtype == ANPD_BF16) return run_step_generic<bf16_t>(m, kv, tokens, M, mode, logits, st, tree, piece);
    bool ran;
    const int32_t rc = run_step_small(m, kv, tokens, M, mode, logits, st, tree, piece, &ran);
    if (rc != ANPD_OK || ran) return rc;
    return run_step_generic<float>(m, kv, tokens, M, mode, logits, st, tree, piece);
}

// The fused bf16 step: per layer QKV(+norm, RoPE, cache write) -> attention -> combine -> O(+residual)
// -> gate/up(+norm, SwiGLU) -> down(+residual); then LM head(+norm) -> argmax / accept.
// A batched step: the sequences' descriptions are in the workspace (Layout::batch); `kv` is unused.
struct BatchLaunch {
    int n_seq, grid_splits /* splits of the longest sequence */;
    bool decode;   // one row per sequence and sequences enough: one block per (head, sequence)
    bool stream;   // keys and values are loaded as a stream
};
// Keys and values of a batch are loaded as a stream (non-temporal) where one block reads each and where they are more than the memory-side
// cache keeps until the next step (256 MB; the line is at 384).  us, ordinary loads -> stream, by what a step reads of them in all
// its layers: 7B shape, 8 layers, 8 sequences x 4 rows of 128 positions (159 MB) 975 -> 1001, 32 x 1 of 32 (159) 1033 -> 1052, of 64 (294) 1068 ->
// 1077, of 128 (562) 1132 -> 1125, of 500 (2122) 1420 -> 1384, of 1000 1835 -> 1753, 16 x 2 of 1000 (2122) 1472 -> 1423; 32 layers, 32 x 1 of 500
// 5582 -> 5359; two layers, 8 x 4 of 500 (137) 305 -> 312, 32 x 1 of 256 (275) 363 -> 364, of 500 (531) 413 -> 406; 13B shape, 8 layers, 16 x 1 of 128
// (351) 1391 -> 1393, 4 x 8 of 500 (359) 1387 -> 1387, 32 x 1 of 128 (703) 1520 -> 1511; d 2048, 8 x 4 of 500 (275) 595 -> 604; d 512, 32 x 1 of 500
// (265) 399 -> 404, of 1000 (527) 484 -> 465.
bool batch_streams(const anpd_model_cfg &c, long long positions)
{
    return kv_heads_of(c) == c.n_heads && positions * c.n_layers * kv_dim_of(c) * 4 > 384ll << 20;
}

int32_t run_step_fast(anpd_model *m, anpd_kv *kv, const StepTokens &tok, int M, int mode, LogitsTo &logits_to, hipStream_t st, bool tree = false,
                      const BatchLaunch *batch = nullptr)
{
    const anpd_model_cfg &c = m->cfg;
    const Layout &L = m->lay;
    char *ws = m->ws;
    const int d = c.d_model, F = c.d_ffn, V = c.vocab, H = c.n_heads, dh = c.head_dim;
    const int Hkv = kv_heads_of(c), kvd = kv_dim_of(c);
    const int cls = window_class(M);
    float *x = (float *)(ws + L.x), *part = (float *)(ws + L.part);
    bf16_t *qp = (bf16_t *)(ws + L.qp);
    uint32_t *head_ctr = (uint32_t *)(ws + L.head_ctr);
    bf16_t *xp_d = (bf16_t *)(ws + L.xp_d), *xp_att = (bf16_t *)(ws + L.xp_att), *xp_f = (bf16_t *)(ws + L.xp_f);
    float *ssp_a = (float *)(ws + L.ssp_a), *ssp_b = (float *)(ws + L.ssp_b), *split_part = (float *)(ws + L.split_part);
    int32_t *result = (int32_t *)(ws + L.result);
    const float scale = 1.0f / sqrtf((float)dh);
    const int n_splits = batch ? batch->grid_splits : n_splits_of(kv->len + M);
    const bool one_page = n_splits <= kSmallSplits;
    const int nks_d = (d + 31) / 32, nks_f = (F + 31) / 32;
    const int32_t *b_row_seq = (const int32_t *)(ws + L.batch);
    const SeqRef *b_seqs = (const SeqRef *)(ws + L.batch + ANPD_MAX_WINDOW * sizeof(int32_t));
    const int32_t *t_parent = (const int32_t *)(ws + L.tree), *t_depth = t_parent + ANPD_MAX_WINDOW;
    const uint32_t *t_mask = (const uint32_t *)(t_parent + 2 * ANPD_MAX_WINDOW);
    int32_t rc;

    FastArgs base;
    std::memset(&base, 0, sizeof(base));
    base.M = M;
    base.cls = cls;
    base.inv_d = 1.0f / (float)d;
    base.eps = c.rms_eps;
    base.n_ss = d / 16;
    base.d = d;
    base.x = x;
    if (!batch) {
        base.pool = (bf16_t *)kv->pool;
        base.page_table = kv->d_table;
        base.len_ptr = kv->d_len;
    }
    base.rope = (const float2 *)(ws + L.rope_tab);
    base.n_layers = c.n_layers;
    base.n_heads = H;
    base.n_kv_heads = Hkv;
    base.head_dim = dh;

    m->ev_used = 0;
    mark(m, -1, st);
    {
        FastArgs a = base;
        a.gain = (const bf16_t *)m->attn_norm[0];
        a.xp_next = xp_d;
        a.ssp_next = ssp_a;
        hipLaunchKernelGGL(embed_fast_kernel, dim3(d / 16), dim3(64), 0, st, (const bf16_t *)m->embed, tok, a);
    }
    mark(m, ANPD_PROF_OTHER, st);
    for (int l = 0; l < c.n_layers; ++l) {
        {
            FastArgs a = base;
            a.Wp = (const uint4 *)(ws + L.wp_qkv[(size_t)l]);
            a.Xp = (const uint4 *)xp_d;
            a.nks = nks_d;
            a.n_tiles = (d + 2 * kvd) / 16;
            a.ssp = ssp_a;
            a.qp = qp;
            a.layer = l;
            a.depth = t_depth;
            a.seqs = b_seqs;
            a.row_seq = b_row_seq;
            rc = batch ? launch_fast<EPI_QKV_BATCH>(a, m->n_cu, false, st)
                       : (tree ? launch_fast<EPI_QKV_TREE>(a, m->n_cu, false, st) : launch_fast<EPI_QKV>(a, m->n_cu, false, st));
            if (rc != ANPD_OK) return rc;
        }
        mark(m, ANPD_PROF_GEMM_QKV, st);
        // (n_splits <= kSmallSplits: every split of the step has one page per wave: the leaner instantiation)
        if (batch) {
#define ANPD_ATTN_B(DH_, MAXP_, STREAM_)                                                                                     \
    hipLaunchKernelGGL((attn_batch_kernel<DH_, MAXP_, STREAM_>), dim3(H, n_splits, batch->n_seq), dim3(kFastThreads), 0, st, \
                       (const uint4 *)qp, b_seqs, M, l, c.n_layers, H, Hkv, L.max_splits, scale, part, \
                       head_ctr, xp_att, cls)
#define ANPD_ATTN_O(DH_, MAXP_) do { if (batch->stream) ANPD_ATTN_B(DH_, MAXP_, true); else ANPD_ATTN_B(DH_, MAXP_, false); } while (0)
            if (batch->decode) {
#define ANPD_ATTN_D(DH_, STREAM_)                                                                                            \
    hipLaunchKernelGGL((attn_decode_kernel<DH_, STREAM_>), dim3(H, batch->n_seq), dim3(kFastThreads), 0, st, (const uint4 *)qp, b_seqs, l, c.n_layers, H, Hkv, \
                       scale, xp_att, cls)
                if (dh == 128) { if (batch->stream) ANPD_ATTN_D(128, true); else ANPD_ATTN_D(128, false); }
                else if (batch->stream) ANPD_ATTN_D(64, true);
                else ANPD_ATTN_D(64, false);
#undef ANPD_ATTN_D
            } else if (dh == 128) { if (one_page) ANPD_ATTN_O(128, 1); else ANPD_ATTN_O(128, kFastPages); }
            else if (one_page) ANPD_ATTN_O(64, 1);
            else ANPD_ATTN_O(64, kFastPages);
#undef ANPD_ATTN_O
#undef ANPD_ATTN_B
        } else {
#define ANPD_ATTN(DH_, TREE_, MAXP_)                                                                                       \
    hipLaunchKernelGGL((attn_fast_kernel<DH_, TREE_, MAXP_>), dim3(H, n_splits, (M + 7) / 8), dim3(kFastThreads), 0, st, (const uint4 *)qp,  \
                       (const bf16_t *)kv->pool, kv->d_table, kv->d_len, M, l, c.n_layers, H, Hkv, L.max_splits, scale, part,   \
                       head_ctr, xp_att, cls, t_mask)
#define ANPD_ATTN_T(DH_, MAXP_) do { if (tree) ANPD_ATTN(DH_, true, MAXP_); else ANPD_ATTN(DH_, false, MAXP_); } while (0)
            if (dh == 128) { if (one_page) ANPD_ATTN_T(128, 1); else ANPD_ATTN_T(128, kFastPages); }
            else if (one_page) ANPD_ATTN_T(64, 1);
            else ANPD_ATTN_T(64, kFastPages);
#undef ANPD_ATTN_T
#undef ANPD_ATTN
        }
        mark(m, ANPD_PROF_ATTN, st);
        {
            FastArgs a = base;
            a.Wp = (const uint4 *)(ws + L.wp_o[(size_t)l]);
            a.Xp = (const uint4 *)xp_att;
            a.nks = nks_d;
            a.n_tiles = d / 16;
            a.gain = (const bf16_t *)m->ffn_norm[l];
            a.xp_next = xp_d;
            a.ssp_next = ssp_b;
            if ((rc = launch_residual(a, m->n_cu, split_part, st)) != ANPD_OK) return rc;
        }
        mark(m, ANPD_PROF_GEMM_O, st);
        {
            FastArgs a = base;
            a.Wp = (const uint4 *)(ws + L.wp_gu[(size_t)l]);
            a.Xp = (const uint4 *)xp_d;
            a.nks = nks_d;
            a.n_tiles = F / 8;
            a.ssp = ssp_b;
            a.ap = xp_f;
            if ((rc = launch_fast<EPI_GATE_UP>(a, m->n_cu, false, st)) != ANPD_OK) return rc;
        }
        mark(m, ANPD_PROF_GEMM_GATE_UP, st);
        {
            FastArgs a = base;
            a.Wp = (const uint4 *)(ws + L.wp_down[(size_t)l]);
            a.Xp = (const uint4 *)xp_f;
            a.nks = nks_f;
            a.n_tiles = d / 16;
            a.gain = (const bf16_t *)(l + 1 < c.n_layers ? m->attn_norm[(size_t)l + 1] : m->final_norm);
            a.xp_next = xp_d;
            a.ssp_next = ssp_a;
            if ((rc = launch_residual(a, m->n_cu, split_part, st)) != ANPD_OK) return rc;
        }
        mark(m, ANPD_PROF_GEMM_DOWN, st);
    }
    HIP_TRY(hipGetLastError());   // (of the launches so far: the lookup clears it)
    float *logits = logits_to.find(m);
    {
        FastArgs a = base;
        a.Wp = (const uint4 *)(ws + L.wp_lm);
        a.Xp = (const uint4 *)xp_d;
        a.nks = nks_d;
        a.n_tiles = V / 16;
        a.ssp = ssp_a;
        a.Y = logits;
        a.ldy = V;
        if ((rc = launch_fast<EPI_LOGITS>(a, m->n_cu, false, st)) != ANPD_OK) return rc;
    }
    mark(m, ANPD_PROF_GEMM_LM_HEAD, st);
    AcceptArgs ac = accept_args(m, batch ? nullptr : kv->d_len);
    ac.parent = t_parent;
    ac.depth = t_depth;
    ac.seqs = b_seqs;
    ac.n_seq = batch ? batch->n_seq : 0;
    launch_accept(batch ? ACCEPT_BATCH : (tree ? ACCEPT_TREE : ACCEPT_CHAIN), logits, V, M, tok, mode, ac, st);
    if (tree)
        hipLaunchKernelGGL(kvf_compact_kernel, dim3((unsigned)(c.n_layers * 2 * Hkv)), dim3(128), 0, st, (bf16_t *)kv->pool,
                           kv->d_table, (const int32_t *)result, kv->len, c.n_layers, Hkv, dh);
    mark(m, ANPD_PROF_OTHER, st);
    HIP_TRY(hipGetLastError());
    return ANPD_OK;
}

// The step as one persistent kernel (window class 8).
// tree (nullable): the pinned draft-tree arrays parent[32], depth[32], mask[32] of a window of at most 8 rows.
// batch (nullable): several sequences side by side (kv is null then): seqs[n_seq], row_seq[M] and the lengths the host
// knows them to have.
struct MegaBatch {
    int n_seq;
    const SeqRef *seqs;
    const int32_t *row_seq;
    const int32_t *len;
};
// logits: where they go (null: nowhere).
int32_t run_step_mega(anpd_model *m, anpd_kv *kv, const int32_t *window, int M, int mode, float *logits, hipStream_t st,
                      const int32_t *tree = nullptr, const MegaBatch *batch = nullptr)
{
    const anpd_model_cfg &c = m->cfg;
    const Layout &L = m->lay;
    char *ws = m->ws;
    MegaArgs g;
    std::memset(&g, 0, sizeof(g));
    g.layers = (const LayerW *)(ws + L.layer_tab);
    g.n_layers = c.n_layers;
    g.wp_lm = (const uint4 *)(ws + L.wp_lm);
    g.final_gain = (const bf16_t *)m->final_norm;
    g.embed = (const bf16_t *)m->embed;
    g.d = c.d_model; g.F = c.d_ffn; g.V = c.vocab; g.n_heads = c.n_heads; g.n_kv_heads = kv_heads_of(c); g.head_dim = c.head_dim;
    g.M = M; g.mode = mode;
    g.inv_d = 1.0f / (float)c.d_model; g.eps = c.rms_eps; g.scale = 1.0f / sqrtf((float)c.head_dim);
    g.x = (float *)(ws + L.x);
    g.xp_layers = (bf16_t *)(ws + L.xp_layers);
    g.xp_stride = L.xp_stride;
    g.qp = (bf16_t *)(ws + L.qp);
    g.ssp_a = (float *)(ws + L.ssp_a); g.ssp_b = (float *)(ws + L.ssp_b); g.part = (float *)(ws + L.part);
    g.head_counter = (uint32_t *)(ws + L.head_ctr);
    if (kv) { g.pool = (bf16_t *)kv->pool; g.page_table = kv->d_table; g.len_ptr = kv->d_len; }
    g.rope = (const float2 *)(ws + L.rope_tab);
    g.max_splits = L.max_splits;
    g.logits = logits;
    g.amax = (unsigned long long *)(ws + L.amax);
    for (int i = 0; i < 16; ++i) g.tok[i] = i < M ? window[i] : 0;
    g.result = (int32_t *)(ws + L.result);
    g.host_result = m->pin_dev + 32;
    g.row_counter = (uint32_t *)(ws + L.row_ctr);
    g.bar = (uint32_t *)(ws + L.bar);
    g.bar_epoch = m->bar_epoch;
    g.error = m->pin_dev + 100;
    g.spin_limit = m->spin_limit;
    g.qkv_ready = (uint32_t *)(ws + L.bar) + kBarStride * 9;
    g.ready_epoch = m->ready_epoch;
    g.trace = m->trace;
    if (tree)
        for (int i = 0; i < 8; ++i) {
            g.parent[i] = tree[i];
            g.depth[i] = tree[ANPD_MAX_WINDOW + i];
            g.mask[i] = (uint32_t)tree[2 * ANPD_MAX_WINDOW + i];
        }
    if (batch) {
        g.n_seq = batch->n_seq;
        g.host_batch = m->pin_dev + 256;
        int tasks = 0;
        for (int s = 0; s < batch->n_seq; ++s) {
            g.seqs[s] = batch->seqs[s];
            g.task0[s] = tasks;
            const int splits = n_splits_of(batch->len[s] + batch->seqs[s].n_rows);
            tasks += splits * c.n_heads;
            g.n_att_blocks += splits;
        }
        g.task0[batch->n_seq] = tasks;
        for (int i = 0; i < M; ++i) g.row_seq[i] = batch->row_seq[i];
    }
    m->ev_used = 0;
    mark(m, -1, st);
    void *args[] = {&g};
    const int form = batch ? MEGA_BATCH : (tree ? MEGA_TREE : MEGA_CHAIN);
    const void *fn128[] = {(const void *)verify_mega_kernel<128, MEGA_CHAIN>, (const void *)verify_mega_kernel<128, MEGA_TREE>,
                           (const void *)verify_mega_kernel<128, MEGA_BATCH>};
    const void *fn64[] = {(const void *)verify_mega_kernel<64, MEGA_CHAIN>, (const void *)verify_mega_kernel<64, MEGA_TREE>,
                          (const void *)verify_mega_kernel<64, MEGA_BATCH>};
    const void *fn = c.head_dim == 128 ? fn128[form] : fn64[form];
    if (M > 8)   // windows of 9 to 16 rows (chains only; the caller has checked mega_rows16)
        fn = c.head_dim == 128 ? (const void *)verify_mega_kernel<128, MEGA_CHAIN, 2> : (const void *)verify_mega_kernel<64, MEGA_CHAIN, 2>;
    else if (m->mega_kc == 10)   // d_model above 4096 (chains only)
        fn = c.head_dim == 128 ? (const void *)verify_mega_kernel<128, MEGA_CHAIN, 1, 10> : (const void *)verify_mega_kernel<64, MEGA_CHAIN, 1, 10>;
    if (m->plain_launch) {
        // profiling aid (see anpd_model_create): an ordinary launch of the same grid
        HIP_TRY(hipLaunchKernel(fn, dim3((unsigned)m->mega_grid), dim3(kFastThreads), args, 0, st));
    } else {
        HIP_TRY(hipLaunchCooperativeKernel(fn, dim3((unsigned)m->mega_grid), dim3(kFastThreads), args, 0, st));
    }
    m->bar_epoch += (uint32_t)kMegaBarriers(c.n_layers);
    m->ready_epoch += (uint32_t)c.n_layers;
    if (tree) {
        // the winning path's K and V to consecutive positions (a no-op kernel when it is the first candidate)
        hipLaunchKernelGGL(kvf_compact_kernel, dim3((unsigned)(c.n_layers * 2 * kv_heads_of(c))), dim3(128), 0, st, (bf16_t *)kv->pool,
                           kv->d_table, (const int32_t *)(ws + L.result), kv->len, c.n_layers, kv_heads_of(c), c.head_dim);
        HIP_TRY(hipGetLastError());
    }
    mark(m, ANPD_PROF_STEP, st);
    return ANPD_OK;
}

// ---- prompt processing on the matrix cores ------------------------------------

// One of the prompt GEMMs: sets the kernel's LDS size once (attr_set: per kernel), then launches it.
template <typename K, typename... Args>
int32_t launch_prefill_kernel(K kernel, bool &attr_set, long long blocks, int threads, size_t lds, hipStream_t st, const Args &...args)
{
    if (!attr_set) {
        HIP_TRY(hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        attr_set = true;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3((unsigned)threads), lds, st, args...);
    HIP_TRY(hipGetLastError());
    return ANPD_OK;
}
// (blocks: of the template's width; see launch_prefill_gemm)
template <int EPI, int TN>
int32_t launch_prefill_wide(const PrefillArgs &a, long long blocks, hipStream_t st)
{
    static bool attr_set = false;
    return launch_prefill_kernel(prefill_gemm_kernel<EPI, TN>, attr_set, blocks, kPgThreads, pg_lds_bytes(TN, 4), st, a);
}
template <int EPI, int TN>
int32_t launch_prefill_narrow(const PrefillArgs &a, long long blocks, hipStream_t st)
{
    static bool attr_set = false;
    return launch_prefill_kernel(prefill_narrow_kernel<EPI, TN>, attr_set, blocks, 256, pg_lds_bytes(TN, 2), st, a);
}
template <int EPI, int TB>
int32_t launch_prefill_mixed(const PrefillArgs &a, int n_a, int tiles_a, long long blocks, hipStream_t st)
{
    static bool attr_set = false;
    return launch_prefill_kernel(prefill_mixed_kernel<EPI, 6, TB>, attr_set, blocks, kPgThreads, pg_lds_bytes(6, 4), st, a, n_a, tiles_a);
}
template <int EPI, int TG, bool ONCE>
int32_t launch_prefill_few(const PrefillArgs &a, int waves, long long blocks, hipStream_t st)
{
    static bool attr_set = false;
    return launch_prefill_kernel(prefill_few_kernel<EPI, TG, ONCE>, attr_set, blocks, (waves + kFewLoaders) * 64, few_lds_bytes(TG), st, a);
}

// Measured time of a block of 64 TN features x 128 rows with the chip full of them, us at K = 4096.
constexpr double kPgBlock[7] = {0, 0, 64, 80, 96, 115, 141};

// When the last of n_a blocks of time ta each and, behind them, n_b of time tb each ends, handed out to n_cu compute
// units as these become free.
double blocks_end(long long n_a, double ta, long long n_b, double tb, int n_cu)
{
    const long long later = n_a % n_cu, sooner = n_cu - later;   // compute units that end the first kind in the last round, and before it
    const double t0 = (double)(n_a / n_cu) * ta, t1 = t0 + ta;
    double end = later ? t1 : t0;
    for (long long k0 = 0, k1 = 0; n_b > 0;) {   // the next group of compute units that is free takes one each
        if (t0 + (double)k0 * tb <= t1 + (double)k1 * tb || later == 0) {
            n_b -= sooner;
            end = std::fmax(end, t0 + (double)++k0 * tb);
        } else {
            n_b -= later;
            end = std::fmax(end, t1 + (double)++k1 * tb);
        }
    }
    return end;
}

// How the product is cut into blocks; an element's sums are the same in every form (each ends with the figures of the
// 7B shape, us).
template <int EPI>
int32_t launch_prefill_gemm(const PrefillArgs &a, int n_cu, hipStream_t st)
{
    const int n_tiles = a.n_tiles - a.tile0, G = a.G - a.g0;
    auto cols = [&](int tiles) { return (long long)((n_tiles + tiles - 1) / tiles) * a.S; };
    // A few row groups: a tile per wave and as many waves per block as one round of blocks takes, if there is one:
    // 64 TN features x 128 rows -> this, QKV of 16 / 32 / 64 / 128 rows 45 -> 17, 45 -> 19, 46 -> 20, 46 -> 27; gate/up
    // of 16 / 32 / 64 rows 48 -> 27, 48 -> 28, 49 -> 31; down 33 -> 16, 33 -> 17, 34 -> 19.  (In two rounds it loses what
    // it gains: gate/up of 128 rows 50 -> 50, down 35 -> 32 against 28 for the narrow form.)
    const int tg = G == 1 ? 1 : 2, n_br2 = (G + tg - 1) / tg;
    for (int waves = 3; waves <= kFewWaves; ++waves) {
        const long long blocks = cols(waves) * n_br2;
        if (blocks > n_cu) continue;
        if (tg == 1) return launch_prefill_few<EPI, 1, true>(a, waves, blocks, st);
        return n_br2 == 1 ? launch_prefill_few<EPI, 2, true>(a, waves, blocks, st) : launch_prefill_few<EPI, 2, false>(a, waves, blocks, st);
    }
    // Up to 128 rows: half as wide, of four waves, where that is at most one block per compute unit: gate/up 50 -> 47,
    // down 35 -> 28 (they read half as much again per MFMA, which more rows would feel: two per compute unit, gate/up
    // of 512 rows 136 -> 153).
    if (G <= 8 && cols(4) <= n_cu) return launch_prefill_narrow<EPI, 2>(a, cols(4), st);
    if (G <= 8 && cols(6) <= n_cu) return launch_prefill_narrow<EPI, 3>(a, cols(6), st);
    // Blocks of 64 TN features: wider ones read less per MFMA, narrower ones leave fewer compute units idle in the
    // last round (512 rows: 6 for gate/up, 3 for QKV, 4 for O and down).  Where the widest take some rounds and a
    // piece of one, the piece in narrower blocks: gate/up of 768 / 1800 / 3584 rows 218 -> 205, 518 -> 481, 964 -> 921,
    // QKV of 3584 538 -> 511, down of 1800 278 -> 259.
    const int n_br = (G + 7) / 8;
    int best = 0, best_b = 0, best_cols = 0;
    double least = 0;
    for (int tn = 6; tn >= 2; --tn) {
        const double t = blocks_end(cols(4 * tn) * n_br, kPgBlock[tn], 0, 0, n_cu);
        if (best == 0 || t < least) { least = t; best = tn; }
    }
    const long long rounds = cols(24) * n_br / n_cu;
    for (long long r = rounds; r >= 1 && r >= rounds - 1; --r) {
        const int wide = (int)(r * n_cu / ((long long)n_br * a.S));   // columns of the widest blocks
        if (wide < 1 || wide * 24 >= n_tiles) continue;
        for (int tb = 4; tb >= 3; --tb) {
            const long long n_b = (long long)((n_tiles - wide * 24 + 4 * tb - 1) / (4 * tb)) * a.S * n_br;
            const double t = blocks_end((long long)wide * a.S * n_br, kPgBlock[6], n_b, kPgBlock[tb], n_cu);
            if (t < 0.98 * least) { least = t; best_b = tb; best_cols = wide; }
        }
    }
    if (best_b) {
        const int n_a = best_cols * a.S * n_br, tiles_a = best_cols * 24;
        const long long blocks = n_a + (long long)((n_tiles - tiles_a + 4 * best_b - 1) / (4 * best_b)) * a.S * n_br;
        return best_b == 4 ? launch_prefill_mixed<EPI, 4>(a, n_a, a.tile0 + tiles_a, blocks, st) : launch_prefill_mixed<EPI, 3>(a, n_a, a.tile0 + tiles_a, blocks, st);
    }
    const long long blocks = cols(4 * best) * n_br;
    switch (best) {
    case 2: return launch_prefill_wide<EPI, 2>(a, blocks, st);
    case 3: return launch_prefill_wide<EPI, 3>(a, blocks, st);
    case 4: return launch_prefill_wide<EPI, 4>(a, blocks, st);
    case 5: return launch_prefill_wide<EPI, 5>(a, blocks, st);
    default: return launch_prefill_wide<EPI, 6>(a, blocks, st);
    }
}

// All P rows at once; per layer norm -> QKV(+RoPE, cache write) -> attention -> O(+residual) -> norm ->
// gate/up(+SwiGLU) -> down(+residual); the last row then goes through the step's LM head and argmax.
int32_t run_prefill_mfma(anpd_model *m, anpd_kv *kv, int P, char *pws, const PrefillLayout &PL, LogitsTo &logits_to, hipStream_t st)
{
    const anpd_model_cfg &c = m->cfg;
    const Layout &L = m->lay;
    char *ws = m->ws;
    const int d = c.d_model, F = c.d_ffn, V = c.vocab, H = c.n_heads, dh = c.head_dim;
    const int len = kv->len, r0 = len & 15;
    const int G = (r0 + P + 15) / 16;
    const int nks_d = (d + 31) / 32, nks_f = (F + 31) / 32;
    const int32_t *tok = (const int32_t *)(pws + PL.tok);
    float *x = (float *)(pws + PL.x), *part = (float *)(pws + PL.part);
    bf16_t *xq = (bf16_t *)(pws + PL.xq), *xq_att = (bf16_t *)(pws + PL.xq_att), *xq_f = (bf16_t *)(pws + PL.xq_f);
    bf16_t *qp = (bf16_t *)(pws + PL.qp);
    const float inv_d = 1.0f / (float)d, scale = 1.0f / sqrtf((float)dh);
    int32_t rc;

    PrefillArgs base;
    std::memset(&base, 0, sizeof(base));
    base.G = G;
    base.L = len;
    base.P = P;
    base.S = 1;
    base.part = part;
    base.d = d;
    base.qp = qp;
    base.pool = (bf16_t *)kv->pool;
    base.page_table = kv->d_table;
    base.rope = (const float2 *)(ws + L.rope_tab);
    base.n_layers = c.n_layers;
    base.n_heads = H;
    base.n_kv_heads = kv_heads_of(c);
    base.head_dim = dh;

    m->ev_used = 0;
    mark(m, -1, st);
    // columns F .. 32 * nks_f of the down projection's operand meet zero weights: they must not hold NaN patterns
    if (F % 32 != 0) HIP_TRY(hipMemsetAsync(xq_f, 0, (size_t)G * nks_f * 2048, st));
    auto norm = [&](const bf16_t *gain, bool embed, int g0) {
#define ANPD_NORM(EMBED_, NV_)                                                                                              \
    hipLaunchKernelGGL((prefill_norm_kernel<EMBED_, NV_>), dim3((unsigned)((G - g0 + 7) / 8 * 128)), dim3(256), 0, st, (const bf16_t *)m->embed, tok, x, \
                       (const float *)part, gain, xq, nks_d, d, g0, G, len, P, inv_d, c.rms_eps)
        if (d <= 4096) { if (embed) ANPD_NORM(true, 4); else ANPD_NORM(false, 4); }
        else if (embed) ANPD_NORM(true, 8);
        else ANPD_NORM(false, 8);
#undef ANPD_NORM
    };
    norm((const bf16_t *)m->attn_norm[0], true, 0);
    mark(m, ANPD_PROF_OTHER, st);
    for (int l = 0; l < c.n_layers; ++l) {
        // Behind the last layer's keys and values only the last row is wanted, so everything from its queries on works on that row's
        // group alone (4 layers, 205 / 512 / 3584 rows 1116 -> 1028 us (ChatGLM3 shape), 1546 -> 1369, 10641 -> 8811; a layer's GEMMs
        // and attention are then 0.11 ms whatever the rows: of 32 layers it saves the better part of one).
        const int g0 = l + 1 == c.n_layers ? G - 1 : 0;
        {
            PrefillArgs a = base;
            a.Wp = (const uint4 *)(ws + L.wp_qkv[(size_t)l]);
            a.Xq = (const uint4 *)xq;
            a.nks = nks_d;
            a.n_tiles = (d + 2 * kv_dim_of(c)) / 16;
            a.layer = l;
            // ... its queries as a launch of their own from 257 rows on, where that is less than the other rows' queries: 256 / 384 / 512
            // / 1800 rows, one layer, in one launch -> two, 7B shape 250 -> 260, 277 -> 271, 295 -> 291, 572 -> 505 us; 13B 302 -> 313,
            // 333 -> 326, 367 -> 357, 764 -> 639; ChatGLM3 269 -> 272, 286 -> 281, 316 -> 294, 465 -> 389.
            if (g0 >= 16) {
                PrefillArgs q = a;
                q.n_tiles = a.tile0 = d / 16;
                q.g0 = g0;
                if ((rc = launch_prefill_gemm<EPI_QKV>(q, m->n_cu, st)) != ANPD_OK) return rc;
            }
            if ((rc = launch_prefill_gemm<EPI_QKV>(a, m->n_cu, st)) != ANPD_OK) return rc;
        }
        mark(m, ANPD_PROF_GEMM_QKV, st);
        {
            const dim3 grid((unsigned)H, (unsigned)((G - g0 + 1) / 2));
            // query rows in LDS where that brings one more block to a compute unit, else in registers (see the kernel)
            const bool shared = (long long)grid.x * grid.y > (dh == 128 ? 1 : 2) * m->n_cu;
#define ANPD_ATTN_P(DH_, Q_)                                                                                                      \
    hipLaunchKernelGGL((prefill_attn_kernel<DH_, Q_>), grid, dim3(256), 0, st, (const uint4 *)qp, (const bf16_t *)kv->pool, kv->d_table, g0, G, \
                       len, P, l, c.n_layers, H, kv_heads_of(c), scale, xq_att, nks_d)
            if (dh == 128) { if (shared) ANPD_ATTN_P(128, true); else ANPD_ATTN_P(128, false); }
            else if (shared) ANPD_ATTN_P(64, true);
            else ANPD_ATTN_P(64, false);
#undef ANPD_ATTN_P
        }
        mark(m, ANPD_PROF_ATTN, st);
        {
            PrefillArgs a = base;
            a.Wp = (const uint4 *)(ws + L.wp_o[(size_t)l]);
            a.Xq = (const uint4 *)xq_att;
            a.nks = nks_d;
            a.n_tiles = d / 16;
            a.g0 = g0;
            a.S = kPgSplit;
            if ((rc = launch_prefill_gemm<EPI_RESIDUAL>(a, m->n_cu, st)) != ANPD_OK) return rc;
        }
        mark(m, ANPD_PROF_GEMM_O, st);
        norm((const bf16_t *)m->ffn_norm[l], false, g0);
        mark(m, ANPD_PROF_OTHER, st);
        {
            PrefillArgs a = base;
            a.Wp = (const uint4 *)(ws + L.wp_gu[(size_t)l]);
            a.Xq = (const uint4 *)xq;
            a.nks = nks_d;
            a.n_tiles = F / 8;
            a.g0 = g0;
            a.out = xq_f;
            a.out_nks = nks_f;
            if ((rc = launch_prefill_gemm<EPI_GATE_UP>(a, m->n_cu, st)) != ANPD_OK) return rc;
        }
        mark(m, ANPD_PROF_GEMM_GATE_UP, st);
        {
            PrefillArgs a = base;
            a.Wp = (const uint4 *)(ws + L.wp_down[(size_t)l]);
            a.Xq = (const uint4 *)xq_f;
            a.nks = nks_f;
            a.n_tiles = d / 16;
            a.g0 = g0;
            a.S = kPgSplit;
            if ((rc = launch_prefill_gemm<EPI_RESIDUAL>(a, m->n_cu, st)) != ANPD_OK) return rc;
        }
        mark(m, ANPD_PROF_GEMM_DOWN, st);
        if (l + 1 < c.n_layers) {
            norm((const bf16_t *)m->attn_norm[(size_t)l + 1], false, 0);
            mark(m, ANPD_PROF_OTHER, st);
        }
    }
    // last row -> the step's LM head, argmax and length update (one appended row)
    hipLaunchKernelGGL(prefill_last_kernel, dim3((unsigned)(d / 16)), dim3(64), 0, st, x + (size_t)(r0 + P - 1) * d,
                       (const float *)(part + (size_t)(r0 + P - 1) * d), kPgSplit, (size_t)G * 16 * d, (const bf16_t *)m->final_norm, (bf16_t *)(ws + L.xp_d), (float *)(ws + L.ssp_a), kv->d_len, len + P - 1);
    mark(m, ANPD_PROF_OTHER, st);
    HIP_TRY(hipGetLastError());   // (of the launches so far: the lookup clears it)
    float *logits = logits_to.find(m);
    {
        FastArgs a;
        std::memset(&a, 0, sizeof(a));
        a.M = 1;
        a.cls = 8;
        a.inv_d = inv_d;
        a.eps = c.rms_eps;
        a.n_ss = d / 16;
        a.d = d;
        a.Wp = (const uint4 *)(ws + L.wp_lm);
        a.Xp = (const uint4 *)(ws + L.xp_d);
        a.nks = nks_d;
        a.n_tiles = V / 16;
        a.ssp = (const float *)(ws + L.ssp_a);
        a.Y = logits;
        a.ldy = V;
        if ((rc = launch_fast<EPI_LOGITS>(a, m->n_cu, false, st)) != ANPD_OK) return rc;
    }
    mark(m, ANPD_PROF_GEMM_LM_HEAD, st);
    launch_accept(ACCEPT_CHAIN, logits, V, 1, StepTokens(), (int)ANPD_APPEND, accept_args(m, kv->d_len), st);
    mark(m, ANPD_PROF_OTHER, st);
    HIP_TRY(hipGetLastError());
    return ANPD_OK;
}

// Left to itself (AUTO) a model below d 2048 takes separate launches: what the one kernel hides in longer phases, the first weights of
// the next one, is not worth its barriers there.  us, one kernel -> launches, 8 layers, 1 row at 512 / 2048 / 4000 positions: d 1024 357 -> 303,
// 388 -> 334, 391 -> 337; d 1536 385 -> 343, 417 -> 379, 421 -> 389; d 1920 414 -> 385, 445 -> 425, 452 -> 436 (8 rows within 1 % of that;
// tree of 7 rows / 2 sequences x 4 rows at 512: d 1024 367 -> 310 / 388 -> 334, d 1920 429 -> 410 / 454 -> 439).  d 256, 2 layers, 1 / 8 rows at
// 200 120 -> 86, 123 -> 87.  Further up the two forms are close, and such models keep the one kernel, though it is the slower form up to
// d 2304: d 2048 421 -> 405, 457 -> 447, 467 -> 456; d 2304 444 -> 435, 479 -> 481, 534 -> 506; d 2432 467 -> 472, 498 -> 509, 556 -> 538; d 2560
// 472 -> 476, 507 -> 521, 563 -> 552; d 3072 521 -> 565, 594 -> 612, 616 -> 646 (grouped heads 1 to 3 % to the launches' side of these).
bool one_kernel_asked(const anpd_model &m) { return m.cfg.gemm_path != ANPD_GEMM_AUTO || m.trace; }   // by name, or by a trace of its barriers
bool one_kernel_taken(const anpd_model &m) { return m.mega && (one_kernel_asked(m) || m.cfg.d_model >= 2048); }
// Windows of 9 to 16 rows, whose GEMMs have a tile per wave as separate launches: those are the faster form, us, one kernel -> launches, 8
// layers, 9 rows at 64 / 512 / 1000 / 2048 / 4000 positions: 7B shape 883 -> 839, 884 -> 852, 894 -> 868, 988 -> 908, 1029 -> 1005; d 3072
// 666 -> 600, 661 -> 603, 663 -> 621, 772 -> 671, 798 -> 709 (eight key / value heads 657 -> 603, 656 -> 609, 654 -> 624, 758 -> 670, 765 -> 698);
// d 2048 529 -> 435, 532 -> 436, 536 -> 441, 585 -> 481, 595 -> 513.  Where key / value heads are few, d is above 3072 and the positions are
// no more than 1024, attention's launch has little to do and the two are level, which is where the one kernel stays: ChatGLM3 shape 955 -> 931,
// 943 -> 941, 953 -> 948 (16 rows 964 -> 953, 954 -> 967, 964 -> 977); d 4096 with four of them 915 -> 882, 905 -> 894, 910 -> 905 (924 -> 899,
// 915 -> 912, 923 -> 925), with eight 929 -> 899, 925 -> 910, 928 -> 923 (938 -> 919, 936 -> 934, 938 -> 946); beyond, at 2048 / 4000, ChatGLM3 shape
// 1036 -> 989, 1043 -> 1020, eight 1024 -> 962, 1043 -> 1055 (16 rows 1034 -> 984, 1056 -> 1083).
bool one_kernel_rows16(const anpd_model &m, int positions)
{
    return one_kernel_asked(m) || (m.cfg.d_model > 3072 && kv_heads_of(m.cfg) < m.cfg.n_heads && n_splits_of(positions) <= kSmallSplits);
}

// After the stream has been synchronised: was there a launch of the small model's kernel of which no block ran where it was to run, so
// that nothing was done?  Then steps are separate launches from here on.
bool small_missed(anpd_model *m)
{
    if (m->xcd < 0 || (uint32_t)m->pin[102] == m->small_launches) return false;
    m->xcd = -1;
    return true;
}

// After the stream has been synchronised: did a grid barrier of the one-kernel step give up?  Then the
// counters are no longer in step: start them over.
bool barrier_gave_up(anpd_model *m, hipStream_t st)
{
    if (m->pin[100] == 0) return false;
    m->pin[100] = 0;
    if (!m->mfma) {   // (the one launch of a small model: nothing else on this path waits)
        if (m->lay.small_stride == 0) return true;
        (void)hipMemsetAsync(m->ws + m->lay.small_ctr, 0, 2 * kSmallLine * sizeof(uint32_t), st);
        (void)hipMemsetAsync(m->ws + m->lay.gen_ctr, 0, (size_t)m->cfg.n_heads * ((m->lay.gen_part_rows + 15) / 16) * 64 * sizeof(uint32_t), st);
        (void)hipStreamSynchronize(st);
        m->small_launches = (uint32_t)m->pin[102];
        return true;
    }
    (void)hipMemsetAsync(m->ws + m->lay.bar, 0, kBarStride * 9 * sizeof(uint32_t) + (size_t)m->cfg.n_heads * kCounterStride * sizeof(uint32_t), st);
    (void)hipStreamSynchronize(st);
    m->bar_epoch = 0;
    m->ready_epoch = 0;
    return true;
}

}  // namespace

extern "C" {

size_t anpd_model_workspace_bytes(const anpd_model_cfg *cfg)
{
    const char *why;
    if (!cfg_ok(cfg, &why)) { fail(ANPD_E_INVAL, "anpd_model_workspace_bytes: %s", why); return 0; }
    return make_layout(cfg).total;
}

int32_t anpd_model_create(const anpd_model_cfg *cfg, const anpd_weights *w, void *workspace, size_t workspace_bytes,
                          void *stream, anpd_model_t **out)
{
    if (!out) return fail(ANPD_E_INVAL, "anpd_model_create: out is NULL");
    *out = nullptr;
    const char *why;
    if (!cfg_ok(cfg, &why)) return fail(ANPD_E_INVAL, "anpd_model_create: %s", why);
    if (!w || !workspace) return fail(ANPD_E_INVAL, "anpd_model_create: NULL weights or workspace");
    if (((uintptr_t)workspace & 255) != 0) return fail(ANPD_E_INVAL, "anpd_model_create: workspace must be 256-byte aligned");
    Layout lay = make_layout(cfg);
    if (workspace_bytes < lay.total)
        return fail(ANPD_E_CAPACITY, "anpd_model_create: workspace has %zu bytes, %zu needed", workspace_bytes, lay.total);
    if (!w->embed || !w->final_norm || !w->lm_head || !w->attn_norm || !w->wq || !w->wk || !w->wv || !w->wo ||
        !w->ffn_norm || !w->w_gate || !w->w_up || !w->w_down)
        return fail(ANPD_E_INVAL, "anpd_model_create: a weight pointer is NULL");
    for (int l = 0; l < cfg->n_layers; ++l)
        if (!w->attn_norm[l] || !w->wq[l] || !w->wk[l] || !w->wv[l] || !w->wo[l] || !w->ffn_norm[l] || !w->w_gate[l] ||
            !w->w_up[l] || !w->w_down[l])
            return fail(ANPD_E_INVAL, "anpd_model_create: a weight pointer of layer %d is NULL", l);

    anpd_model *m = new (std::nothrow) anpd_model;
    if (!m) return fail(ANPD_E_NOMEM, "anpd_model_create: out of memory");
    m->cfg = *cfg;
    m->lay = lay;
    m->ws = (char *)workspace;
    m->mfma = wants_mfma(cfg);
    {
        int dev = 0;
        hipDeviceProp_t prop;
        m->n_cu = 256;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0)
            m->n_cu = prop.multiProcessorCount;
        // (where the workspace lies, which is where the step runs)
        hipPointerAttribute_t at;
        m->device = dev;
        if (hipPointerGetAttributes(&at, workspace) == hipSuccess) m->device = at.device;
        else (void)hipGetLastError();
    }
    m->embed = w->embed;
    m->final_norm = w->final_norm;
    m->lm_head = w->lm_head;
    const size_t nl = (size_t)cfg->n_layers;
    m->attn_norm.assign(w->attn_norm, w->attn_norm + nl);
    m->wq.assign(w->wq, w->wq + nl);
    m->wk.assign(w->wk, w->wk + nl);
    m->wv.assign(w->wv, w->wv + nl);
    m->wo.assign(w->wo, w->wo + nl);
    m->ffn_norm.assign(w->ffn_norm, w->ffn_norm + nl);
    m->w_gate.assign(w->w_gate, w->w_gate + nl);
    m->w_up.assign(w->w_up, w->w_up + nl);
    m->w_down.assign(w->w_down, w->w_down + nl);
    m->pin = nullptr;
    m->prof = false;
    m->ev_used = 0;
    m->prof_steps = 0;
    for (int i = 0; i < ANPD_PROF_NCAT; ++i) { m->prof_ms[i] = 0.0; m->prof_launches[i] = 0; }

    hipStream_t st = (hipStream_t)stream;
    // cos/sin of pos * base^(-2i/head_dim), evaluated in double, stored as float
    const int half = cfg->head_dim / 2;
    std::vector<float2> tab((size_t)cfg->max_positions * half);
    for (int i = 0; i < half; ++i) {
        double theta = std::pow((double)cfg->rope_base, -2.0 * (double)i / (double)cfg->head_dim);
        for (int p = 0; p < cfg->max_positions; ++p) {
            double ang = (double)p * theta;
            tab[(size_t)p * half + i] = make_float2((float)std::cos(ang), (float)std::sin(ang));
        }
    }
    hipError_t e = hipHostMalloc((void **)&m->pin, 1024 * sizeof(int32_t), hipHostMallocDefault);
    if (e != hipSuccess) { delete m; return fail(ANPD_E_HIP, "hipHostMalloc: %s", hipGetErrorString(e)); }
    std::memset(m->pin, 0, 1024 * sizeof(int32_t));
    e = hipHostGetDevicePointer((void **)&m->pin_dev, m->pin, 0);
    if (e != hipSuccess) { (void)hipHostFree(m->pin); delete m; return fail(ANPD_E_HIP, "hipHostGetDevicePointer: %s", hipGetErrorString(e)); }
    e = hipMemsetAsync(m->ws, 0, m->mfma ? lay.wp_lm : lay.total, st);
    if (e == hipSuccess) e = hipMemcpyAsync(m->ws + lay.rope_tab, tab.data(), tab.size() * sizeof(float2), hipMemcpyHostToDevice, st);
    int32_t prc = ANPD_OK;
    m->mega = false;
    m->mega_tree = false;
    m->mega_batch = false;
    m->trace = nullptr;
    m->mega_grid = 0;
    m->bar_epoch = 0;
    m->ready_epoch = 0;
    m->xcd = -1;
    m->small_launches = m->small_launch = 0;
    m->spin_limit = 1 << 21;
    // ANPD_MEGA_PLAIN_LAUNCH=1: an ordinary launch of the same grid.  Only for profilers that cannot
    // cope with the cooperative queue; all blocks are resident only if nothing else runs on the device
    // (otherwise a barrier wait times out and anpd_verify reports it).
    {
        const char *pl = std::getenv("ANPD_MEGA_PLAIN_LAUNCH");
        m->plain_launch = pl && pl[0] == '1';
    }
    m->mega_rows16 = false;
    m->mega_kc = (cfg->d_model + 31) / 32 <= 2 * kChunk * kFastWaves ? kChunk : 10;
    if (e == hipSuccess && m->mfma && cfg->gemm_path != ANPD_GEMM_MFMA_LAUNCHES && (cfg->d_model + 31) / 32 <= 2 * 10 * kFastWaves) {
        // the persistent step needs every block resident at once: one block per compute unit
        int per_cu = 0;
        hipError_t oe;
        if (m->mega_kc == kChunk)
            oe = cfg->head_dim == 128 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, verify_mega_kernel<128>, kFastThreads, 0)
                                      : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, verify_mega_kernel<64>, kFastThreads, 0);
        else
            oe = cfg->head_dim == 128
                     ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, verify_mega_kernel<128, MEGA_CHAIN, 1, 10>, kFastThreads, 0)
                     : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, verify_mega_kernel<64, MEGA_CHAIN, 1, 10>, kFastThreads, 0);
        if (oe == hipSuccess && per_cu >= 1) {
            std::vector<LayerW> tab((size_t)cfg->n_layers);
            for (int l = 0; l < cfg->n_layers; ++l) {
                tab[(size_t)l].qkv = (const uint4 *)(m->ws + lay.wp_qkv[(size_t)l]);
                tab[(size_t)l].o = (const uint4 *)(m->ws + lay.wp_o[(size_t)l]);
                tab[(size_t)l].gu = (const uint4 *)(m->ws + lay.wp_gu[(size_t)l]);
                tab[(size_t)l].down = (const uint4 *)(m->ws + lay.wp_down[(size_t)l]);
                tab[(size_t)l].attn_gain = (const bf16_t *)m->attn_norm[(size_t)l];
                tab[(size_t)l].ffn_gain = (const bf16_t *)m->ffn_norm[(size_t)l];
            }
            e = hipMemcpyAsync(m->ws + lay.layer_tab, tab.data(), tab.size() * sizeof(LayerW), hipMemcpyHostToDevice, st);
            if (e == hipSuccess) e = hipStreamSynchronize(st);  // `tab` is about to go out of scope
            m->mega = true;
            m->mega_grid = m->n_cu;
            int per_cu_t = 0;
            hipError_t te = cfg->head_dim == 128
                                ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_t, verify_mega_kernel<128, MEGA_TREE>, kFastThreads, 0)
                                : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_t, verify_mega_kernel<64, MEGA_TREE>, kFastThreads, 0);
            m->mega_tree = te == hipSuccess && per_cu_t >= 1 && m->mega_kc == kChunk;
            if (te != hipSuccess) (void)hipGetLastError();
            int per_cu_b = 0;
            te = cfg->head_dim == 128
                     ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_b, verify_mega_kernel<128, MEGA_BATCH>, kFastThreads, 0)
                     : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_b, verify_mega_kernel<64, MEGA_BATCH>, kFastThreads, 0);
            m->mega_batch = te == hipSuccess && per_cu_b >= 1 && m->mega_kc == kChunk;
            if (te != hipSuccess) (void)hipGetLastError();
            int per_cu_r = 0;
            te = cfg->head_dim == 128
                     ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_r, verify_mega_kernel<128, MEGA_CHAIN, 2>, kFastThreads, 0)
                     : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_r, verify_mega_kernel<64, MEGA_CHAIN, 2>, kFastThreads, 0);
            m->mega_rows16 = te == hipSuccess && per_cu_r >= 1 && m->mega_kc == kChunk;
            if (te != hipSuccess) (void)hipGetLastError();

        } else {
            (void)hipGetLastError();
        }
    }
    if (e == hipSuccess && m->mfma) {
        // repack every matrix into MFMA-fragment order inside the workspace
        const int d = cfg->d_model, F = cfg->d_ffn, dh = cfg->head_dim, kvd = kv_dim_of(*cfg);
        for (int l = 0; l < cfg->n_layers && prc == ANPD_OK; ++l) {
            prc = launch_pack(m->wq[l], m->wk[l], m->wv[l], m->ws + lay.wp_qkv[(size_t)l], PACK_QKV, (d + 2 * kvd) / 16, d, d, dh, kvd, st);
            if (prc == ANPD_OK) prc = launch_pack(m->wo[l], nullptr, nullptr, m->ws + lay.wp_o[(size_t)l], PACK_PLAIN, d / 16, d, d, dh, kvd, st);
            if (prc == ANPD_OK) prc = launch_pack(m->w_gate[l], m->w_up[l], nullptr, m->ws + lay.wp_gu[(size_t)l], PACK_GATE_UP, F / 8, d, d, dh, kvd, st);
            if (prc == ANPD_OK) prc = launch_pack(m->w_down[l], nullptr, nullptr, m->ws + lay.wp_down[(size_t)l], PACK_PLAIN, d / 16, F, d, dh, kvd, st);
        }
        if (prc == ANPD_OK) prc = launch_pack(m->lm_head, nullptr, nullptr, m->ws + lay.wp_lm, PACK_PLAIN, cfg->vocab / 16, d, d, dh, kvd, st);
    }
    if (e == hipSuccess && small_model(*cfg)) {
        // where blocks of such a grid run: the XCD with the most of them
        uint32_t *count = (uint32_t *)(m->ws + lay.small_ctr), seen[16];
        std::vector<GenLayer> tab(nl);
        for (size_t l = 0; l < nl; ++l)
            tab[l] = {m->attn_norm[l], m->wq[l], m->wk[l], m->wv[l], m->wo[l], m->ffn_norm[l], m->w_gate[l], m->w_up[l], m->w_down[l]};
        e = hipMemcpyAsync(m->ws + lay.small_layers, tab.data(), nl * sizeof(GenLayer), hipMemcpyHostToDevice, st);
        hipLaunchKernelGGL(xcd_census_kernel, dim3(kSmallBlocks), dim3(512), 0, st, count);
        if (e == hipSuccess) e = hipGetLastError();
        if (e == hipSuccess) e = hipMemcpyAsync(seen, count, sizeof(seen), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipMemsetAsync(count, 0, sizeof(seen), st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        for (int i = 0; e == hipSuccess && i < 16; ++i)
            if (seen[i] >= 16 && (m->xcd < 0 || seen[i] > seen[m->xcd])) m->xcd = i;
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess || prc != ANPD_OK) {
        (void)hipHostFree(m->pin);
        delete m;
        return prc != ANPD_OK ? prc : fail(ANPD_E_HIP, "anpd_model_create: %s", hipGetErrorString(e));
    }
    *out = m;
    return ANPD_OK;
}

void anpd_model_destroy(anpd_model_t *m)
{
    if (!m) return;
    if (m->pin) (void)hipHostFree(m->pin);
    for (hipEvent_t e : m->ev) (void)hipEventDestroy(e);
    delete m;
}

int32_t anpd_model_trace(anpd_model_t *m, void *buffer, size_t bytes)
{
    if (!m) return fail(ANPD_E_INVAL, "anpd_model_trace: NULL handle");
    if (buffer && (!m->mega || bytes < (size_t)m->mega_grid * kTraceEvents * sizeof(long long)))
        return fail(ANPD_E_CAPACITY, "anpd_model_trace: needs %zu bytes and the one-kernel step",
                    (size_t)m->mega_grid * kTraceEvents * sizeof(long long));
    m->trace = (long long *)buffer;
    return m->mega ? m->mega_grid : 0;
}

int32_t anpd_model_set_barrier_spin_limit(anpd_model_t *m, int32_t spins)
{
    if (!m) return fail(ANPD_E_INVAL, "anpd_model_set_barrier_spin_limit: NULL handle");
    if (spins < 0) return fail(ANPD_E_INVAL, "anpd_model_set_barrier_spin_limit: spins must be >= 0");
    m->spin_limit = spins == 0 ? (1 << 21) : spins;
    return ANPD_OK;
}

int32_t anpd_model_profile(anpd_model_t *m, int32_t enable)
{
    if (!m) return fail(ANPD_E_INVAL, "anpd_model_profile: NULL handle");
    m->prof = enable != 0;
    m->prof_steps = 0;
    for (int i = 0; i < ANPD_PROF_NCAT; ++i) { m->prof_ms[i] = 0.0; m->prof_launches[i] = 0; }
    return ANPD_OK;
}

int32_t anpd_model_profile_read(const anpd_model_t *m, double *out_ms, int64_t *out_launches, int64_t *out_steps)
{
    if (!m || !out_ms || !out_launches || !out_steps) return fail(ANPD_E_INVAL, "anpd_model_profile_read: NULL argument");
    for (int i = 0; i < ANPD_PROF_NCAT; ++i) { out_ms[i] = m->prof_ms[i]; out_launches[i] = m->prof_launches[i]; }
    *out_steps = m->prof_steps;
    return ANPD_OK;
}

size_t anpd_kv_pool_bytes(const anpd_model_t *m, int32_t max_tokens)
{
    if (!m || max_tokens < 1 || max_tokens > m->cfg.max_positions) {
        fail(ANPD_E_INVAL, "anpd_kv_pool_bytes: bad argument");
        return 0;
    }
    const int pt = m->cfg.page_tokens;
    size_t pages = (size_t)(max_tokens + pt - 1) / pt;
    return align_up(pages * page_bytes_of(m->cfg)) + align_up((pages + 1) * sizeof(int32_t));
}

int32_t anpd_kv_create(const anpd_model_t *m, void *pool, size_t pool_bytes, int32_t max_tokens, anpd_kv_t **out)
{
    if (!out) return fail(ANPD_E_INVAL, "anpd_kv_create: out is NULL");
    *out = nullptr;
    if (!m || !pool) return fail(ANPD_E_INVAL, "anpd_kv_create: NULL model or pool");
    if (max_tokens < 1 || max_tokens > m->cfg.max_positions)
        return fail(ANPD_E_CAPACITY, "anpd_kv_create: max_tokens %d outside 1..max_positions (%d)", max_tokens, m->cfg.max_positions);
    if (((uintptr_t)pool & 255) != 0) return fail(ANPD_E_INVAL, "anpd_kv_create: pool must be 256-byte aligned");
    size_t need = anpd_kv_pool_bytes(m, max_tokens);
    if (pool_bytes < need) return fail(ANPD_E_CAPACITY, "anpd_kv_create: pool has %zu bytes, %zu needed", pool_bytes, need);
    anpd_kv *kv = new (std::nothrow) anpd_kv;
    if (!kv) return fail(ANPD_E_NOMEM, "anpd_kv_create: out of memory");
    const int pt = m->cfg.page_tokens;
    kv->m = m;
    kv->pool = (char *)pool;
    kv->n_pages = (max_tokens + pt - 1) / pt;
    kv->max_tokens = max_tokens;
    kv->len = 0;
    kv->page_bytes = page_bytes_of(m->cfg);
    kv->table.assign((size_t)kv->n_pages, -1);
    kv->dev_table.assign((size_t)kv->n_pages, -1);
    for (int p = kv->n_pages - 1; p >= 0; --p) kv->free_list.push_back(p);  // page 0 is handed out first
    char *tail = kv->pool + align_up((size_t)kv->n_pages * kv->page_bytes);
    kv->d_len = (int32_t *)tail;
    kv->d_table = kv->d_len + 1;
    kv->table_dirty = true;
    kv->pin = nullptr;
    hipError_t e = hipHostMalloc((void **)&kv->pin, ((size_t)kv->n_pages + 1) * sizeof(int32_t), hipHostMallocDefault);
    if (e == hipSuccess) e = hipMemset(kv->pool, 0, need);  // unwritten slots must read as zeros, never as NaN patterns
    if (e == hipSuccess) {
        kv->pin[0] = 0;
        e = hipMemcpy(kv->d_len, kv->pin, sizeof(int32_t), hipMemcpyHostToDevice);
    }
    if (e != hipSuccess) {
        if (kv->pin) (void)hipHostFree(kv->pin);
        delete kv;
        return fail(ANPD_E_HIP, "anpd_kv_create: %s", hipGetErrorString(e));
    }
    *out = kv;
    return ANPD_OK;
}

void anpd_kv_destroy(anpd_kv_t *kv)
{
    if (!kv) return;
    if (kv->pin) (void)hipHostFree(kv->pin);
    delete kv;
}

int32_t anpd_kv_length(const anpd_kv_t *kv) { return kv ? kv->len : fail(ANPD_E_INVAL, "anpd_kv_length: NULL handle"); }

int32_t anpd_kv_num_pages(const anpd_kv_t *kv) { return kv ? kv->n_pages : fail(ANPD_E_INVAL, "anpd_kv_num_pages: NULL handle"); }

int32_t anpd_kv_set_page_order(anpd_kv_t *kv, const int32_t *perm, int32_t n_pages)
{
    if (!kv || !perm) return fail(ANPD_E_INVAL, "anpd_kv_set_page_order: NULL argument");
    if (n_pages != kv->n_pages) return fail(ANPD_E_INVAL, "anpd_kv_set_page_order: expected %d entries", kv->n_pages);
    if ((int)kv->free_list.size() != kv->n_pages) return fail(ANPD_E_INVAL, "anpd_kv_set_page_order: cache is not empty");
    std::vector<char> seen((size_t)n_pages, 0);
    for (int i = 0; i < n_pages; ++i) {
        if (perm[i] < 0 || perm[i] >= n_pages || seen[(size_t)perm[i]])
            return fail(ANPD_E_INVAL, "anpd_kv_set_page_order: not a permutation");
        seen[(size_t)perm[i]] = 1;
    }
    for (int i = 0; i < n_pages; ++i) kv->free_list[(size_t)(n_pages - 1 - i)] = perm[i];
    return ANPD_OK;
}

int32_t anpd_kv_truncate(anpd_kv_t *kv, int32_t new_len, void *stream)
{
    if (!kv) return fail(ANPD_E_INVAL, "anpd_kv_truncate: NULL handle");
    if (new_len < 0 || new_len > kv->max_tokens)
        return fail(ANPD_E_CAPACITY, "anpd_kv_truncate: length %d outside 0..%d", new_len, kv->max_tokens);
    hipStream_t st = (hipStream_t)stream;
    int32_t rc = ensure_pages(kv, new_len, st);
    if (rc != ANPD_OK) return rc;
    kv->pin[0] = new_len;
    HIP_TRY(hipMemcpyAsync(kv->d_len, kv->pin, sizeof(int32_t), hipMemcpyHostToDevice, st));
    HIP_TRY(hipStreamSynchronize(st));
    kv->len = new_len;
    release_pages(kv, new_len);
    return ANPD_OK;
}

static int32_t kv_copy(anpd_kv *kv, int32_t layer, int32_t pos0, int32_t n, float *k, float *v, bool to_cache, void *stream)
{
    if (!kv || ((!k || !v) && n != 0)) return fail(ANPD_E_INVAL, "anpd_kv_read/write: NULL argument");
    const anpd_model_cfg &c = kv->m->cfg;
    if (layer < 0 || layer >= c.n_layers || pos0 < 0 || n < 0 || pos0 + n > kv->max_tokens)
        return fail(ANPD_E_CAPACITY, "anpd_kv_read/write: layer %d, positions %d..%d out of range", layer, pos0, pos0 + n);
    if (n == 0) return ANPD_OK;
    hipStream_t st = (hipStream_t)stream;
    if (to_cache) {
        int32_t rc = ensure_pages(kv, pos0 + n, st);
        if (rc != ANPD_OK) return rc;
    } else {
        const int pt = c.page_tokens;
        for (int lp = pos0 / pt; lp <= (pos0 + n - 1) / pt; ++lp)
            if (kv->table[(size_t)lp] < 0) return fail(ANPD_E_INVAL, "anpd_kv_read: position %d has no page", lp * pt);
    }
#define KV_COPY(KT, TO)                                                                                          \
    hipLaunchKernelGGL((kv_copy_kernel<KT, TO>), dim3(n), dim3(256), 0, st, (KT *)kv->pool, kv->d_table, k, v, pos0, \
                       layer, c.n_layers, kv_heads_of(c), c.head_dim, c.page_tokens)
    if (kv->m->mfma) {
        if (to_cache)
            hipLaunchKernelGGL((kvf_copy_kernel<true>), dim3(n), dim3(256), 0, st, (bf16_t *)kv->pool, kv->d_table, k, v, pos0,
                               layer, c.n_layers, kv_heads_of(c), c.head_dim);
        else
            hipLaunchKernelGGL((kvf_copy_kernel<false>), dim3(n), dim3(256), 0, st, (bf16_t *)kv->pool, kv->d_table, k, v, pos0,
                               layer, c.n_layers, kv_heads_of(c), c.head_dim);
    } else if (c.dtype == ANPD_BF16) { if (to_cache) KV_COPY(bf16_t, true); else KV_COPY(bf16_t, false); }
    else { if (to_cache) KV_COPY(float, true); else KV_COPY(float, false); }
#undef KV_COPY
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(st));
    return ANPD_OK;
}

int32_t anpd_kv_write(anpd_kv_t *kv, int32_t layer, int32_t pos0, int32_t n, const float *k, const float *v, void *stream)
{
    return kv_copy(kv, layer, pos0, n, const_cast<float *>(k), const_cast<float *>(v), true, stream);
}

int32_t anpd_kv_read(const anpd_kv_t *kv, int32_t layer, int32_t pos0, int32_t n, float *k, float *v, void *stream)
{
    return kv_copy(const_cast<anpd_kv *>(kv), layer, pos0, n, k, v, false, stream);
}

int32_t anpd_verify(anpd_model_t *m, anpd_kv_t *kv, const int32_t *window, int32_t n_window, int32_t mode,
                    int32_t *out_accepted, int32_t *out_next, int32_t *out_predicts, float *out_logits, void *stream)
{
    if (!m || !kv || !window || !out_accepted || !out_next) return fail(ANPD_E_INVAL, "anpd_verify: NULL argument");
    if (kv->m != m) return fail(ANPD_E_INVAL, "anpd_verify: the cache belongs to another model");
    if (mode != ANPD_VERIFY && mode != ANPD_APPEND) return fail(ANPD_E_INVAL, "anpd_verify: unknown mode %d", mode);
    if (n_window < 1) return fail(ANPD_E_INVAL, "anpd_verify: n_window must be >= 1");
    if (n_window > m->cfg.max_window)
        return fail(ANPD_E_CAPACITY, "anpd_verify: n_window %d exceeds max_window %d", n_window, m->cfg.max_window);
    if (kv->len + n_window > kv->max_tokens)
        return fail(ANPD_E_CAPACITY, "anpd_verify: length %d + window %d exceeds capacity %d", kv->len, n_window, kv->max_tokens);
    for (int i = 0; i < n_window; ++i)
        if (window[i] < 0 || window[i] >= m->cfg.vocab)
            return fail(ANPD_E_RANGE, "anpd_verify: token %d at window[%d] outside [0, %d)", window[i], i, m->cfg.vocab);

    hipStream_t st = (hipStream_t)stream;
    int32_t rc = ensure_pages(kv, kv->len + n_window, st);
    if (rc != ANPD_OK) return rc;
    // The window goes to the kernels by value, and they write the result (and the persistent kernel its error
    // flag) into the pinned buffer themselves.
    const bool one_kernel = one_kernel_taken(*m) && (n_window <= 8 || (n_window <= 16 && m->mega_rows16 && one_kernel_rows16(*m, kv->len + n_window)));
    const int32_t *res = m->pin + 32;
    LogitsTo logits = {out_logits, (size_t)n_window * m->cfg.vocab, nullptr};
    if (one_kernel) rc = run_step_mega(m, kv, window, n_window, mode, out_logits ? logits.find(m) : nullptr, st);
    else if (m->mfma) rc = run_step_fast(m, kv, step_tokens(window, n_window), n_window, mode, logits, st);
    else rc = run_step_weights(m, kv, window, n_window, mode, logits, st);
    if (rc != ANPD_OK) return rc;
    if (logits.elsewhere())
        HIP_TRY(hipMemcpyAsync(out_logits, logits.at, sizeof(float) * (size_t)n_window * m->cfg.vocab, hipMemcpyDeviceToDevice, st));
    HIP_TRY(hipStreamSynchronize(st));
    if (barrier_gave_up(m, st)) return fail(ANPD_E_HIP, "anpd_verify: a wait inside the step's kernel timed out");
    if (small_missed(m)) return anpd_verify(m, kv, window, n_window, mode, out_accepted, out_next, out_predicts, out_logits, stream);
    collect_marks(m);
    *out_accepted = res[0];
    *out_next = res[1];
    if (out_predicts) std::memcpy(out_predicts, res + 2, sizeof(int32_t) * (size_t)n_window);
    kv->len += 1 + res[0];
    release_pages(kv, kv->len);
    return ANPD_OK;
}

int32_t anpd_verify_tree(anpd_model_t *m, anpd_kv_t *kv, const int32_t *window, const int32_t *parent, int32_t n_window,
                         int32_t *out_accepted, int32_t *out_next, int32_t *out_path, int32_t *out_predicts, float *out_logits,
                         void *stream)
{
    if (!m || !kv || !window || !parent || !out_accepted || !out_next) return fail(ANPD_E_INVAL, "anpd_verify_tree: NULL argument");
    if (kv->m != m) return fail(ANPD_E_INVAL, "anpd_verify_tree: the cache belongs to another model");
    if (n_window < 1) return fail(ANPD_E_INVAL, "anpd_verify_tree: n_window must be >= 1");
    if (n_window > m->cfg.max_window)
        return fail(ANPD_E_CAPACITY, "anpd_verify_tree: n_window %d exceeds max_window %d", n_window, m->cfg.max_window);
    if (kv->len + n_window > kv->max_tokens)
        return fail(ANPD_E_CAPACITY, "anpd_verify_tree: length %d + window %d exceeds capacity %d", kv->len, n_window, kv->max_tokens);
    if (parent[0] != -1) return fail(ANPD_E_INVAL, "anpd_verify_tree: parent[0] must be -1");
    for (int i = 0; i < n_window; ++i) {
        if (window[i] < 0 || window[i] >= m->cfg.vocab)
            return fail(ANPD_E_RANGE, "anpd_verify_tree: token %d at window[%d] outside [0, %d)", window[i], i, m->cfg.vocab);
        if (i > 0 && (parent[i] < 0 || parent[i] >= i))
            return fail(ANPD_E_INVAL, "anpd_verify_tree: parent[%d] = %d is not an earlier row", i, parent[i]);
    }
    hipStream_t st = (hipStream_t)stream;
    int32_t rc = ensure_pages(kv, kv->len + n_window, st);
    if (rc != ANPD_OK) return rc;
    // depth and visibility (self + ancestors) of every row
    int32_t *tp = m->pin + 128, *td = tp + ANPD_MAX_WINDOW;
    uint32_t *tm = (uint32_t *)(td + ANPD_MAX_WINDOW);
    for (int i = 0; i < ANPD_MAX_WINDOW; ++i) { tp[i] = 0; td[i] = 0; tm[i] = 0; }
    tp[0] = -1;
    tm[0] = 1u;
    for (int i = 1; i < n_window; ++i) {
        tp[i] = parent[i];
        td[i] = td[parent[i]] + 1;
        tm[i] = tm[parent[i]] | (1u << i);
    }
    const int32_t *res = m->pin + 32;
    LogitsTo logits = {out_logits, (size_t)n_window * m->cfg.vocab, nullptr};
    // windows of up to 8 rows: the one-kernel step in its draft-tree form (tree by value as well); otherwise one
    // launch per operation, the tree written to device memory by a kernel in front
    const bool one_kernel = one_kernel_taken(*m) && m->mega_tree && n_window <= 8;
    if (one_kernel) {
        rc = run_step_mega(m, kv, window, n_window, ANPD_APPEND, out_logits ? logits.find(m) : nullptr, st, tp);
    } else {
        UploadWords up;
        std::memcpy(up.w, tp, sizeof(int32_t) * 3 * ANPD_MAX_WINDOW);
        hipLaunchKernelGGL(upload_kernel, dim3(1), dim3(kUploadWords), 0, st, (uint32_t *)(m->ws + m->lay.tree), up, 3 * ANPD_MAX_WINDOW);
        if (m->mfma) rc = run_step_fast(m, kv, step_tokens(window, n_window), n_window, ANPD_APPEND, logits, st, true);
        else rc = run_step_weights(m, kv, window, n_window, ANPD_APPEND, logits, st, true);
    }
    if (rc != ANPD_OK) return rc;
    if (logits.elsewhere())
        HIP_TRY(hipMemcpyAsync(out_logits, logits.at, sizeof(float) * (size_t)n_window * m->cfg.vocab, hipMemcpyDeviceToDevice, st));
    HIP_TRY(hipStreamSynchronize(st));
    if (barrier_gave_up(m, st)) return fail(ANPD_E_HIP, "anpd_verify_tree: a wait inside the step's kernel timed out");
    if (small_missed(m)) return anpd_verify_tree(m, kv, window, parent, n_window, out_accepted, out_next, out_path, out_predicts, out_logits, stream);
    collect_marks(m);
    *out_accepted = res[0];
    *out_next = res[1];
    if (out_predicts) std::memcpy(out_predicts, res + 2, sizeof(int32_t) * (size_t)n_window);
    if (out_path) std::memcpy(out_path, res + 34, sizeof(int32_t) * (size_t)(res[0] + 1));
    kv->len += 1 + res[0];
    release_pages(kv, kv->len);
    return ANPD_OK;
}

int32_t anpd_verify_batch(anpd_model_t *m, anpd_kv_t *const *kvs, int32_t n_seq, const int32_t *const *windows,
                          const int32_t *n_windows, int32_t mode, int32_t *out_accepted, int32_t *out_next, float *out_logits,
                          void *stream)
{
    if (!m || !kvs || !windows || !n_windows || !out_accepted || !out_next) return fail(ANPD_E_INVAL, "anpd_verify_batch: NULL argument");
    if (mode != ANPD_VERIFY && mode != ANPD_APPEND) return fail(ANPD_E_INVAL, "anpd_verify_batch: unknown mode %d", mode);
    if (n_seq < 1 || n_seq > ANPD_MAX_WINDOW) return fail(ANPD_E_INVAL, "anpd_verify_batch: n_seq must be in 1..%d", ANPD_MAX_WINDOW);
    if (!m->mfma) return fail(ANPD_E_UNIMPLEMENTED, "anpd_verify_batch: needs the matrix-core path (bf16 weights)");
    int total = 0;
    for (int s = 0; s < n_seq; ++s) {
        anpd_kv *kv = kvs[s];
        if (!kv || !windows[s]) return fail(ANPD_E_INVAL, "anpd_verify_batch: NULL cache or window of sequence %d", s);
        if (kv->m != m) return fail(ANPD_E_INVAL, "anpd_verify_batch: cache %d belongs to another model", s);
        for (int t = 0; t < s; ++t)
            if (kvs[t] == kv) return fail(ANPD_E_INVAL, "anpd_verify_batch: sequences %d and %d share a cache", t, s);
        if (n_windows[s] < 1) return fail(ANPD_E_INVAL, "anpd_verify_batch: n_windows[%d] must be >= 1", s);
        if (kv->len + n_windows[s] > kv->max_tokens)
            return fail(ANPD_E_CAPACITY, "anpd_verify_batch: sequence %d: length %d + window %d exceeds capacity %d", s, kv->len,
                        n_windows[s], kv->max_tokens);
        for (int i = 0; i < n_windows[s]; ++i)
            if (windows[s][i] < 0 || windows[s][i] >= m->cfg.vocab)
                return fail(ANPD_E_RANGE, "anpd_verify_batch: token %d at window %d row %d outside [0, %d)", windows[s][i], s, i, m->cfg.vocab);
        total += n_windows[s];
        if (total > m->cfg.max_window)
            return fail(ANPD_E_CAPACITY, "anpd_verify_batch: %d rows in all exceed max_window %d", total, m->cfg.max_window);
    }
    hipStream_t st = (hipStream_t)stream;
    for (int s = 0; s < n_seq; ++s) {
        int32_t rc = ensure_pages(kvs[s], kvs[s]->len + n_windows[s], st);
        if (rc != ANPD_OK) return rc;
    }
    // joint window, sequence of every row, sequences
    int32_t *row_seq = m->pin + 384;
    SeqRef *seqs = (SeqRef *)(m->pin + 512);
    BatchLaunch bl = {n_seq, 0, false, false};
    int row = 0;
    long long positions = 0;
    long long pages = 0, longest = 0;   // that one wave of attn_decode_kernel goes through: of all sequences, of the longest
    for (int s = 0; s < n_seq; ++s) {
        anpd_kv *kv = kvs[s];
        seqs[s].pool = (bf16_t *)kv->pool;
        seqs[s].page_table = kv->d_table;
        seqs[s].len_ptr = kv->d_len;
        seqs[s].row0 = row;
        seqs[s].n_rows = n_windows[s];
        const int splits = n_splits_of(kv->len + n_windows[s]);
        if (splits > bl.grid_splits) bl.grid_splits = splits;
        positions += kv->len + n_windows[s];
        const long long walk = kv->len / (16 * kFastWaves) + 1;
        pages += walk;
        if (walk > longest) longest = walk;
        for (int i = 0; i < n_windows[s]; ++i, ++row) {
            m->pin[row] = windows[s][i];
            row_seq[row] = s;
        }
    }
    // One row per sequence: one block per (head, sequence) once those fill the chip (two fit a compute unit), with a
    // margin where the sequences are long and a half-empty last round costs more (7B shape, 4 layers, us per step, cut
    // into splits -> not cut: 500 positions, 10 / 16 / 18 / 32 sequences 597 -> 608, 675 -> 659, 760 -> 750, 917 -> 843;
    // 2500 positions, 10 / 16 / 18 / 24 / 32 sequences 854 -> 958, 1103 -> 1126, 1236 -> 1267, 1491 -> 1476, 1778 -> 1744;
    // 13B shape, 13 sequences, a second round of 8 blocks: 500 positions 874 -> 871, 1000 positions 991 -> 1003)
    // - unless one long sequence would be walked alone, by eight waves a page after the other, while the chip has nothing
    // else to do: the pages per slot (two a compute unit) have to be at least 2/3 of the longest walk, half of it where
    // query heads share keys and values, whose pages then come from L2.  Beside 100-position sequences, 7B shape: 31 +
    // one of 4000 834 -> 956, 23 + one 779 -> 928, 28 + 4 of 4000 969 -> 1006, 9 + 9 of 1000 788 -> 821 (below the
    // line); 24 + 8 of 1000 858 -> 842, 24 of 300 + 8 of 3000 1164 -> 1135, 100 to 4000 in equal steps, 24 / 32
    // sequences 1333 -> 1357, 1575 -> 1565 (above it); ChatGLM3 shape: 31 + one of 4000 868 -> 993, 28 + 4 of 1000 847 -> 849
    // (below), 24 + 8 of 3000 1010 -> 965, 100 to 4000 1337 -> 1203 (above).
    const bool filled = (long long)n_seq * m->cfg.n_heads >= (bl.grid_splits <= kSmallSplits ? 2 : 3) * m->n_cu;
    const bool even = 3 * pages * m->cfg.n_heads >= (kv_heads_of(m->cfg) < m->cfg.n_heads ? 3 : 4) * longest * m->n_cu;
    bl.decode = total == n_seq && bl.grid_splits <= kDecodeSplits && filled && even;
    bl.stream = batch_streams(m->cfg, positions);
    // At most 8 rows in all (decoding batches, short windows): the persistent kernel takes the sequences by
    // value and writes the results into the pinned buffer itself; otherwise copies and the fused launches.
    const bool one_kernel = one_kernel_taken(*m) && m->mega_batch && total <= 8;
    const int32_t *res = m->pin + 256;
    LogitsTo logits = {out_logits, (size_t)total * m->cfg.vocab, nullptr};
    int32_t rc;
    if (one_kernel) {
        int32_t lens[8];
        for (int s = 0; s < n_seq; ++s) lens[s] = kvs[s]->len;
        MegaBatch mb = {n_seq, seqs, row_seq, lens};
        rc = run_step_mega(m, nullptr, m->pin, total, mode, out_logits ? logits.find(m) : nullptr, st, nullptr, &mb);
    } else {
        // sequence of every row, then the sequences (Layout::batch)
        static_assert(sizeof(SeqRef) % 4 == 0 && sizeof(UploadWords) == ANPD_MAX_WINDOW * (sizeof(int32_t) + sizeof(SeqRef)), "a batch's description");
        UploadWords up;
        std::memcpy(up.w, row_seq, ANPD_MAX_WINDOW * sizeof(int32_t));
        std::memcpy(up.w + ANPD_MAX_WINDOW, seqs, ANPD_MAX_WINDOW * sizeof(SeqRef));
        hipLaunchKernelGGL(upload_kernel, dim3(1), dim3(kUploadWords), 0, st, (uint32_t *)(m->ws + m->lay.batch), up, kUploadWords);
        rc = run_step_fast(m, nullptr, step_tokens(m->pin, total), total, mode, logits, st, false, &bl);
    }
    if (rc != ANPD_OK) return rc;
    if (logits.elsewhere())
        HIP_TRY(hipMemcpyAsync(out_logits, logits.at, sizeof(float) * (size_t)total * m->cfg.vocab, hipMemcpyDeviceToDevice, st));
    HIP_TRY(hipStreamSynchronize(st));
    if (one_kernel && barrier_gave_up(m, st)) return fail(ANPD_E_HIP, "anpd_verify_batch: a wait inside the step's kernel timed out");
    collect_marks(m);
    for (int s = 0; s < n_seq; ++s) {
        out_accepted[s] = res[2 * s];
        out_next[s] = res[2 * s + 1];
        kvs[s]->len += 1 + res[2 * s];
        release_pages(kvs[s], kvs[s]->len);
    }
    return ANPD_OK;
}

size_t anpd_prefill_workspace_bytes(const anpd_model_t *m, int32_t n_tokens)
{
    if (!m || n_tokens < 1 || n_tokens > m->cfg.max_positions) {
        fail(ANPD_E_INVAL, "anpd_prefill_workspace_bytes: bad argument");
        return 0;
    }
    return m->mfma ? make_prefill_layout(m->cfg, n_tokens).total : 0;
}

int32_t anpd_prefill(anpd_model_t *m, anpd_kv_t *kv, const int32_t *tokens, int32_t n_tokens, int32_t *out_next,
                     float *out_logits, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!m || !kv || !tokens || !out_next) return fail(ANPD_E_INVAL, "anpd_prefill: NULL argument");
    if (kv->m != m) return fail(ANPD_E_INVAL, "anpd_prefill: the cache belongs to another model");
    if (n_tokens < 1) return fail(ANPD_E_INVAL, "anpd_prefill: n_tokens must be >= 1");
    if (kv->len + n_tokens > kv->max_tokens)
        return fail(ANPD_E_CAPACITY, "anpd_prefill: length %d + %d tokens exceeds capacity %d", kv->len, n_tokens, kv->max_tokens);
    for (int i = 0; i < n_tokens; ++i)
        if (tokens[i] < 0 || tokens[i] >= m->cfg.vocab)
            return fail(ANPD_E_RANGE, "anpd_prefill: token %d at tokens[%d] outside [0, %d)", tokens[i], i, m->cfg.vocab);
    hipStream_t st = (hipStream_t)stream;
    const size_t V = (size_t)m->cfg.vocab;

    if (!m->mfma) {
        // models on the caller's weights: the prompt goes through the step's kernels in pieces of up to kGenPieceRows
        // appended rows, all enqueued before the first is waited for; logits and prediction of the last row only
        const int32_t len0 = kv->len;
        auto pieces = [&]() -> int32_t {
            int32_t rc = ensure_pages(kv, len0 + n_tokens, st);
            if (rc != ANPD_OK) return rc;
            LogitsTo logits = {out_logits, V, nullptr};
            for (int i = 0, n; i < n_tokens; i += n) {
                n = n_tokens - i < m->lay.gen_rows ? n_tokens - i : m->lay.gen_rows;
                const Piece piece = i + n < n_tokens ? PIECE_CACHE : PIECE_LAST;
                rc = run_step_weights(m, kv, tokens + i, n, ANPD_APPEND, logits, st, false, piece);
                if (rc != ANPD_OK) return rc;
                kv->len += n;
                if (m->prof) {
                    HIP_TRY(hipStreamSynchronize(st));
                    collect_marks(m);
                }
            }
            if (logits.elsewhere()) HIP_TRY(hipMemcpyAsync(out_logits, logits.at, V * sizeof(float), hipMemcpyDeviceToDevice, st));
            HIP_TRY(hipStreamSynchronize(st));
            return barrier_gave_up(m, st) ? fail(ANPD_E_HIP, "anpd_prefill: a wait inside the step's kernel timed out") : ANPD_OK;
        };
        int32_t rc = pieces();
        const bool missed = rc == ANPD_OK && small_missed(m);
        if (rc != ANPD_OK || missed) {
            // some pieces may have run, some not: the cache is what it was, on the host and on the device
            (void)hipStreamSynchronize(st);
            kv->len = len0;
            kv->pin[0] = len0;
            (void)hipMemcpyAsync(kv->d_len, kv->pin, sizeof(int32_t), hipMemcpyHostToDevice, st);
            (void)hipStreamSynchronize(st);
            release_pages(kv, len0);
            return missed ? anpd_prefill(m, kv, tokens, n_tokens, out_next, out_logits, workspace, workspace_bytes, stream) : rc;
        }
        *out_next = m->pin[33];
        return ANPD_OK;
    }

    if (m->cfg.d_model > 8192) return fail(ANPD_E_UNIMPLEMENTED, "anpd_prefill: d_model above 8192 is not supported in one pass");
    const PrefillLayout PL = make_prefill_layout(m->cfg, n_tokens);
    if (!workspace || ((uintptr_t)workspace & 255) != 0) return fail(ANPD_E_INVAL, "anpd_prefill: workspace must be a 256-byte aligned device buffer");
    if (workspace_bytes < PL.total)
        return fail(ANPD_E_CAPACITY, "anpd_prefill: workspace has %zu bytes, %zu needed", workspace_bytes, PL.total);
    int32_t rc = ensure_pages(kv, kv->len + n_tokens, st);
    if (rc != ANPD_OK) return rc;
    char *pws = (char *)workspace;
    HIP_TRY(hipMemcpyAsync(pws + PL.tok, tokens, sizeof(int32_t) * (size_t)n_tokens, hipMemcpyHostToDevice, st));
    LogitsTo logits = {out_logits, V, nullptr};
    rc = run_prefill_mfma(m, kv, n_tokens, pws, PL, logits, st);
    if (rc != ANPD_OK) return rc;
    const int32_t *res = m->pin + 32;
    if (logits.elsewhere())
        HIP_TRY(hipMemcpyAsync(out_logits, logits.at, V * sizeof(float), hipMemcpyDeviceToDevice, st));
    HIP_TRY(hipStreamSynchronize(st));
    collect_marks(m);
    *out_next = res[1];
    kv->len += n_tokens;
    return ANPD_OK;
}

size_t anpd_linear_workspace_bytes(int32_t M, int32_t K)
{
    if (M < 1 || M > ANPD_MAX_WINDOW || K < 8) return 0;
    return align_up((size_t)((K + 31) / 32) * 4 * 1024);
}

size_t anpd_packed_bytes(int32_t N, int32_t K)
{
    if (N < 16 || N % 16 != 0 || K < 8 || K % 8 != 0) return 0;
    return packed_bytes((size_t)N / 16, K);
}

int32_t anpd_pack_weights(const void *W, int32_t N, int32_t K, void *packed, size_t packed_bytes_given, void *stream)
{
    if (!W || !packed) return fail(ANPD_E_INVAL, "anpd_pack_weights: NULL argument");
    size_t need = anpd_packed_bytes(N, K);
    if (need == 0) return fail(ANPD_E_INVAL, "anpd_pack_weights: need N %% 16 == 0 and K %% 8 == 0");
    if (packed_bytes_given < need) return fail(ANPD_E_CAPACITY, "anpd_pack_weights: buffer has %zu bytes, %zu needed", packed_bytes_given, need);
    return launch_pack(W, nullptr, nullptr, packed, PACK_PLAIN, N / 16, K, 0, 0, 0, (hipStream_t)stream);
}

int32_t anpd_linear(const float *X, const void *W, float *Y, int32_t M, int32_t N, int32_t K, int32_t dtype,
                    int32_t path, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!X || !W || !Y) return fail(ANPD_E_INVAL, "anpd_linear: NULL argument");
    if (M < 1 || M > ANPD_MAX_WINDOW || K < 8 || K % 8 != 0 || N < 16 || N % 16 != 0)
        return fail(ANPD_E_INVAL, "anpd_linear: need 1 <= M <= %d, K %% 8 == 0, N %% 16 == 0", ANPD_MAX_WINDOW);
    if (dtype != ANPD_F32 && dtype != ANPD_BF16) return fail(ANPD_E_INVAL, "anpd_linear: unknown dtype");
    hipStream_t st = (hipStream_t)stream;
    if (path == ANPD_GEMM_DOT) {
        GenArgs g;
        std::memset(&g, 0, sizeof(g));
        g.X = X;
        g.M = M;
        g.K = K;
        g.W0 = W;
        g.Y = Y;
        g.ldy = N;
        int dev = 0, n_cu = 256;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) (void)hipGetLastError();
        return dtype == ANPD_BF16 ? launch_gen_few<bf16_t, GEN_PLAIN>(g, N / 16, n_cu, st) : launch_gen<float, GEN_PLAIN>(g, N / 16, st);
    }
    if (path != ANPD_GEMM_MFMA && path != ANPD_GEMM_MFMA_STREAM)
        return fail(ANPD_E_INVAL, "anpd_linear: unknown path %d", path);
    if (dtype != ANPD_BF16) return fail(ANPD_E_INVAL, "anpd_linear: the MFMA path needs bf16 weights");
    if (!workspace || workspace_bytes < anpd_linear_workspace_bytes(M, K))
        return fail(ANPD_E_CAPACITY, "anpd_linear: workspace too small");
    int n_cu = 256, dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0)
        n_cu = prop.multiProcessorCount;
    const int cls = window_class(M);
    launch_split(X, (bf16_t *)workspace, M, K, cls, st);
    FastArgs a;
    std::memset(&a, 0, sizeof(a));
    a.Wp = (const uint4 *)W;
    a.Xp = (const uint4 *)workspace;
    a.nks = (K + 31) / 32;
    a.n_tiles = N / 16;
    a.M = M;
    a.cls = cls;
    a.Y = Y;
    a.ldy = N;
    return launch_fast<EPI_PLAIN>(a, n_cu, path == ANPD_GEMM_MFMA_STREAM, st);
}

}  // extern "C"

// ---- anpd_linear without a workspace argument and without any allocation ---------------------
//
// The split form of X lives in a file-scope device array.  Each device holds its own copy of the
// array at its own address, so the address is looked up once per device (with that device current)
// and kept; host code never uses the array's name for anything but that lookup.
namespace {

constexpr size_t kStaticScratchBytes = (size_t)(ANPD_LINEAR_STATIC_MAX_K / 32) * 4 * 1024;
constexpr int kMaxDevices = 64;

struct StaticScratch {
    void *ptr;
    int n_cu;
};
StaticScratch g_static_scratch[kMaxDevices];   // zero-initialised: ptr == nullptr means "not looked up yet"

}  // namespace

static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

extern "C" int32_t anpd_linear_static(const float *X, const void *W, float *Y, int32_t M, int32_t N, int32_t K, void *stream)
{
    if (!X || !W || !Y) return fail(ANPD_E_INVAL, "anpd_linear_static: NULL argument");
    if (M < 1 || M > ANPD_MAX_WINDOW || K < 8 || K % 8 != 0 || N < 16 || N % 16 != 0)
        return fail(ANPD_E_INVAL, "anpd_linear_static: need 1 <= M <= %d, K %% 8 == 0, N %% 16 == 0", ANPD_MAX_WINDOW);
    if (K > ANPD_LINEAR_STATIC_MAX_K)
        return fail(ANPD_E_CAPACITY, "anpd_linear_static: K = %d exceeds the built-in scratch (K <= %d); use anpd_linear with a workspace",
                    K, ANPD_LINEAR_STATIC_MAX_K);
    const size_t need = anpd_linear_workspace_bytes(M, K);
    if (need == 0 || need > kStaticScratchBytes) return fail(ANPD_E_CAPACITY, "anpd_linear_static: operand does not fit the built-in scratch");
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(ANPD_E_CAPACITY, "anpd_linear_static: device index %d not supported", dev);
    StaticScratch &sc = g_static_scratch[dev];
    if (!sc.ptr) {
        void *p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(ANPD_E_HIP, "anpd_linear_static: the scratch array has no address on device %d", dev);
        int n_cu = 0;
        HIP_TRY(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
        sc.n_cu = n_cu > 0 ? n_cu : 256;
        sc.ptr = p;
    }
    hipStream_t st = (hipStream_t)stream;
    const int cls = window_class(M);
    launch_split(X, (bf16_t *)sc.ptr, M, K, cls, st);
    FastArgs a;
    std::memset(&a, 0, sizeof(a));
    a.Wp = (const uint4 *)W;
    a.Xp = (const uint4 *)sc.ptr;
    a.nks = (K + 31) / 32;
    a.n_tiles = N / 16;
    a.M = M;
    a.cls = cls;
    a.Y = Y;
    a.ldy = N;
    return launch_fast<EPI_PLAIN>(a, sc.n_cu, false, st);
}
