// Internal launch interface between the host API and the gfx950 kernels.
// Not part of the public ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>
#include <stdint.h>
#include <atomic>
#include "attn_plan.h"
#include "../../include/confspec.h"

// The slices of the workspace that only passes over few rows use (confspec_api.hip), for checks of the layout on the host:
// their number (0: such a pass takes the general kernels), the end of what they share with the other passes, the total.
extern "C" __attribute__((visibility("hidden"))) int confspec_few_row_slices(const confspec_ctx *ctx, int32_t T, int32_t B,
    const confspec_batch *exact, size_t *h_offsets /*[16]*/, size_t *h_bytes, size_t *from, size_t *total);

namespace cs {

typedef __hip_bfloat16 bf16;

// fp32 -> IEEE half, round to nearest even, saturating: a finite value beyond the half range becomes +-65504 rather
// than an infinity (one infinity in an activation would turn the residual stream, and with it the confidence, into
// NaN).  Every store of the fp16 activation format goes through this.
__device__ __forceinline__ __half to_half_sat(float v) {
    return __float2half_rn(__builtin_amdgcn_fmed3f(v, -65504.0f, 65504.0f));
}

// Launch-shape settings of one context (confspec_tune); the kernels' launchers and the planners take them as an
// argument, nothing here is process-wide.
struct GemmTune {
    int tile = 0;      // 0 = heuristic; 1 = 128x128, 4 = 256x256 / 8 wavefronts, 7 = 192x96 / 6 wavefronts
    int group_m = 0;   // 0 = heuristic; otherwise tile rows per band of the tile order
    int splitk = 0;    // 0 = heuristic; otherwise the split-K factor of every GEMM that has scratch (1 = never split)
    int short_tile = 1;   // 1 = products of at most 32 rows use 32 x 128 tiles with four LDS stages
};
// hipFuncSetAttribute(MaxDynamicSharedMemorySize) once per device and kernel: `mask` holds one bit per device.
inline hipError_t set_dynamic_lds_once(std::atomic<uint32_t> &mask, const void *fn, int bytes) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint32_t bit = 1u << (dev & 31);
    if (mask.load(std::memory_order_acquire) & bit) return hipSuccess;
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
    mask.fetch_or(bit, std::memory_order_release);
    return hipSuccess;
}

// Activations of a pass over few rows are kept in fragment order: element (row, k) of a matrix of width K (K % 32 == 0).  The 16 rows x 32 k
// of one 16x16x32 MFMA operand are 1 KiB in lane order: [k / 8 % 4][row % 16][k % 8].  Rows are padded to a multiple of 16.
__host__ __device__ inline size_t frag_index(int row, int k, int K) {
    return ((size_t)(row >> 4) * (K >> 5) + (k >> 5)) * 512 + ((k & 31) >> 3) * 128 + (row & 15) * 8 + (k & 7);
}

// ---- attention work description and planner arithmetic: attn_plan.h ----

enum Epilogue : int { EPI_STORE_F32 = 0, EPI_RESID_F32 = 1, EPI_SWIGLU = 2, EPI_ROPE = 3 };

// EPI_ROPE (bf16 model, head_dim 128): the GEMM is the QKV projection with the rows of every head of W
// reordered [0..31, 64..95, 32..63, 96..127], so that a wavefront's 64 output columns hold 32 rotation pairs
// (i, i + 64).  The epilogue rotates q and k heads by the token's position and writes q, k and v in the natural
// head layout, in bf16; the *_lo buffers (all or none) receive bf16(value - bf16(value)).
struct RopeArgs {
    const float *cos_t, *sin_t;   // [M, 64]
    void *q, *k, *v;              // [M, Hq, 128], [M, Hkv, 128], [M, Hkv, 128]
    void *q_lo, *k_lo, *v_lo;
    int32_t Hq, Hkv;
};

// Work of the few-row attention (attn_few.hip).
// One tile of query rows: rows row0 .. of context unit (traces from b0; first packed suffix token cu0, n_rows = G * suffix
// tokens, context length L); its rows see suffix tokens k_start .. k_start + n_keys - 1 at most.  n_rows == 0: unused.
struct FewTile {
    int32_t b0, cu0, row0, n_rows, L, k_start, n_keys, pad;
};

// ---- small kernels (templated on storage type: float or bf16) ----
// What a pass needs to know about its tokens, in one launch: trace and position of every token, the last row of every
// trace, and where asked for (pointers not null) the rotary tables [T, hd / 2] and the fp32 embedding rows x [T, d].
struct FrontArgs {
    const int32_t *cu, *plens;
    int32_t B, T, max_L;
    int32_t *tok_trace, *tok_pos, *last_row;
    float *cos_t, *sin_t;
    int32_t half_hd;
    float theta;
    const int32_t *ids;
    const void *E;
    float *x;
    int32_t d, vocab;
    // passes over few rows (null otherwise): control block to clear (n_ctl ints); operand, power of two and sums of
    // squares of the first projection as SkinnyGemm has them (gain g, 16-bit storage)
    int32_t *ctl;
    int32_t n_ctl;
    const void *g;
    void *xg;
    float *ssq, *sc;
    int32_t ssq_n, xg_fmt;
    float eps;
    // write-back (n_append not null): token row of the cache each token goes to, or -1
    const int32_t *table, *n_append;
    int32_t max_blocks, n_blocks, block_size;
    int32_t *kv_row;
    // tiles of few_rows query rows (few_tiles not null; at most 128 units): G rows per token; group_start as in attn_plan.h
    FewTile *few_tiles;
    const int32_t *group_start;
    int32_t n_units, n_few_tiles, few_rows, G;
};
hipError_t launch_front(int dtype, const FrontArgs &a, hipStream_t s);
// x fp32 [T,d] -> out (storage dtype) [T, d]; terms == 2 (bf16 only): [T, 2d] hi | lo two-term form;
// terms == 3 (bf16 only): IEEE half values
hipError_t launch_rmsnorm(int dtype, const float *x, const void *g, void *out, int T, int d, float eps,
                          int terms, hipStream_t s);
// qkv fp32 [T, (Hq+2Hkv) hd] -> q [T,Hq,hd], ksuf [T,Hkv,hd], vsuf [T,Hkv,hd] (storage dtype), q and k rotated
// q_lo / k_lo / v_lo (bf16 only, all or none): receive bf16(value - bf16(value))
hipError_t launch_rope_split(int dtype, const float *qkv, const float *cos_t, const float *sin_t, void *q,
                             void *ksuf, void *vsuf, void *q_lo, void *k_lo, void *v_lo, int T, int Hq, int Hkv,
                             int hd, hipStream_t s);
// dst row b = src row rows[b] (rows == nullptr: row b), row_bytes a multiple of 16
hipError_t launch_gather_rows(const void *src, void *dst, const int32_t *rows, int n_rows, int n_src_rows,
                              size_t row_bytes, hipStream_t s);
hipError_t launch_bf16_to_f16(const void *src, void *dst, size_t n, hipStream_t s);
// dst rows = src rows with the two middle 32-row blocks of every 128-row head swapped (n_heads * 128 rows of d elements)
hipError_t launch_permute_heads(const void *src, void *dst, int n_heads, int d, hipStream_t s);
hipError_t launch_pack_gate_up(int dtype, const void *src, void *dst, int F, int d, hipStream_t s);

struct VerdictArgs {
    int32_t ids[8];
    float tau[8];
    int32_t n_verdict, n_tau;
};
// last_row == nullptr: trace b reads row b of x
hipError_t launch_verdict(int dtype, const float *x, const int32_t *last_row, const void *final_norm,
                          const void *lm_head, VerdictArgs va, int B, int T, int d, float eps, float *logits,
                          float *conf, int32_t *verdict, uint8_t *accept, hipStream_t s);

// Arg max / max / log-sum-exp of every row of logits [B, V]; conf_full (may be null) from verdict_logits [B, n_verdict].
hipError_t launch_head_reduce(const float *logits, int B, int V, const float *verdict_logits, int n_verdict, int32_t *token,
                              float *max_logit, float *lse, float *conf_full, hipStream_t s);

// ---- GEMM: C[M,N] = A[M,K] . W[N,K]^T with an epilogue ----
//  EPI_STORE_F32: out fp32 [M,N]
//  EPI_RESID_F32: out fp32 [M,N] += result (in place)
//  EPI_SWIGLU   : W rows are gate/up interleaved in groups of 32; out (storage dtype) [M, N/2]
// fp32 storage.  g (not null: store, SwiGLU, rotating epilogue): A holds rows x of the residual stream and the operand is
// RMSNorm(x) * g.  EPI_ROPE: rope (float pointers, no second terms) and hd, W rows in their natural order.
struct GemmF32 {
    const float *A, *W;
    float *out;
    int32_t M, N, K;
    const float *g;
    float eps;
    RopeArgs rope;
    int32_t hd;
};
hipError_t launch_gemm_f32(const GemmF32 &p, int epi, hipStream_t s);
// Activation formats (a_terms / out_terms): 1 = bf16; 2 = two bf16 terms, A is [M, 2K] = hi | lo and a
// SwiGLU result is written as [M, 2 * N/2] = hi | lo; 3 = fp16 (A and W hold IEEE half values, a SwiGLU
// result is written as fp16).
// splitk_ws (may be null): scratch for the split-K path that outputs with too few 128 x 128 tiles to fill the
// chip, and long k ranges over few 256 x 256 tiles, take (gemm_splitk_factor > 1); it needs
// gemm_splitk_bytes(M, N, K * a_terms) bytes, otherwise the call falls back to one workgroup per tile.
// pf (may be null; used by the SwiGLU epilogue's wide kernel only): memory the kernel reads once, front to back,
// while it works, so that it sits in the last-level cache for the kernel that follows; n16 = 16-byte vectors.
struct PrefetchArgs {
    const void *ptr = nullptr;
    unsigned n16 = 0;
};
// norm (may be null; residual epilogue only): the RMSNorm that follows the projection in the pass.  When the call takes
// the split-K path, the kernel that adds the slices to the residual stream also writes RMSNorm(updated row) * g to
// norm->h (format norm->terms) and *norm_done becomes true; otherwise the caller runs the RMSNorm kernel itself.
struct NormAfter {
    const void *g = nullptr;
    void *h = nullptr;
    float eps = 0.f;
    int terms = 1;
};
hipError_t launch_gemm_bf16(const GemmTune &tune, const bf16 *A, const bf16 *W, void *out, int M, int N, int K, int epi,
                            int a_terms, int out_terms, float *splitk_ws, size_t splitk_ws_bytes, hipStream_t s,
                            const PrefetchArgs *pf = nullptr, const NormAfter *norm = nullptr, bool *norm_done = nullptr);
hipError_t launch_gemm_bf16_rope(const GemmTune &tune, const bf16 *A, const bf16 *W_perm, int M, int N, int K, int a_terms,
                                 const RopeArgs &rope, float *splitk_ws, size_t splitk_ws_bytes, hipStream_t s);
// How a product of M rows runs.  feed: 0 gemm_bf16_kernel, else the tile of gemm_feed_kernel (1 = 64x64, 2 = 64x128, 3 = 128x128,
// 4 = 256x128, 5 = 256x192); splits: k slices; big: they are 256 x 256 tiles.
struct GemmPlan { int feed = 0, splits = 1; bool big = false; };
GemmPlan gemm_plan(const GemmTune &tune, int M, int N, int K_total, int epi, bool norm_after, bool can_split);
int gemm_band_rows(const GemmTune &tune, int BM, int BN, int smem, int tiles_m, int tiles_n);
int gemm_splitk_factor(const GemmTune &tune, int M, int N, int K_total);   // of a residual projection with a norm behind it
size_t gemm_splitk_bytes(const GemmTune &tune, int M, int N, int K_total);
size_t gemm_splitk_max_bytes(const GemmTune &tune, int max_M, int N, int K_total);   // at least gemm_splitk_bytes for every M <= max_M

// ---- attention ----
struct AttnArgs {
    const void *q;          // [T, Hq, hd]
    const void *ksuf;       // [T, Hkv, hd] suffix keys (rotated)
    const void *vsuf;       // [T, Hkv, hd]
    const void *q_lo;       // second bf16 terms of q / ksuf / vsuf (same layouts), or nullptr: when all
    const void *ksuf_lo;    // three are given the bf16 kernel runs its two-term variant (q, suffix k/v
    const void *vsuf_lo;    // and the probabilities each carried as hi + lo)
    const void *k_pages;    // this layer's pages [n_blocks, Hkv, bs, hd]
    const void *v_pages;
    const int32_t *block_table;  // [B, max_blocks]
    const int32_t *cu;           // [B+1]
    const int32_t *plens;        // [B]
    const int32_t *tok_trace;    // [T] trace of every packed suffix token (written by the prep kernel)
    void *out;              // [T, Hq*hd] in activation format out_terms: 1 storage dtype, 2 bf16 hi | lo
                            // ([T, 2*Hq*hd]), 3 IEEE half
    int32_t B, T, Hq, Hkv, hd, n_blocks, block_size, max_blocks;
    float scale;            // 1/sqrt(hd)
    int32_t out_terms;
    int32_t part_rows;      // rows of a partial result (AttnPlanCounts), a multiple of 32 up to ATTN_BM
};
hipError_t launch_attn_f32(const AttnArgs &a, int max_S, hipStream_t s);   // max_S: longest suffix of the batch

// group_start: null (every trace is its own context unit) or n_units + 1 trace indices, dev (attn_plan.h)
hipError_t launch_attn_plan(const int32_t *cu, const int32_t *plens, const int32_t *group_start, int n_units, int B,
                            int T, int max_L, int G, int Hkv, int chunks_per_item, int equalize, int last_only,
                            int max_tiles, int max_items, AttnTile *tiles, AttnItem *items,
                            int32_t *counts /*[11]: tiles, items, first item of XCD 0..8*/, hipStream_t s);
// The attention kernel over the planned items; pieces of split tiles leave fp32 partial results in part_o / part_ml
// ([slots, a.part_rows, hd] and [slots, a.part_rows, 2]).
// avg_chunks: average number of key chunks per item (chooses the main loop)
hipError_t launch_attn_bf16(const AttnTune &tune, const AttnArgs &a, const AttnItem *items, const int32_t *counts,
                            int n_items_host, int max_xcd_items, int avg_chunks, float *part_o, float *part_ml, hipStream_t s);
// Combines the partial results of every split tile in a fixed order and writes the output rows.
hipError_t launch_attn_merge(const AttnArgs &a, const AttnTile *tiles, const int32_t *counts, int n_tiles_host, int n_items_host,
                             const float *part_o, const float *part_ml, hipStream_t s);

// Suffix keys / values [T, Hkv, hd] of the tokens i < n_append[b] of every trace into rows L_b + i of the paged cache
// of one layer (k_pages / v_pages point at that layer).
hipError_t launch_kv_append(const void *ksuf, const void *vsuf, void *k_pages, void *v_pages, const int32_t *table,
                            const int32_t *cu, const int32_t *plens, const int32_t *n_append, const int32_t *tok_trace,
                            int B, int T, int Hkv, size_t head_row_bytes, int block_size, int max_blocks, int n_blocks,
                            hipStream_t s);

// ---- passes over few rows (skinny_bf16.hip) ----
constexpr int SK_MAX_ROWS = 128;          // suffix tokens of a pass that takes these projections
constexpr int SK_MAX_TILES_CUT = 256;     // workgroup tiles of a projection whose k range is cut (one arrival counter each)
enum SkinnyEpilogue : int { SK_EPI_ROPE = 0, SK_EPI_RESID = 1, SK_EPI_SWIGLU = 2 };
// One projection: out = X[M, K] . W[N, K]^T, M <= SK_MAX_ROWS, K % 64 == 0, then the epilogue.
struct SkinnyGemm {
    const bf16 *X;            // [M, K] in fragment order, bf16 or (f16) IEEE half
    const bf16 *W;            // [N, K], same element type
    int32_t M, K;
    int32_t n_ct;             // 16-column tiles of the accumulator: N / 16 (ROPE, RESID), N / 16 = F / 8 (SWIGLU)
    int32_t S, ms;            // k slices, blocks of rows (set by the launcher)
    float *planes;            // skinny_plane_bytes; null when that is 0
    int32_t *tile_cnt;        // SK_MAX_TILES_CUT arrival counters (zero before and after the launch)
    // ROPE, SWIGLU: X holds x * gain * sc; ssq_in [M, ssq_n] are partial sums of squares of the rows x of width d_norm, negative
    // where an element of X left the format's range; the result rows are scaled by 1 / sqrt(sum / d_norm + eps) / sc_in.  Rows
    // that X does not hold are taken from x [M, K] fp32 and the gains g_next.
    // RESID with xg_out: the same two of the rows before the update, which the new power of two is taken from.
    const float *ssq_in, *sc_in;
    int32_t ssq_n, d_norm;
    float eps;
    // RESID: x [M, N] fp32 += product.  With xg_out (may be null) it also writes the next projection's operand
    // x * g_next * sc in format xg_fmt (1 bf16, 3 half) [M, N] in fragment order, the powers of two sc_out [M], and
    // ssq_out [M, N / 16].
    float *x;
    void *xg_out;
    const bf16 *g_next;
    float *ssq_out, *sc_out;
    int32_t xg_fmt;
    // SWIGLU: W rows are gate / up interleaved in groups of 32; act [M, F] in fragment order, format act_fmt (1 or 3)
    void *act;
    int32_t act_fmt;
    // ROPE: the QKV projection, W rows of every head ordered [0..31 | 64..95 | 32..63 | 96..127].  With kv_row (may be
    // null) the key / value of row m also goes to token row kv_row[m] of this layer's pages where that is not negative.
    RopeArgs rope;
    const int32_t *kv_row;
    void *k_pages, *v_pages;
};
struct SkinnyPlan { int mb, ms, ct, S; };
SkinnyPlan skinny_plan(int epi, int M, int K, int n_ct);
bool skinny_has_kernel(int epi, const SkinnyPlan &p);
size_t skinny_plane_bytes(int epi, int M, int K, int n_ct);      // for up to M rows; 0 when no k range is cut
hipError_t launch_skinny(SkinnyGemm a, int epi, bool f16, hipStream_t s);
// control block (int32) of a pass over few rows: the arrival counters
constexpr int FEW_CTL_TILE = 0;                                   // + tile of a projection whose k range is cut
constexpr int FEW_CTL_ATTN = FEW_CTL_TILE + SK_MAX_TILES_CUT;     // + attention tile * Hkv + kv head
constexpr int FEW_MAX_TILES_KV = 4096;                            // attention tiles * kv heads
constexpr int FEW_MAX_G = 64;                                     // q heads per kv head of the few-row attention
constexpr int FEW_MAX_G_ONE = 16;                                 // ... of its form for one token per trace
constexpr int FEW_RECORDS = 256;                                  // partial results of the attention's pieces
constexpr int FEW_CTL_INTS = FEW_CTL_ATTN + FEW_MAX_TILES_KV;

// ---- generation steps: one new token per trace (decode_bf16.hip) ----
constexpr int DEC_MAX_ROWS = 32;     // traces the language-model head of these kernels takes
constexpr int DEC_MAX_KT = 24;       // k-tiles (of 64) of the head's rows

// Head over the whole vocabulary: X is [M, 2 K] two-term bf16 (hi | lo), W the [16 n_ct, K] head; every one of the nwg
// workgroups leaves (max, index of the first max, sum of exp(z - max)) of its columns per row in part [nwg, 32, 4] fp32.
struct DecHead {
    const bf16 *X, *W;
    int32_t M, K, n_ct, nwg;
    float *part;
};
hipError_t launch_dec_head(const DecHead &a, hipStream_t s);
// token / max logit / log-sum-exp (and conf_full, with verdict logits) of B rows from the nwg records per row
hipError_t launch_dec_head_final(const float *part, int nwg, int B, const float *verdict_logits, int n_verdict, int32_t *token,
                                 float *max_logit, float *lse, float *conf_full, hipStream_t s);

// ---- attention of passes over few rows (attn_few.hip) ----
struct FewAttn {
    const bf16 *q, *q_lo;             // [T, Hq, 128]; q_lo (may be null): second bf16 terms, then those of ksuf / vsuf too
    const bf16 *ksuf, *vsuf;          // [T, Hkv, 128]: keys / values of the suffix tokens
    const bf16 *ksuf_lo, *vsuf_lo;    // (may be null where every trace has one token: single terms)
    const bf16 *k_pages, *v_pages;    // this layer's pages [n_blocks, Hkv, 16, 128]
    const int32_t *table, *plens, *cu, *tok_trace;
    const FewTile *tiles;             // [n_tiles]; null: one suffix token per trace, tile = trace
    int32_t *arrived;                 // n_tiles * Hkv arrival counters, zero before and after
    void *out;                        // [T, Hq * 128] in fragment order, format out_fmt (1 bf16, 3 half)
    float *part_o, *part_ml;          // FEW_RECORDS of [rows, 128] and [rows, 2] fp32, rows = few_attn_rows
    int32_t B, T, Hq, Hkv, G, max_blocks, n_blocks, max_L, out_fmt, n_tiles;
    int32_t pieces, wave_pages, fold, inv_G;     // set by the launcher
    float scale_log2;                 // log2(e) / sqrt(head_dim)
};
// What launch_few_attn takes: query heads per kv head and attention tiles (one: one suffix token per trace).
inline bool few_attn_takes(int64_t n_tiles, int Hkv, int G, int T, bool one) {
    return n_tiles >= 1 && Hkv >= 1 && n_tiles * Hkv <= FEW_MAX_TILES_KV && G >= 1 && G <= (one ? FEW_MAX_G_ONE : FEW_MAX_G) && T <= SK_MAX_ROWS;
}
// Tiles of a batch (host copies; one: one suffix token per trace), rows of a tile.
int64_t few_attn_tiles(const int32_t *h_cu, int B, const int32_t *h_group_start, int n_units, int G, bool one);
int few_attn_rows(bool one);
void few_attn_pieces(FewAttn &a, bool one);      // from n_tiles, Hkv and max_L: pieces, wave_pages, fold
hipError_t launch_few_attn(FewAttn a, hipStream_t s);

// ---- cascade (cascade.hip) ----
hipError_t launch_cascade_select(const uint8_t *keep, const int32_t *verdict_d, const int32_t *req_start, const int32_t *parent,
                                 int R, int B, const int32_t *cu, const int32_t *plens, int T, uint8_t *open_flag,
                                 uint8_t *target_ran, int32_t *pos_of, int32_t *sel_idx, int32_t *cu_out, int32_t *plens_out,
                                 int32_t *n_out, hipStream_t s);
hipError_t launch_cascade_gather(const int32_t *pos_of, const int32_t *cu, const int32_t *cu_out, const int32_t *ids,
                                 int32_t *ids_out, const int32_t *table, int32_t *table_out, int max_blocks, int B, int T,
                                 hipStream_t s);
hipError_t launch_cascade_merge(const uint8_t *keep, const int32_t *verdict_d, const float *conf_d, const int32_t *pos_of,
                                const float *conf_t_c, const int32_t *verdict_t_c, const int32_t *req_start,
                                const int32_t *parent, int R, int B, int n_target, float *conf_t, int32_t *verdict_t,
                                int32_t *decision, uint8_t *escalated, uint8_t *selected, float *conf_used, int32_t *accepted,
                                hipStream_t s);

}  // namespace cs
