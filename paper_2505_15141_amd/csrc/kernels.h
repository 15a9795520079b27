// Launchers of the forward-pass kernels (internal).
#pragma once
#include <hip/hip_ext.h>
#include "common.h"

namespace bs {

struct GemmArgs {
    const void* x;        // activations [M, K]: float, or bf16 hi plane (lo plane x_plane elements further)
    size_t x_plane;
    const void* w[3];     // up to three weight matrices stacked along N
    int seg_rows[2];      // rows of segment 0 and 1 (segment 2 takes the rest); N for a single matrix
    float* out;           // split-K partials [KS][M][ldo] float32 (slice stride ks_stride elements)
    size_t ks_stride;
    int M, N, K, ldo, KS;
    int tiled;            // weights are in the 64x32-block layout written by launch_pack_weights
    int stream;           // many-row GEMM: the model's weights are more than the memory-side cache holds (streams_past_cache)
    int x_tiled;          // many-row GEMM: R = many_tiled(M) if the planes of x are tiled (xt_index, x_plane = R K), else 0 (row-major)
};

// Fused projection for a handful of rows (see gemm_dec_kernel): tiled bf16 weights, activations as planes.
constexpr int DEC_MAX_ROWS = 2;
enum { EPI_RESID = 0, EPI_QKV = 1, EPI_SWIGLU = 2 };
struct DecArgs {
    const uint16_t* xh; size_t x_plane;       // input planes [M][K] (hi; lo x_plane elements further); gemm_rows: tiled (xt_index), x_plane = R K, R = rows_tiled(M)
    const void* w[3]; int seg_rows[2];        // tiled matrices stacked along N (QKV), or gate and up (SWIGLU)
    int M, N, K;                              // N: output columns (per matrix for SWIGLU)
    const float* ssq_in; int ssq_tiles; float eps;     // input rows' partial sums of squares [M][ssq_tiles] (QKV, SWIGLU)
    float* x; const float* gain_next; uint16_t* out_planes; size_t out_plane; float* ssq_out;   // RESID; out_planes also SWIGLU
    int out_tiled;                            // R = rows_tiled(M) (gemm_rows) or many_tiled(M) (gemm_big) if the output planes are tiled (xt_index; out_plane = R N), else 0
    const int32_t* pos; const float2* rope; int q_len, H, KVH, hd, cache_len;                    // QKV
    float* q_out; uint16_t* k_cache; uint16_t* v_cache;
    const float* att_part; int att_splits;    // RESID with the attention's per-split partials as input instead of planes (uses H, hd)
};
bool gemm_dec_fits(int M, int K);
int launch_gemm_dec(int epi, const DecArgs& a, hipStream_t s);
inline int many_tiled(int M) { return (M + 15) / 16 * 16; }    // rows of the tiled activation planes of the many-row projections
constexpr int ROWS_MAX = 32;                                 // rows the whole-K projections take
inline int rows_tiled(int M) { return M <= 16 ? 16 : 32; }   // rows of their tiled activation planes
// The same epilogues for up to ROWS_MAX rows of a wide model: one workgroup per compute unit owns several
// 16-column units over the whole K.  gemm_rows_units: units per workgroup at most (0: the kernel does not apply), *grid: workgroups.
int gemm_rows_units(int epi, int M, int N, int K, int* grid);
int launch_gemm_rows(int epi, const DecArgs& a, bool stream, hipStream_t s);
int launch_embed_dec(const int32_t* tok, const void* embed, const float* gain, int M, int d, float* x, void* planes,
                     size_t plane, float* ssq, hipStream_t s);

// One resident kernel for a whole forward pass over one or two rows of a small model (see step.hip).
constexpr int STEP_MAXL = 16;            // layers whose pointers travel as kernel arguments
struct StepArgs {
    const uint16_t* w[STEP_MAXL][7];     // tiled wq wk wv wo w_gate w_up w_down
    const float* an[STEP_MAXL];          // attention / feed-forward norm gains
    const float* fn[STEP_MAXL];
    const uint16_t* embed; const float* final_norm; const uint16_t* lm_head;
    int n_layers, d, H, KVH, hd, ff, V; float eps;
    int B, q_len, M, logit_rows;
    const int32_t* pos; const int32_t* tok; const float2* rope;      // written by the prep kernel
    char* kv; size_t kv_layer; int cache_len;
    void *X, *Q, *KVN, *PA, *ACT;        // exchange buffers of 8-byte cells {value, flag}: residual [copies][M][d], queries [M][nq],
                                         // new keys|values [M][2 nkv], attention partials [M][H][splits + 1][hd + 4] (the last slot:
                                         // the keys of the pass's own rows), SwiGLU output [M][ff]; every flag is zero when the
                                         // kernel starts (the prep kernel clears them)
    int32_t* status; int splits;
    float* logits; size_t logits_bstride;
    unsigned spin_limit;                 // polls of a cell before a workgroup gives up (status bit 16)
    int kp;                              // set by the launcher: padded row of the staged planes
};
bool step_fits(const bs_model_cfg& c, int B, int q_len, int n_layers);
// splits of the cached keys the resident step uses for B sequences and this cache length; 0: no room for the units
int step_splits(const bs_model_cfg& c, int B, int max_len);
// bytes of the exchange buffers X, Q, KVN, PA, ACT (each 256-byte aligned, in this order; off[i] = where buffer i starts)
size_t step_exchange_bytes(const bs_model_cfg& c, int M, int splits, size_t off[5]);
int step_grid();                         // workgroups of the resident kernel = compute units of the device
int device_cus();                        // the same; without a device (sizes asked for ahead) those of a whole one
int launch_step(const StepArgs& a, hipStream_t s);

int gemm_splits(int dtype, int N, int K, int M);
int profile_enable(int on);
int profile_collect(int mt_filter, double* total_ms, double* total_bytes, long long* launches);
// events of a launch that is timed (both null while the record is off), and the record of such a launch
int prof_events(hipStream_t s, hipEvent_t* e0, hipEvent_t* e1);
void prof_record(hipEvent_t e0, hipEvent_t e1, double bytes, int cls);
// A kernel launch that, while the measurement hook is on (e0 != nullptr), carries its own start and stop events: they
// take the dispatch's begin and end times, so the elapsed time is the kernel's and nothing else (two events recorded
// around a launch also measure 2-3 us of dispatch).
#define BS_LAUNCH_TIMED(kernel, grid, block, lds, stream, e0, e1, ...) \
    do { if (e0) hipExtLaunchKernelGGL(kernel, grid, block, (std::uint32_t)(lds), stream, e0, e1, 0, __VA_ARGS__); \
         else hipLaunchKernelGGL(kernel, grid, block, lds, stream, __VA_ARGS__); } while (0)
int launch_gemm(int dtype, GemmArgs a, hipStream_t s);
int launch_gemm_big(const GemmArgs& a, hipStream_t s);   // 33 rows and more, K % 32 == 0
// The many-row projections with their consumer's work behind them (gemm_big.hip): how the work items are cut (n_tiles: tiles
// of columns; EPI_RESID leaves 2 / wm sums of squares per row and tile), the bytes of partial sums that needs, and whether it is
// expected to beat launch_gemm with a consumer kernel.
// epi: EPI_QKV, N = stacked columns; EPI_SWIGLU, N = columns of one matrix; EPI_RESID.  plain_ks: the ranges of K launch_gemm takes if not fused.
struct BigPlan { int nt, mt, wm, n_mb, full, rem, ks, n_tiles, plain_ks; size_t part_bytes; bool once, fused; };
// How launch_gemm_big cuts the output: n_tiles x n_mb tiles of `cols` columns and 16 mt rows, eight wavefronts as 8 / wm columns x wm rows.
struct BigTiles { int wm, mt, n_mb, cols, n_tiles; };
BigTiles big_tiles(int N, int K, int M, int ks, bool stream);
int big_splits(int N, int K, int M);                     // ranges of K it is given
bool big_fused_applies(int epi, int N, int K, int M);
BigPlan big_plan(int epi, int N, int K, int M, bool stream, bool tiled);
int launch_gemm_big_fused(int epi, const GemmArgs& g, const DecArgs& e, const BigPlan& p, float* part,     // p = big_plan of the same sizes
                          size_t part_bytes, hipStream_t s);
size_t packed_elems(int N, int K);                       // elements of the tiled copy of an [N][K] matrix
int launch_pack_weights(const void* src, void* dst, int N, int K, hipStream_t s);

// ap.parts != nullptr: also into how many parts the attention cuts the keys of every sequence, `few` or, of one much longer than the
// others, up to `most`, and the work items of one kv head, (sequence | part << 16 | parts << 24) << 32 | first position (32 bits), -1 behind them
struct AttnParts { int32_t* parts; long long* items; int few, most, n_items, kv_heads, cus; };
// clear_bytes > 0: also zeroes that many bytes at `clear` (a multiple of 16, 16-byte aligned): the exchange cells of the
// resident step kernel that follows
int launch_prep(const int32_t* q_tokens, int q_stride, const int32_t* kv_len, int kv_base, int B, int q_len,
                int max_len, int V, int hd, float rope_base, int32_t* pos, int32_t* tok, float2* rope,
                int32_t* status, void* clear, size_t clear_bytes, const AttnParts& ap, hipStream_t s);
int launch_embed(int dtype, const int32_t* tok, const void* embed, int M, int d, float* x, hipStream_t s);
int launch_rmsnorm(int dtype, float* x, const float* pend, int pend_ks, size_t pend_stride, const float* gain, int d,
                   float eps, int n_seq, int rows_in, int rows_out, size_t plane, void* out, int tiled, hipStream_t s);
// bf16 models: residual completion + planes of gain .* x + per-chunk sums of squares [rows][norm_chunks(d)]; the
// consumers below apply the rows' RMS scale when given such sums (ssq != nullptr), ssq_n of them per row: other writers of x
// leave another number
int norm_chunks(int d);
// tiled = R > 0 (here, above and below): planes in the layout of xt_index, [d/32][R][32], plane = R*d elements
int launch_resid_sum(float* x, const float* pend, int pend_ks, size_t pend_stride, const float* gain, int d, int rows,
                     size_t plane, void* out, float* ssq, int tiled, hipStream_t s);
int launch_swiglu(int dtype, const float* part, int ks, size_t ks_stride, int M, int ff, size_t plane, void* out, int tiled,
                  const float* ssq, int ssq_n, int d, float eps, hipStream_t s);
// fp32 projections with the work around them (f32_fused_kernel), for the layers of passes where f32_fused_applies, and for the LM head of those where
// f32_head_applies (M: logit rows)
enum { F32_QKV, F32_SWIGLU, F32_RESID, F32_HEAD };
struct F32Args {
    const float* x; const int32_t* tok;       // input rows [.][K]: row m, or where tok is given (QKV) row tok[m] of the embedding
    const float* gain; float eps;             // RMSNorm of the input rows (not RESID)
    const float* w[3];                        // [N][K]; QKV: q, k, v; SWIGLU: gate, up
    float* out;                               // QKV: q [M][nq]; SWIGLU: [M][N]; RESID: x [M][N], added to (tok: to rows tok[m] of x_old); HEAD: row stride ldo
    const float* x_old;
    int M, N, K, ldo, rows_in, rows_out;      // HEAD: the last rows_out of every rows_in input rows
    const int32_t* pos; const float2* rope; int q_len, nq, nkv, hd, cache_len;      // QKV
    float* k_cache; float* v_cache;
};
bool f32_fused_applies(int M, int d, int ff, int nqkv, int nq);
bool f32_head_applies(int M, int vocab, int d);
int launch_f32_fused(int epi, const F32Args& a, hipStream_t s);
int launch_rope_kv(int dtype, const float* part, int ks, size_t ks_stride, const int32_t* pos, const float2* rope, int M,
                   int q_len, int H, int KVH, int hd, int max_len, float* q_out, void* k_cache, void* v_cache,
                   const float* ssq, int ssq_n, int d, float eps, hipStream_t s);
// out == nullptr: the splits are left un-merged in `part` (the consumer combines them)
// Exchange cells for combining the key splits inside the attention kernel (at most 16 query rows per head group, all
// workgroups resident together; otherwise a merge kernel runs): zero when the pass starts, one flag per layer.
struct AttnCells { void* buf; size_t bytes; unsigned flag, spin_limit; int32_t* status; };
size_t attn_cells_bytes(int rows, int H, int hd, int n_splits);
// prompt chunks (attn_prompt.hip): whole output, planes row-major or tiled (rows of the planes, xt_index)
bool attn_prompt_applies(int B, int q_len, int H, int KVH, int hd);
int launch_attn_prompt(const float* q, const uint16_t* k_cache, const uint16_t* v_cache, const int32_t* pos, int B, int q_len, int H, int KVH,
                       int hd, int cache_len, uint16_t* out, size_t plane, int tiled, hipStream_t s);
// key splits that a launch with `out` uses over a cache of cache_len rows when it may use up to n_splits: `splits`, or where `most` is
// more a count for every sequence between the two (AttnParts); and whether its workgroups combine them themselves (AttnCells)
// if the caller has cells.  `part` holds `most` partials a row.
constexpr int ATTN_CELL_ROWS = 16;
struct AttnPlan { int splits, most, n_items; bool in_kernel; };
AttnPlan attn_plan(int dtype, int B, int q_len, int H, int KVH, int hd, int cache_len, int n_splits);
int launch_attention(int dtype, const float* q, const void* k_cache, const void* v_cache, const int32_t* pos, int B,
                     int q_len, int H, int KVH, int hd, int max_len, int n_splits, float* part, size_t plane, void* out, int out_tiled, const AttnCells* cells,
                     const AttnParts* ap, bool stream, hipStream_t s);

}  // namespace bs
