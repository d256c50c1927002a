// Host-side launchers of the stage kernels.  Every launcher only enqueues on `s`.
// Shapes are validated by the caller (stage.cpp) before any launch.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "common.h"

// Row bookkeeping of one call: token row i belongs to sequence row_seq[i] at absolute
// position row_pos[i] (device int32 arrays).  For decode they are derived on the device from the
// cache's committed lengths, so one step needs no host->device traffic.
struct RowMap {
    const int32_t *row_seq;   // [T]
    const int32_t *row_pos;   // [T]
};

// Blocks that the decode attention cuts a context into at most: what its merge holds in registers, what the workspaces have
// room for, and what the rule and the hook that choose the number may ask for.
constexpr int kAttnMaxSplit = 8;

// KV cache geometry of one (layer, sequence, kv head) slab; see kernels_bf16_attn.hip
struct KvGeom {
    int d;            // head dim (64 | 128)
    int hkv_l;        // local kv heads
    int smax;         // positions per sequence, multiple of 32
    int64_t seq_stride;   // elements between sequences  (= hkv_l * smax * d)
};

// ---- layout / utility (kernels_layout.hip) -------------------------------------------------
// Weights are packed k-tile-major: tile (kt, nt) of a matrix with dst_n_tiles feature tiles sits at
// ((kt * dst_n_tiles + nt) * 64 + lane) * 8 elements.  All blocks of a projection walk kt together, so at
// any moment the chip streams one contiguous window of HBM instead of hundreds of scattered slabs.
// dst tile (dst_tile0 + nt * dst_tile_stride) <- src[k0 + k][c0 + nt*16 + i], src row-major with
// leading dimension ld (elements), K % 32 == 0, N % 16 == 0.
// rope_d > 0 (fused QKV weight): columns are heads of width rope_d; each 16-row tile of a head holds 8
// rotary pairs (rows 0-7 = head columns 8*tl .. 8*tl+7, rows 8-15 = those + rope_d/2), so one MFMA tile is
// self-contained for RoPE.  The QKV projection output is in this permuted column order.
void launch_pack_weight(const h16_t *src, int64_t ld, int k0, int c0, int K, int N, h16_t *dst,
                        int dst_tile0, int dst_tile_stride, int dst_n_tiles, int rope_d, hipStream_t s);
void launch_accumulate_f32(float *dst, const float *src, int64_t n, hipStream_t s);
void launch_advance_lens(int32_t *lens, int b, hipStream_t s);

// plain streaming kernels of known size (HBM calibration for the benchmarks and profiler counters)
void launch_stream_copy(const void *src, void *dst, int64_t bytes, int blocks, hipStream_t s);
void launch_stream_read(const void *src, float *sink, int64_t bytes, int blocks, hipStream_t s);
// register-resident MFMA loops: 4 waves per block, per wave and iteration 2^20 flop (one 128 x 128 x 32 k-step)
void launch_mfma_probe(int variant, float *sink, int iters, int blocks, hipStream_t s);

// ---- 16-bit path (kernels_bf16_*.hip, compiled once per element type: namespaces bf16 and f16) --------------------

// ---- decode projections with fused epilogues (kernels_bf16_decode.hip) ---------------------------
enum { DEC_RAW = 0, DEC_QKV = 1, DEC_RESID = 2, DEC_SWIGLU = 3, DEC_BEST = 4 };
#define DEC_SCRATCH_RSTD 64    // floats at the end of the split projections' scratch: the rows' 1 / rms
struct DecodeEpi {
    int mode;                  // DEC_*
    // RMSNorm statistics of the rows feeding this projection: sums of squares per token and 16-column unit,
    // [token][units] (a wave adds a token's up from contiguous loads); NULL when the input is not a normalised
    // residual stream (W_O, W2)
    const float *ssq_in;
    int ssq_units, norm_dim;
    float eps;
    float *raw_out;            // RAW: [T][N] fp32
    // BEST (decode only): per row and unit of columns (decode_best_units) the largest of the first `valid` columns' values and
    // its index, lowest index on ties; -infinity and 0x7fffffff where there is none
    float *best_val;
    int32_t *best_id;
    int valid;
    // QKV
    int hq_l;
    KvGeom kg;
    const int32_t *row_pos;
    const float *cos_tab, *sin_tab;
    h16_t *q_hi, *q_lo, *kc, *vc;
    // RESID
    float *h;                  // residual stream [T][N] fp32, updated in place
    const float *g_next;       // gain of the next RMSNorm
    h16_t *hg;                // (h * g_next) as hi/lo decode operand (dec_act_offset)
    float *ssq_out;            // [token][N / 16]
    int last_layer;            // 1: write out_partial / out_resid (bf16 [T][N]) instead of updating h
    h16_t *out_partial, *out_resid;
    // SWIGLU
    h16_t *u;                 // hi/lo decode operand [T][F_l]
    int F_l;
};
// What the decode attention needs to finish a QKV projection whose contraction was split over blocks: it adds up the
// partial sums of its own heads, applies 1/rms and the rotary embedding, appends the new K / V row to the cache and
// goes on with q in registers -- the projection then needs no finishing launch (launch_decode_qkv, launch_attn_decode).
struct QkvTail {
    const float *part;         // [splits][T][N] partial sums; NULL: q and the cache rows are complete already
    int splits, T, N;
    const float *rstd;         // [T] 1/rms of the rows, left by the split kernel (decode kernels' layouts) ...
    const float *cos_tab, *sin_tab;
    const float *ssq;          // ... or [norm_dim / 128][T] the rows' sums of squares (prefill kernels' layouts)
    int norm_dim;
    float eps;
};
// ---- prefill projections with fused epilogues (kernels_bf16_gemm.hip) ----------------------------
// Same epilogue roles as in decode (DEC_* modes), on packed operands: the input Xp is (h * gain) in
// fragment tiles, RMSNorm enters as the per-token scale rstd derived from `ssq_in`.
#define GEMM_SSQ_COLS 128      // features per sum-of-squares partial: ssq[H / 128][T]
struct GemmEpi {
    int mode;                  // DEC_RAW | DEC_QKV | DEC_RESID | DEC_SWIGLU
    const float *ssq_in;       // [norm_dim / 128][T] sums of squares of the input rows, NULL = not normalised
    int norm_dim;
    float eps;
    float *raw_out;            // RAW: [T][N] fp32
    // QKV
    int hq_l;
    KvGeom kg;
    RowMap rm;
    const float *cos_tab, *sin_tab;
    h16_t *q, *kc, *vc;       // q: fragment tiles [T/16][hq_l * d / 32]
    // RESID
    float *h;                  // residual stream, fp32, 32 x 32 tiled (h_tile_offset), updated in place
    const float *g_next;
    h16_t *hg;                // (h * g_next) in fragment tiles [T/16][N/32]
    float *ssq_out;            // [N / 128][T]
    int last_layer;
    h16_t *out_partial, *out_resid;
    // SWIGLU
    h16_t *u;                 // fragment tiles [T/16][F_l/32]
    int F_l;
    // counters of the skinny kernel, one per 128 features, even between launches: blocks of a contraction in two splits that have arrived,
    // the second of which finishes the tile.  NULL: a launch of its own does
    unsigned *arrived;
};
// per row of logits [n][ld]: the largest of the first `valid` entries and its index + id0 (lowest index wins ties)
void launch_row_argmax(const float *logits, int64_t ld, int valid, int n, int id0, int32_t *token_out, float *logit_out,
                       hipStream_t s);
// the same over per-unit candidates val / id [n][units] (DEC_BEST)
void launch_row_best(const float *val, const int32_t *id, int units, int n, int id0, int32_t *token_out, float *logit_out,
                     hipStream_t s);
// rows_out[i] = table[clamp(tokens[i], 0, vocab - 1)], rows of row_bytes bytes (a multiple of 4)
void launch_embed_rows(const void *table, int64_t row_bytes, int vocab, const int32_t *tokens, int n, void *rows_out,
                       hipStream_t s);

// p[0 .. bytes) = 0 with a kernel; p 4-byte aligned, bytes a multiple of 4
void launch_fill_zero(void *p, size_t bytes, hipStream_t s);


// ---- fp32 path (kernels_f32.hip): plain row-major layouts, fp32 matrix instructions -------------------------------
// One projection out = f(x) . w.  F32_PLAIN: out[T][cols] = the product; F32_RESID: resid + product -> resid_out, or, with
// resid_out == NULL (the stage's last projection), the product -> out and resid -> out_resid (may be NULL); F32_SWIGLU:
// w holds `cols` gate columns, then `cols` up columns, out = silu(gate) * up.  Rows of `out`, `resid`, ... are `cols` wide.
enum { F32_PLAIN = 0, F32_RESID = 1, F32_SWIGLU = 2 };
struct F32Proj {
    const float *x, *x2;       // [T][K]; x2 (may be NULL, only with F32_PLAIN, g and T <= 32) is added to x
    const float *g;            // RMSNorm gain [K]: x is normalised first; NULL = as it is
    const float *w;            // [Kp][N], rows K .. Kp - 1 zero
    int T, K, Kp, N, cols;     // K a multiple of 4, Kp of 32, cols of 16
    float eps;
    float *out;
    const float *resid;
    float *resid_out, *out_resid;
    int32_t *lens;             // not NULL (T <= 32 only): lens[0 .. T) += 1 once every earlier launch is through
};
// n_buf [T][K] (normalised rows) and part (partial sums, kF32PartFloats or NULL: no tile is cut) are needed for T > 32 only.
// Each of 256 blocks has at most two pieces of a 64 x 128 tile to leave there, whatever the shape: 16 MB
constexpr size_t kF32PartFloats = (size_t)2 * 256 * 64 * 128;
void f32_launch_proj(int mode, const F32Proj &p, float *n_buf, float *part, hipStream_t s);
void f32_launch_rope_append(const float *qkv, int T, int hq_l, int hkv_l, int d, int smax, RowMap rm,
                            const float *cos_tab, const float *sin_tab, float *q_out, float *kc, float *vc,
                            hipStream_t s);
// causal attention of packed new rows whose keys and values are in the cache already; items as in launch_attn_prefill
void f32_launch_attn_prefill(const float *q, float *kc, float *vc, int hq_l, int hkv_l, int d, int smax, const int32_t *pos0,
                             const int32_t *cu_rows, const int32_t *items, int n_items, float *o, hipStream_t s);
// one new row per sequence at pos[seq]: rotary embedding and cache append of the raw projection qkv, then the attention
void f32_launch_attn_decode(const float *qkv, float *kc, float *vc, int b, int hq_l, int hkv_l, int d, int smax, const int32_t *pos,
                            const float *cos_tab, const float *sin_tab, float *o, hipStream_t s);
// The same and the W_O projection behind it (p: F32_RESID with resid_out, p.x not read) in one launch, where f32_attn_wo_fits: T rows of `cols`
// columns, the longest context `positions`, the new one included
bool f32_attn_wo_fits(int T, int hq_l, int hkv_l, int d, int cols, int positions);
void f32_launch_attn_wo(const float *qkv, float *kc, float *vc, int hq_l, int hkv_l, int d, int smax, const int32_t *pos, const float *cos_tab,
                        const float *sin_tab, const F32Proj &p, hipStream_t s);
void f32_launch_kv_copy(float *kc, float *vc, float *k, float *v, int hkv_l, int d, int smax, int seq,
                        int pos0, int n, int to_cache, hipStream_t s);

// ---- launchers that depend on the 16-bit element type: the same declarations in namespace bf16 and in namespace f16 ----
#define HX_DECL_NS bf16
#include "kernels_h16.inc"
#undef HX_DECL_NS
#define HX_DECL_NS f16
#include "kernels_h16.inc"
#undef HX_DECL_NS
