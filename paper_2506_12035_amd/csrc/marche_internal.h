// Internal declarations shared by the host API and the HIP kernels of
// libmarche.so.  Not part of the public ABI (include/marche.h is).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace marche {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Where active row r of the packed activations lives: image b, token tok,
// and its row in the [batch][n_tokens][d_model] residual stream.
struct RowMap {
  int32_t x_row;  // b * n_tokens + tok
  int32_t b;
  int32_t tok;
  int32_t pad;
};

// Kernel timing of the library's profiling mode (marche_profile_*): while a
// timed call runs on a thread, the first kernel it launches through
// launch_kernel() (device_common.h) carries the call's two events on its
// dispatch (hipExtLaunchKernel), so they hold the kernel's own start and end,
// not the stream's dispatch gap before it.
struct KernelEvents {
  hipEvent_t start = nullptr, stop = nullptr;
  bool used = false;
};
// This thread's slot: the timed call in progress, or nullptr.
KernelEvents *&kernel_events();

// Element type of the packed activations, weights and KV cache.
enum class DType { F32 = 0, BF16 = 1 };

// ---- elementwise / indexing (k_elementwise.hip) ----
hipError_t launch_row_map(RowMap *map, const int32_t *a_idx, const int32_t *a_off, int32_t batch,
                          int32_t n_tokens, hipStream_t s);
hipError_t launch_gather_ln(DType dt, void *out, const float *x, const RowMap *map, const float *g,
                            const float *b, int32_t rows, int32_t d_model, float eps, hipStream_t s);
hipError_t launch_decoder_input(float *x, const float *cls, const float *value, const float *mask,
                                const float *pos, const int32_t *rank, int32_t batch,
                                int32_t n_tokens, int32_t n_buf, int32_t d_model, int32_t n_known,
                                hipStream_t s);
hipError_t launch_fill_zero(void *dst, size_t bytes, hipStream_t s);
// Debug-mode check of a step's active lists; report[0] = 0 or 1 + code*batch + image
// (codes: 0 offsets, 1 token range, 2 duplicate token, 3 n_gen).
hipError_t launch_check_active(const int32_t *a_idx, const int32_t *a_off, const int32_t *n_gen,
                               int32_t batch, int32_t n_tokens, int32_t a_total, int32_t a_max,
                               int32_t gen_max, int32_t *report, hipStream_t s);

// ---- the rest of a MAR step (k_mar.hip) ----
// Encoder input rows [batch][n_buf + n_known][d_model] (Eq. 1).
hipError_t launch_encoder_input(float *x, const float *cls, const float *tok, const float *w_z,
                                const float *b_z, const float *pe, const int32_t *known,
                                int32_t batch, int32_t n_buf, int32_t n_img, int32_t n_known,
                                int32_t d_model, int32_t c_tok, hipStream_t s);
// Masked rows of the decoder input (Eq. 2).
hipError_t launch_mask_fill(float *x, const float *mask, const float *pe, const int32_t *rank,
                           int32_t batch, int32_t n_tokens, int32_t n_buf, int32_t n_known,
                           int32_t d_model, hipStream_t s);
// out[r] = LN(x[rows ? rows[r] : r]) * g + b (+ add[src % n_tokens - n_buf]).
hipError_t launch_ln_rows(DType dt, void *out, const float *x, const int32_t *rows_idx,
                          const float *g, const float *b, const float *add, int32_t rows,
                          int32_t n_tokens, int32_t n_buf, int32_t d_model, float eps,
                          hipStream_t s);
// Sinusoidal time embedding table [n_steps][freq].
hipError_t launch_time_sinus(DType dt, void *out, int32_t n_steps, int32_t freq, hipStream_t s);
// sc = SiLU(cond + temb_row), [rows][width].
hipError_t launch_silu_cond(DType dt, void *sc, const float *cond, const float *temb, int32_t rows,
                            int32_t width, hipStream_t s);
// w_t = w^T for a [rows][cols] float32 matrix.
hipError_t launch_transpose_f32(float *w_t, const float *w, int32_t rows, int32_t cols,
                                hipStream_t s);
// a = LN(h) (1 + scale) + shift (slices of mod at the offsets).
hipError_t launch_head_mod(DType dt, void *a, const float *h, const void *mod, int32_t mod_ld,
                           int32_t shift_off, int32_t scale_off, int32_t rows, int32_t width,
                           float eps, hipStream_t s);
// Coefficients of one DDPM step (see head_step_kernel).
struct HeadStep {
  float sra, srm1, c1, c2, sigma;
};
// Everything between two sampling steps' blocks, row by row (see
// head_step_kernel).  `out`: this step's output projection and DDPM update
// (final modulation at shift_off, scale_off); `in`: the next step's input
// projection and first modulated norm (slices 0 and width of mod; a == NULL:
// without the norm, which the next launch forms itself); sc != NULL:
// SiLU(cond + temb) into it.
struct HeadRows {
  bool out, in;
  float *h;
  void *a;
  const void *mod;
  int32_t mod_ld, shift_off, scale_off;
  const float *w_out, *b_out;    // [C][W], [C]
  const float *w_in, *w_in_t;    // [W][C] and its transpose
  const float *b_in;             // [W]
  const float *x_cur, *noise;    // [rows][C]
  float *x_next, *tok_out;       // tok_out: last step only
  const int32_t *out_rows;
  HeadStep st;
  void *sc;
  const float *cond, *temb;      // [rows][W], [W]
  int32_t rows, c_tok;
  float eps;
};
hipError_t launch_head_step(DType dt, const HeadRows &p, int32_t width, hipStream_t s);

// ---- GEMMs with fused epilogues (k_gemm.hip) ----
// C[M][N] = A[M][K] . W[N][K]^T (+ bias) followed by one epilogue:
//   qkv:   columns [0,D) -> q [M][D]; [D,2D) -> K cache, [2D,3D) -> V cache
//          (scattered to [b][h][tok][d] of one layer's cache)
//   resid: x[map[r].x_row][c] += C + bias        (float32 residual stream)
//   gelu:  h[r][c] = GELU(C + bias)
struct QkvOut {
  void *q;
  void *k_cache;  // layer base
  void *v_cache;  // layer base
  int32_t d_model, head_dim, n_heads, n_tokens;
};
// `shared`: the call computes a part of its cache's images, so that others may
// run beside it (see gemm_tile_kind).
hipError_t launch_gemm_qkv(DType dt, const void *a, const void *w, const float *bias, int32_t m,
                           int32_t n, int32_t k, const RowMap *map, QkvOut out, bool shared,
                           hipStream_t s);
// tag: 0 = output projection, 1 = fc2 (separate kernel symbols)
hipError_t launch_gemm_resid(DType dt, const void *a, const void *w, const float *bias, int32_t m,
                             int32_t n, int32_t k, const RowMap *map, float *x, int32_t tag,
                             bool shared, hipStream_t s);
hipError_t launch_gemm_gelu(DType dt, const void *a, const void *w, const float *bias, int32_t m,
                            int32_t n, int32_t k, void *h, bool shared, hipStream_t s);
// Sampler GEMMs: out[r][c] = act(C + bias) as out_dt (row-major, row stride
// ld), act SiLU or the identity; a float32 GEMM writes float32 only.
hipError_t launch_gemm_plain(DType dt, const void *a, const void *w, const float *bias, int32_t m,
                             int32_t n, int32_t k, void *out, DType out_dt, bool silu_act,
                             int32_t ld, hipStream_t s);
// The two products of a sampler block (width x width): y = SiLU(a w^T + bias),
// and h += gate (a w^T + bias) with the gate a slice of the modulations.  Side
// products out = a w^T + bias (bf16, same rows and reduction length as the
// main one, n columns a multiple of 128, ld = HeadSides::ld) share the launch:
// a block product of a few hundred rows leaves most compute units idle.
struct HeadSide {
  const void *a, *w;
  const float *bias;
  void *out;
  int32_t n;
};
struct HeadSides {
  HeadSide s[2];
  int32_t ld;
};
// 128-column side tiles per launch that fit beside the main product in one
// wave of workgroups (0: none, or no side products for this type).
int head_side_tiles(DType dt, int32_t m, int32_t width);
hipError_t launch_head_gemm_silu(DType dt, const void *a, const void *w, const float *bias,
                                 int32_t m, int32_t width, void *y, const HeadSides &sides,
                                 hipStream_t s);
// The first with its activations a = LN(h) (1 + scale) + shift formed in the
// same launch (bf16, where head_norm_fits: up to 16 rows, by width).
bool head_norm_fits(DType dt, int32_t m, int32_t width);
hipError_t launch_head_gemm_norm_silu(const float *h, const void *mod, int32_t mod_ld,
                                      int32_t shift_off, int32_t scale_off, float eps,
                                      const void *w, const float *bias, int32_t m, int32_t width,
                                      void *y, const HeadSides &sides, hipStream_t s);
hipError_t launch_head_gemm_gate(DType dt, const void *a, const void *w, const float *bias,
                                 int32_t m, int32_t width, float *h, const void *gate,
                                 int32_t mod_ld, const HeadSides &sides, hipStream_t s);
// Decoder embedding of the encoder rows scattered to their sequence positions
// (n = d_model): x[b][j][c] = C + bias + pe[j][c], j the position encoder row
// r = b * n_enc + i holds (i < n_buf: i; else n_buf + known[b][i - n_buf]).
hipError_t launch_gemm_embed(DType dt, const void *a, const void *w, const float *bias, int32_t m,
                             int32_t n, int32_t k, float *x, const float *pe, const int32_t *known,
                             int32_t n_enc, int32_t n_buf, int32_t n_known, int32_t n_tokens,
                             hipStream_t s);
// bf16 GEMM workgroup tile of an M x N x K product (rows x columns).
enum GemmTile {
  GEMM_TILE_256 = 0, GEMM_TILE_320, GEMM_TILE_64x128, GEMM_TILE_128, GEMM_TILE_192x128,
  GEMM_TILE_256x128, GEMM_TILE_64x64, GEMM_TILE_32x64, GEMM_TILE_32x32, GEMM_TILE_COUNT
};
int gemm_tile_kind(DType dt, int32_t m, int32_t n, int32_t k, bool shared = false);
// The tile of a sampler block's bf16 product (width x width) with side products
// of n_side columns.
int head_tile_kind(int32_t m, int32_t width, int32_t n_side);
// Whether a sampler launch of m rows and n columns (side products among them)
// over K = k runs the few-row kernel instead.
bool gemm_few_rows(DType dt, int32_t m, int32_t n, int32_t k);
// Compute units of the current device (queried once per device, then cached).
int device_cu_count();

// ---- attention (k_attn.hip) ----
struct AttnArgs {
  const void *q;        // [a_total][D] packed queries
  const void *k_cache;  // layer base [B][H][N][dh] (keys 0..N-1; the first segment)
  const void *v_cache;
  void *o;              // [a_total][D]
  const int32_t *a_off; // CSR rows per image; NULL: image b owns rows [b*a_max, (b+1)*a_max)
  const RowMap *map;
  int32_t batch, n_heads, n_tokens, head_dim, d_model, a_total, a_max;
  // Optional second key/value segment [B][H][n2][dh], attended after the
  // first in the same online-softmax pass (bf16 attention only).
  const void *k2 = nullptr;
  const void *v2 = nullptr;
  int32_t n2 = 0;
  // Optional attention mass of the generating rows (the first n_gen[b] rows
  // of image b), scores[b][h][j], written by the same kernel where
  // attn_fuses_scores() holds (one key segment).
  const int32_t *n_gen = nullptr;
  float *scores = nullptr;
  int32_t gen_max = 0;  // largest n_gen[b]
  // Optional row statistics [a_total][n_heads][2] (maximum logit, 1 / sum) for
  // launch_attn_scores, written by the kernels that run where
  // attn_fuses_scores() does not hold (and by every fp32 one).
  float *stats = nullptr;
};
hipError_t launch_attention(DType dt, const AttnArgs &a, hipStream_t s);
// Whether these bf16 arguments run the resident-K/V kernel (one workgroup per
// (image, head)).
bool attn_resident(const AttnArgs &a);
// Whether bf16 attention with these sizes runs the register-staged streaming
// kernel (head width 64, one key segment of whole tiles).
bool attn_streams(int32_t head_dim, int32_t n_tokens, bool two_segments);
// Wavefronts of 32 queries per workgroup of the streaming kernel that these
// bf16 arguments run (where the resident one does not).
int attn_query_blocks(const AttnArgs &a);
// Whether bf16 attention with these sizes can write the score pass itself:
// the resident kernel (every key of a head in LDS), or the streaming kernel
// when the generating rows fit its first query chunk.
bool attn_fuses_scores(int32_t a_max, int32_t n_tokens, int32_t head_dim, int32_t gen_max);
// dst[b][h] = [a[b][h] (na rows) ; c[b][h] (nc rows)], rows of dh elements, for
// K and V: the concatenation of the active and cached segments.
hipError_t launch_concat_kv(DType dt, void *k_dst, void *v_dst, const void *k_a, const void *v_a,
                            const void *k_c, const void *v_c, int32_t bh, int32_t na, int32_t nc,
                            int32_t head_dim, hipStream_t s);
// scores[b][h][j] = sum over the first n_gen[b] active rows i of P_h[i][j]
hipError_t launch_attn_scores(DType dt, const AttnArgs &a, const int32_t *n_gen, float *scores,
                              hipStream_t s);

// ---- selection (k_select.hip) ----
// lowest = false: highest scores first; true: lowest scores first.
hipError_t launch_select_topk(const float *scores, int32_t n_parts, const int32_t *excl_idx,
                              const int32_t *excl_off, int32_t batch, int32_t n_tokens, int32_t k,
                              int32_t *out_idx, const int32_t *out_off, bool lowest,
                              hipStream_t s);

}  // namespace marche
