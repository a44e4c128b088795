// The rest of a MAR step around the decoder: the encoder's input rows (Eq. 1),
// the decoder input's masked rows (Eq. 2), LayerNorm of gathered rows, and the
// kernels of the sampler of Eq. 3 between its GEMMs (time embedding table,
// condition SiLU, modulated LayerNorms, output projection + DDPM step + input
// projection).
//
// Except for the last of these, row kernels run one wavefront per row, four
// rows per 256-thread workgroup;
// a row of width NV * 256 is NV float4 chunks per lane.  LayerNorm statistics
// are float32: the mean, then the population variance of the centred values,
// eps inside the square root.
#include "device_common.h"

namespace marche {

namespace {

template <typename T>
__device__ __forceinline__ void store_row4(T *p, float a, float b, float c, float d) {
  if constexpr (sizeof(T) == 4) {
    *reinterpret_cast<float4 *>(p) = make_float4(a, b, c, d);
  } else {
    bf16x4 pk = {(bf16)a, (bf16)b, (bf16)c, (bf16)d};
    *reinterpret_cast<bf16x4 *>(p) = pk;
  }
}

template <typename T>
__device__ __forceinline__ float4 load_row4(const T *p) {
  if constexpr (sizeof(T) == 4) {
    return *reinterpret_cast<const float4 *>(p);
  } else {
    const bf16x4 v = *reinterpret_cast<const bf16x4 *>(p);
    return make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
  }
}

// Mean and reciprocal standard deviation of a row held as v[NV] (centres v).
template <int NV>
__device__ __forceinline__ float centre_rstd(float4 (&v)[NV], float eps) {
  constexpr float inv_d = 1.0f / (NV * 256);
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
  const float mean = wave_sum(s) * inv_d;
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    v[i].x -= mean; v[i].y -= mean; v[i].z -= mean; v[i].w -= mean;
    ss += (v[i].x * v[i].x + v[i].y * v[i].y) + (v[i].z * v[i].z + v[i].w * v[i].w);
  }
  return 1.0f / sqrtf(wave_sum(ss) * inv_d + eps);
}

}  // namespace

// ---- Eq. 1: encoder input rows -------------------------------------------
// Row i of image b (b = row / n_enc): i < n_buf -> cls[b] + pe[i]; else the
// known image token p = known[b][i - n_buf]: w_z . tok[b][p] + b_z + pe[n_buf + p].
//
// Bound by writing x.  Every lane keeps the CM weights of its V columns in
// registers for `per_wave` rows; a wavefront that read them again for each row
// (strided by a weight row from lane to lane) took 271 us for 64 images x 195
// rows x 1024 columns x 16 channels, and 21 us now (30 and 4.9 for one image).
// The weights come through LDS, where the copy is coalesced and one padding
// word in 32 spreads the lanes' strided reads over the banks.  Rows go four at
// a time with their loads up front.  V x CM <= 128 registers of weights.
template <int CM>
struct EncIn {
  static constexpr int V = CM >= 64 ? 2 : 4;  // columns per lane
  static constexpr int COLS = 64 * V;         // columns per workgroup
  static constexpr int SLAB = COLS * CM;      // weights of those columns
};

template <int CM>
__global__ __launch_bounds__(256) void encoder_input_kernel(
    float *__restrict__ x, const float *__restrict__ cls, const float *__restrict__ tok,
    const float *__restrict__ w_z, const float *__restrict__ b_z, const float *__restrict__ pe,
    const int32_t *__restrict__ known, int rows, int n_enc, int n_buf, int n_img, int n_known,
    int C, int D, int per_wave) {
  using E = EncIn<CM>;
  constexpr int V = E::V, RB = 4;
  typedef float Vec __attribute__((ext_vector_type(V)));
  __shared__ float slab[E::SLAB + E::SLAB / 32];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col0 = blockIdx.x * E::COLS;
  const int d0 = col0 + V * lane;  // D is a multiple of COLS

  float w[V][CM];
  Vec bz = {};
  if (n_known > 0) {
    const float *ws = w_z + (size_t)col0 * C;
#pragma unroll 8
    for (int i = threadIdx.x; i < E::COLS * C; i += 256) slab[i + (i >> 5)] = ws[i];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < V; ++e)
#pragma unroll
      for (int c = 0; c < CM; ++c) {
        const int i = (V * lane + e) * C + min(c, C - 1);
        w[e][c] = c < C ? slab[i + (i >> 5)] : 0.f;
      }
    bz = *reinterpret_cast<const Vec *>(b_z + d0);
  } else {
#pragma unroll
    for (int e = 0; e < V; ++e)
#pragma unroll
      for (int c = 0; c < CM; ++c) w[e][c] = 0.f;
  }

  const int first = (blockIdx.y * 4 + wave) * per_wave;
  const int last = min(rows, first + per_wave);
  for (int r0 = first; r0 < last; r0 += RB) {
    float t[RB];
    Vec cl[RB], q[RB];
    bool buf[RB];
#pragma unroll
    for (int j = 0; j < RB; ++j) {
      const int row = min(r0 + j, last - 1);
      const int b = row / n_enc, i = row - b * n_enc;
      buf[j] = i < n_buf;
      t[j] = 0.f;
      cl[j] = bz;
      int at = i;
      if (buf[j]) {
        cl[j] = *reinterpret_cast<const Vec *>(cls + (size_t)b * D + d0);
      } else {
        const int p = known[(size_t)b * n_known + (i - n_buf)];
        // token value, zero-padded to CM channels
        if (lane < C) t[j] = tok[((size_t)b * n_img + p) * C + lane];
        at = n_buf + p;
      }
      q[j] = *reinterpret_cast<const Vec *>(pe + (size_t)at * D + d0);
    }
#pragma unroll
    for (int j = 0; j < RB; ++j) {
      if (r0 + j >= last) break;
      Vec o = cl[j];
      if (!buf[j]) {
        float acc[V] = {};
#pragma unroll
        for (int c = 0; c < CM; ++c) {
          const float tc = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t[j]), c));
#pragma unroll
          for (int e = 0; e < V; ++e) acc[e] = fmaf(w[e][c], tc, acc[e]);
        }
#pragma unroll
        for (int e = 0; e < V; ++e) o[e] = acc[e] + bz[e];
      }
#pragma unroll
      for (int e = 0; e < V; ++e) o[e] += q[j][e];
      *reinterpret_cast<Vec *>(x + (size_t)(r0 + j) * D + d0) = o;
    }
  }
}

// ---- Eq. 2: masked rows of the decoder input ------------------------------
// x[b][n_buf + p] = mask + pe[n_buf + p] for every image token p with
// rank[b][p] >= n_known; known tokens and buffer rows are left to the
// embedding GEMM.
template <int NV>
__global__ __launch_bounds__(256) void mask_fill_kernel(float *__restrict__ x,
                                                        const float *__restrict__ mask,
                                                        const float *__restrict__ pe,
                                                        const int32_t *__restrict__ rank, int rows,
                                                        int n_tokens, int n_buf, int n_img,
                                                        int n_known) {
  constexpr int D = NV * 256;
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);  // b * n_img + p
  if (row >= rows) return;
  if (rank[row] < n_known) return;
  const int b = row / n_img, j = n_buf + (row - b * n_img);
  const float4 *m4 = reinterpret_cast<const float4 *>(mask);
  const float4 *p4 = reinterpret_cast<const float4 *>(pe + (size_t)j * D);
  float4 *o = reinterpret_cast<float4 *>(x + ((size_t)b * n_tokens + j) * D);
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const float4 a = m4[lane + 64 * k], q = p4[lane + 64 * k];
    o[lane + 64 * k] = make_float4(a.x + q.x, a.y + q.y, a.z + q.z, a.w + q.w);
  }
}

// ---- LayerNorm of gathered rows -------------------------------------------
// out[r] = LN(x[src]) * g + b (+ add[tok - n_buf]), src = rows ? rows[r] : r,
// tok = src % n_tokens.  The encoder's final norm (rows = NULL, add = NULL)
// and the condition of Eq. 3 (decoder norm of the generating rows plus the
// head's positional embedding).
template <typename OutT, int NV>
__global__ __launch_bounds__(256) void ln_rows_kernel(OutT *__restrict__ out,
                                                      const float *__restrict__ x,
                                                      const int32_t *__restrict__ rows_idx,
                                                      const float *__restrict__ g,
                                                      const float *__restrict__ bta,
                                                      const float *__restrict__ add, int rows,
                                                      int n_tokens, int n_buf, float eps) {
  constexpr int D = NV * 256;
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows) return;
  const int src = rows_idx ? rows_idx[r] : r;
  const float4 *xr = reinterpret_cast<const float4 *>(x + (size_t)src * D);
  float4 v[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = xr[lane + 64 * i];
  const float rstd = centre_rstd<NV>(v, eps);
  const float4 *g4 = reinterpret_cast<const float4 *>(g);
  const float4 *b4 = reinterpret_cast<const float4 *>(bta);
  const float4 *a4 =
      add ? reinterpret_cast<const float4 *>(add + (size_t)(src % n_tokens - n_buf) * D) : nullptr;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c4 = lane + 64 * i;
    const float4 gg = g4[c4], bb = b4[c4];
    float4 y = make_float4(v[i].x * rstd * gg.x + bb.x, v[i].y * rstd * gg.y + bb.y,
                           v[i].z * rstd * gg.z + bb.z, v[i].w * rstd * gg.w + bb.w);
    if (a4) {
      const float4 q = a4[c4];
      y.x += q.x; y.y += q.y; y.z += q.z; y.w += q.w;
    }
    store_row4(out + (size_t)r * D + 4 * c4, y.x, y.y, y.z, y.w);
  }
}

// ---- Eq. 3: sampler --------------------------------------------------------
// Sinusoidal embedding of timesteps 0..n_steps-1: out[i][f] = cos(i w_f) for
// f < F/2, sin(i w_{f - F/2}) otherwise, w_j = 10000^(-j / (F/2)).
template <typename OutT>
__global__ __launch_bounds__(256) void time_sinus_kernel(OutT *__restrict__ out, int n_steps, int F) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= n_steps * F) return;
  const int i = idx / F, f = idx - i * F, half = F / 2;
  const int j = f < half ? f : f - half;
  const float w = expf(-9.210340371976184f * (float)j / (float)half);  // ln 10000
  const float a = (float)i * w;
  out[idx] = (OutT)(f < half ? cosf(a) : sinf(a));
}

// sc[r][c] = SiLU(cond[r][c] + temb[c]) for one timestep's embedding row.
template <typename OutT>
__global__ __launch_bounds__(256) void silu_cond_kernel(OutT *__restrict__ sc,
                                                        const float *__restrict__ cond,
                                                        const float *__restrict__ temb, int rows,
                                                        int W) {
  const int w4 = W / 4;
  const int idx = blockIdx.x * 256 + threadIdx.x;  // float4 index
  if (idx >= rows * w4) return;
  const int c4 = idx % w4;
  const float4 a = reinterpret_cast<const float4 *>(cond)[idx];
  const float4 t = reinterpret_cast<const float4 *>(temb)[c4];
  store_row4(sc + (size_t)idx * 4, silu(a.x + t.x), silu(a.y + t.y), silu(a.z + t.z),
             silu(a.w + t.w));
}

// w_t[c][d] = w[d][c] for a [rows][cols] float32 matrix (the input
// projection, so that lanes over d read it coalesced).
__global__ __launch_bounds__(256) void transpose_f32_kernel(float *__restrict__ w_t,
                                                            const float *__restrict__ w, int rows,
                                                            int cols) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= rows * cols) return;
  const int d = idx / cols, c = idx - d * cols;
  w_t[(size_t)c * rows + d] = w[idx];
}

// a[r] = LN(h[r]) * (1 + scale) + shift, shift and scale W-wide slices of
// mod[r] at the given offsets: the modulated norm between two blocks (the
// gated residual is the epilogue of the block's second product).
template <typename T, int NV>
__global__ __launch_bounds__(256) void head_mod_kernel(T *__restrict__ a_out,
                                                       const float *__restrict__ h,
                                                       const T *__restrict__ mod, int mod_ld,
                                                       int shift_off, int scale_off, int rows,
                                                       float eps) {
  constexpr int W = NV * 256;
  constexpr float inv_w = 1.0f / W;
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows) return;
  const T *mr = mod + (size_t)r * mod_ld;
  const float4 *hr = reinterpret_cast<const float4 *>(h + (size_t)r * W);
  float4 v[NV], t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = hr[lane + 64 * k];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    t.x += v[k].x; t.y += v[k].y; t.z += v[k].z; t.w += v[k].w;
  }
  const float mean = norm_mean(norm_sum4(t.x, t.y, t.z, t.w), inv_w);
  t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    v[k] = make_float4(norm_centre(v[k].x, mean), norm_centre(v[k].y, mean),
                       norm_centre(v[k].z, mean), norm_centre(v[k].w, mean));
    t = make_float4(fmaf(v[k].x, v[k].x, t.x), fmaf(v[k].y, v[k].y, t.y),
                    fmaf(v[k].z, v[k].z, t.z), fmaf(v[k].w, v[k].w, t.w));
  }
  const float rstd = norm_rstd(norm_sum4(t.x, t.y, t.z, t.w), inv_w, eps);
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int c = 4 * (lane + 64 * k);
    const float4 sh = load_row4(mr + shift_off + c), sc = load_row4(mr + scale_off + c);
    store_row4(a_out + (size_t)r * W + c, norm_mod(v[k].x, rstd, sc.x, sh.x),
               norm_mod(v[k].y, rstd, sc.y, sh.y), norm_mod(v[k].z, rstd, sc.z, sh.z),
               norm_mod(v[k].w, rstd, sc.w, sh.w));
  }
}

// Sum over a workgroup of 256 threads; `red` holds four floats.
__device__ __forceinline__ float block_sum(float v, float *red) {
  v = wave_sum_dpp(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// Everything between two sampling steps' blocks, one workgroup per row (the
// row's columns are spread over 256 threads, NV each):
//   out: a = LN(h) (1 + scale_f) + shift_f;  eps = w_out a + b_out;
//        x0 = sra x - srm1 eps;  x' = c1 x0 + c2 x + sigma noise  (sigma =
//        tau * sqrt(posterior variance), 0 at the last step, where the
//        result also goes to tok_out[out_rows[r]]);
//   in:  h = w_in x' + b_in;  a = LN(h) (1 + scale_0) + shift_0;
//   sc:  SiLU(cond + temb) of a later step's modulations.
// Its time is its chain of dependent loads and sums; as four kernels of one
// wavefront per row (norm, output + update, input + norm, SiLU) the same work
// took 29 us per sampling step at 512 rows of width 1280.
// The weights of both projections do not depend on the row: where they fit
// the registers (PRE) their loads go out first, beside those of the row.
template <typename T, int NV, int CM>
__global__ __launch_bounds__(256) void head_step_kernel(HeadRows p) {
  constexpr int W = NV * 256;
  constexpr float inv_w = 1.0f / W;
  constexpr int CW = (CM + 3) / 4;               // output channels per wavefront
  constexpr bool PRE = NV * CM <= 96;
  constexpr int PO = PRE ? CW * NV : 1, PI = PRE ? CM / 4 * NV : 1;
  __shared__ float red[4][4];
  __shared__ __attribute__((aligned(16))) float as[W];
  __shared__ float ev[CM];
  __shared__ __attribute__((aligned(16))) float xv[CM];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int C = p.c_tok;
  // w_in rows are whole, aligned float4s
  const bool vec_in = C == CM && (reinterpret_cast<uintptr_t>(p.w_in) & 15) == 0;

  // (the row's loads before the weights': they return in order)
  const int r = blockIdx.x;
  float *hr = p.h + (size_t)r * W;
  const T *mr = static_cast<const T *>(p.mod) + (size_t)r * p.mod_ld;
  float v[NV], fsc[NV], fsh[NV], sc0[NV], sh0[NV];
  float xc = 0.f, nz = 0.f;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int col = tid + 256 * k;
    if (p.out) {
      v[k] = hr[col];
      fsc[k] = to_f32(mr[p.scale_off + col]);
      fsh[k] = to_f32(mr[p.shift_off + col]);
    }
    if (p.in && p.a) {
      sc0[k] = to_f32(mr[W + col]);
      sh0[k] = to_f32(mr[col]);
    }
  }
  if (tid < C) {
    const size_t idx = (size_t)r * C + tid;
    xc = p.x_cur[idx];
    if (p.out && p.st.sigma != 0.f) nz = p.noise[idx];
  }
  float4 wo[PO], wi[PI];
  float bi[NV];
  // channel wave * CW + i of the output projection; channels past C repeat the last
  auto w_out4 = [&](int i, int k) {
    const int c = min(wave * CW + i, C - 1);
    return *reinterpret_cast<const float4 *>(p.w_out + (size_t)c * W + 4 * (lane + 64 * k));
  };
  auto w_in4 = [&](int k, int c4) {
    return *reinterpret_cast<const float4 *>(p.w_in + (size_t)(tid + 256 * k) * CM + 4 * c4);
  };
  if constexpr (PRE) {
    if (p.out) {
#pragma unroll
      for (int i = 0; i < CW; ++i)
#pragma unroll
        for (int k = 0; k < NV; ++k) wo[i * NV + k] = w_out4(i, k);
    }
    if (p.in && vec_in) {
#pragma unroll
      for (int k = 0; k < NV; ++k)
#pragma unroll
        for (int c4 = 0; c4 < CM / 4; ++c4) wi[k * (CM / 4) + c4] = w_in4(k, c4);
    }
  }
  if (p.in) {
#pragma unroll
    for (int k = 0; k < NV; ++k) bi[k] = p.b_in[tid + 256 * k];
  }
  const float bo = p.out && tid < C ? p.b_out[tid] : 0.f;
  if (tid < CM) xv[tid] = xc;  // channels past C hold 0
  if (p.out) {
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < NV; ++k) s += v[k];
    const float mean = norm_mean(block_sum(s, red[0]), inv_w);
    float ss = 0.f;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      v[k] = norm_centre(v[k], mean);
      ss = fmaf(v[k], v[k], ss);
    }
    const float rstd = norm_rstd(block_sum(ss, red[1]), inv_w, p.eps);
#pragma unroll
    for (int k = 0; k < NV; ++k) as[tid + 256 * k] = norm_mod(v[k], rstd, fsc[k], fsh[k]);
    __syncthreads();
    float acc[CW];
#pragma unroll
    for (int i = 0; i < CW; ++i) acc[i] = 0.f;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const float4 a = *reinterpret_cast<const float4 *>(as + 4 * (lane + 64 * k));
#pragma unroll
      for (int i = 0; i < CW; ++i) {
        float4 w;
        if constexpr (PRE) w = wo[i * NV + k];
        else w = w_out4(i, k);
        acc[i] = fmaf(a.x, w.x, fmaf(a.y, w.y, fmaf(a.z, w.z, fmaf(a.w, w.w, acc[i]))));
      }
    }
#pragma unroll
    for (int i = 0; i < CW; ++i) {
      const float t = wave_sum_dpp(acc[i]);
      if (lane == 0 && wave * CW + i < CM) ev[wave * CW + i] = t;
    }
    __syncthreads();
    if (tid < C) {
      const size_t idx = (size_t)r * C + tid;
      const float eps_v = ev[tid] + bo;
      const float x0 = p.st.sra * xc - p.st.srm1 * eps_v;
      float xn = p.st.c1 * x0 + p.st.c2 * xc;
      if (p.st.sigma != 0.f) xn = fmaf(p.st.sigma, nz, xn);
      p.x_next[idx] = xn;
      if (p.tok_out) p.tok_out[(size_t)p.out_rows[r] * C + tid] = xn;
      xv[tid] = xn;
    }
  }
  if (p.in) {
    __syncthreads();
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int col = tid + 256 * k;
      float h = bi[k];
      if (vec_in) {
#pragma unroll
        for (int c4 = 0; c4 < CM / 4; ++c4) {
          const float4 x = *reinterpret_cast<const float4 *>(xv + 4 * c4);
          float4 w;
          if constexpr (PRE) w = wi[k * (CM / 4) + c4];
          else w = w_in4(k, c4);
          h = fmaf(w.x, x.x, h);
          h = fmaf(w.y, x.y, h);
          h = fmaf(w.z, x.z, h);
          h = fmaf(w.w, x.w, h);
        }
      } else {
#pragma unroll 8
        for (int c = 0; c < C; ++c) h = fmaf(p.w_in_t[(size_t)c * W + col], xv[c], h);
      }
      hr[col] = h;
      v[k] = h;
      s += h;
    }
    if (p.a) {
      const float mean = norm_mean(block_sum(s, red[2]), inv_w);
      float ss = 0.f;
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        v[k] = norm_centre(v[k], mean);
        ss = fmaf(v[k], v[k], ss);
      }
      const float rstd = norm_rstd(block_sum(ss, red[3]), inv_w, p.eps);
      T *ar = static_cast<T *>(p.a) + (size_t)r * W;
#pragma unroll
      for (int k = 0; k < NV; ++k)
        ar[tid + 256 * k] = from_f32<T>(norm_mod(v[k], rstd, sc0[k], sh0[k]));
    }
  }
  if (p.sc) {
    T *sr = static_cast<T *>(p.sc) + (size_t)r * W;
    const float *cr = p.cond + (size_t)r * W;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int col = tid + 256 * k;
      sr[col] = from_f32<T>(silu(cr[col] + p.temb[col]));
    }
  }
}

// ------------------------------------------------------------------ launchers

#define MARCHE_NV_SWITCH(nv, CALL)        \
  switch (nv) {                           \
    case 1: CALL(1); break;               \
    case 2: CALL(2); break;               \
    case 3: CALL(3); break;               \
    case 4: CALL(4); break;               \
    case 5: CALL(5); break;               \
    case 6: CALL(6); break;               \
    case 7: CALL(7); break;               \
    case 8: CALL(8); break;               \
    case 9: CALL(9); break;               \
    case 10: CALL(10); break;             \
    case 11: CALL(11); break;             \
    case 12: CALL(12); break;             \
    case 13: CALL(13); break;             \
    case 14: CALL(14); break;             \
    case 15: CALL(15); break;             \
    case 16: CALL(16); break;             \
    default: return hipErrorInvalidValue; \
  }

// Token channels rounded up to 4, 8, 16, 32 or 64 (compile-time loops).  Rows
// per wavefront: enough wavefronts to fill the chip (16 per compute unit)
// before any takes a second row, then up to 32 rows for one load of the
// weights.
template <int CM>
static void encoder_input_go(hipStream_t s, float *x, const float *cls, const float *tok,
                             const float *w_z, const float *b_z, const float *pe,
                             const int32_t *known, int rows, int n_enc, int n_buf, int n_img,
                             int n_known, int c, int d) {
  const int cols = d / EncIn<CM>::COLS;
  const int64_t waves = 16 * (int64_t)device_cu_count();
  int per_wave = (int)(((int64_t)rows * cols + waves - 1) / waves);
  per_wave = per_wave > 32 ? 32 : per_wave;
  // the grid's second dimension holds 65535
  const int need = (rows + 4 * 65535 - 1) / (4 * 65535);
  if (per_wave < need) per_wave = need;
  const int groups = (rows + 4 * per_wave - 1) / (4 * per_wave);
  launch_kernel(encoder_input_kernel<CM>, dim3(cols, groups), 256, 0, s, x, cls, tok, w_z, b_z, pe, known,
                rows, n_enc, n_buf, n_img, n_known, c, d, per_wave);
}

hipError_t launch_encoder_input(float *x, const float *cls, const float *tok, const float *w_z,
                                const float *b_z, const float *pe, const int32_t *known,
                                int32_t batch, int32_t n_buf, int32_t n_img, int32_t n_known,
                                int32_t d_model, int32_t c_tok, hipStream_t s) {
  const int n_enc = n_buf + n_known, rows = batch * n_enc;
  if (rows == 0) return hipSuccess;
  if (d_model % 256 != 0 || d_model > 4096 || c_tok < 1 || c_tok > 64) return hipErrorInvalidValue;
#define E_(CM) encoder_input_go<CM>(s, x, cls, tok, w_z, b_z, pe, known, rows, n_enc, n_buf, n_img, \
                                    n_known, c_tok, d_model)
  if (c_tok <= 4) E_(4);
  else if (c_tok <= 8) E_(8);
  else if (c_tok <= 16) E_(16);
  else if (c_tok <= 32) E_(32);
  else E_(64);
#undef E_
  return hipGetLastError();
}

hipError_t launch_mask_fill(float *x, const float *mask, const float *pe, const int32_t *rank,
                            int32_t batch, int32_t n_tokens, int32_t n_buf, int32_t n_known,
                            int32_t d_model, hipStream_t s) {
  const int n_img = n_tokens - n_buf, rows = batch * n_img;
  if (rows == 0) return hipSuccess;
  if (d_model % 256 != 0) return hipErrorInvalidValue;
  const int grid = (rows + 3) / 4;
#define L_(NV)                                                                          \
  launch_kernel(mask_fill_kernel<NV>, grid, 256, 0, s, x, mask, pe, rank, rows, n_tokens, n_buf, n_img, \
                                            n_known)
  MARCHE_NV_SWITCH(d_model / 256, L_)
#undef L_
  return hipGetLastError();
}

hipError_t launch_ln_rows(DType dt, void *out, const float *x, const int32_t *rows_idx,
                          const float *g, const float *b, const float *add, int32_t rows,
                          int32_t n_tokens, int32_t n_buf, int32_t d_model, float eps,
                          hipStream_t s) {
  if (rows == 0) return hipSuccess;
  if (d_model % 256 != 0) return hipErrorInvalidValue;
  const int grid = (rows + 3) / 4;
  if (dt == DType::F32) {
#define L_(NV)                                                                                  \
  launch_kernel(ln_rows_kernel<float, NV>, grid, 256, 0, s, static_cast<float *>(out), x, rows_idx, g, b, add, \
                                                 rows, n_tokens, n_buf, eps)
    MARCHE_NV_SWITCH(d_model / 256, L_)
#undef L_
  } else {
#define L_(NV)                                                                                \
  launch_kernel(ln_rows_kernel<bf16, NV>, grid, 256, 0, s, static_cast<bf16 *>(out), x, rows_idx, g, b, add, \
                                                rows, n_tokens, n_buf, eps)
    MARCHE_NV_SWITCH(d_model / 256, L_)
#undef L_
  }
  return hipGetLastError();
}

hipError_t launch_time_sinus(DType dt, void *out, int32_t n_steps, int32_t freq, hipStream_t s) {
  const int n = n_steps * freq;
  if (n == 0) return hipSuccess;
  const int grid = (n + 255) / 256;
  if (dt == DType::F32)
    launch_kernel(time_sinus_kernel<float>, grid, 256, 0, s,
                  static_cast<float *>(out), n_steps, freq);
  else
    launch_kernel(time_sinus_kernel<bf16>, grid, 256, 0, s,
                  static_cast<bf16 *>(out), n_steps, freq);
  return hipGetLastError();
}

hipError_t launch_silu_cond(DType dt, void *sc, const float *cond, const float *temb, int32_t rows,
                            int32_t width, hipStream_t s) {
  const int n4 = rows * (width / 4);
  if (n4 == 0) return hipSuccess;
  if (width % 4 != 0) return hipErrorInvalidValue;
  const int grid = (n4 + 255) / 256;
  if (dt == DType::F32)
    launch_kernel(silu_cond_kernel<float>, grid, 256, 0, s,
                  static_cast<float *>(sc), cond, temb, rows, width);
  else
    launch_kernel(silu_cond_kernel<bf16>, grid, 256, 0, s,
                  static_cast<bf16 *>(sc), cond, temb, rows, width);
  return hipGetLastError();
}

hipError_t launch_transpose_f32(float *w_t, const float *w, int32_t rows, int32_t cols,
                                hipStream_t s) {
  const int n = rows * cols;
  if (n == 0) return hipSuccess;
  launch_kernel(transpose_f32_kernel, (n + 255) / 256, 256, 0, s, w_t, w, rows, cols);
  return hipGetLastError();
}

hipError_t launch_head_mod(DType dt, void *a, const float *h, const void *mod, int32_t mod_ld,
                           int32_t shift_off, int32_t scale_off, int32_t rows, int32_t width,
                           float eps, hipStream_t s) {
  if (rows == 0) return hipSuccess;
  if (width % 256 != 0) return hipErrorInvalidValue;
  const int grid = (rows + 3) / 4;
  if (dt == DType::F32) {
#define L_(NV)                                                                               \
  launch_kernel(head_mod_kernel<float, NV>, grid, 256, 0, s, static_cast<float *>(a), h,     \
                static_cast<const float *>(mod), mod_ld, shift_off, scale_off, rows, eps)
    MARCHE_NV_SWITCH(width / 256, L_)
#undef L_
  } else {
#define L_(NV)                                                                               \
  launch_kernel(head_mod_kernel<bf16, NV>, grid, 256, 0, s, static_cast<bf16 *>(a), h,       \
                static_cast<const bf16 *>(mod), mod_ld, shift_off, scale_off, rows, eps)
    MARCHE_NV_SWITCH(width / 256, L_)
#undef L_
  }
  return hipGetLastError();
}

template <typename T, int NV>
static void head_step_dispatch(const HeadRows &p, hipStream_t s) {
#define E_(CM) launch_kernel(head_step_kernel<T, NV, CM>, p.rows, 256, 0, s, p)
  if (p.c_tok <= 4) E_(4);
  else if (p.c_tok <= 8) E_(8);
  else if (p.c_tok <= 16) E_(16);
  else if (p.c_tok <= 32) E_(32);
  else E_(64);
#undef E_
}

hipError_t launch_head_step(DType dt, const HeadRows &p, int32_t width, hipStream_t s) {
  if (p.rows == 0) return hipSuccess;
  if (width % 256 != 0 || p.c_tok < 1 || p.c_tok > 64) return hipErrorInvalidValue;
  if (dt == DType::F32) {
#define L_(NV) head_step_dispatch<float, NV>(p, s)
    MARCHE_NV_SWITCH(width / 256, L_)
#undef L_
  } else {
#define L_(NV) head_step_dispatch<bf16, NV>(p, s)
    MARCHE_NV_SWITCH(width / 256, L_)
#undef L_
  }
  return hipGetLastError();
}

#undef MARCHE_NV_SWITCH

}  // namespace marche
