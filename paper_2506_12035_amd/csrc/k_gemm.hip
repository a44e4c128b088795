// GEMMs on the ragged active set with fused epilogues.
//
// C[M][N] = A[M][K] . W[N][K]^T: A is the packed activation of the active
// rows (M = active rows of all images, any value), W a weight in nn.Linear
// layout.  Both operands are K-contiguous, which is the layout MFMA wants for
// both sides.  The epilogue adds the bias and then either
//   - splits q|k|v: q to the packed query buffer, k and v scattered into the
//     layer's KV cache at [b][h][tok][d]           (QKV projection + cache write)
//   - adds into the float32 residual stream row     (output projection, fc2)
//   - applies exact GELU and stores the hidden row  (fc1)
//
// bf16 path (v_mfma_f32_32x32x16_bf16, fp32 accumulators), one workgroup per
// CU: a 256x256 tile (four wavefronts for K >= 2048, eight below) or a 320x256
// tile (whole 320-token images per tile row, eight wavefronts) for shapes that
// fill the chip in whole waves, else 256, 192, 128 or 64 rows x 128 columns, or
// 64 x 64 to 32 x 32 for a few hundred rows.
// All load operands straight from global memory into XOR-swizzled LDS stages
// and write back through LDS in row-major order.  The sampler's products on up
// to 40 rows have a kernel of their own.
//
// fp32 path: fp32 matrix instructions, a 64x64 tile or, for few rows, a
// workgroup per 16 columns whose wavefronts split K.
#include <algorithm>

#include "device_common.h"

namespace marche {

// ------------------------------------------------------------------ epilogues
//
// Every epilogue works on four consecutive output columns col0..col0+3 of one
// row (col0 a multiple of 4), so each lane issues 8- or 16-byte stores.  Four
// consecutive columns never straddle a q|k|v third or a head (d_model and
// head_dim are multiples of 4).
//
// The write-back issues every load (row addressing data, biases, residual
// priors) before the stores it feeds: on this architecture the vector-memory
// counter also counts stores, so a load issued after a store would wait for
// the store's acknowledgement.

template <typename T>
__device__ __forceinline__ void store4(T *p, f32x4 v) {
  if constexpr (sizeof(T) == 4) {
    *reinterpret_cast<f32x4 *>(p) = v;
  } else {
    bf16x4 pk = {(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]};
    *reinterpret_cast<bf16x4 *>(p) = pk;
  }
}

__device__ __forceinline__ f32x4 load_bias4(const float *bias, int col0) {
  return *reinterpret_cast<const f32x4 *>(bias + col0);
}

// Epilogue interface: row(r) per-row addressing data (may load the row map);
// col(c0) per-column addressing data for the four columns c0..c0+3, computed
// once per lane where the columns of a lane are fixed; bias4(c0); prior(row,
// col) what the result is combined with (residual epilogues: the value it is
// added to); combine(acc + bias, prior) the value stored; store(row, r, col,
// v).  Epilogues without a prior (kPrior = false) store acc + bias.

// Epilogues that combine with nothing, or by adding.
struct PlainPrior {
  static constexpr bool kPrior = false;
  using Prior = f32x4;
  __device__ __forceinline__ f32x4 combine(f32x4 v, const Prior &) const { return v; }
};
struct AddPrior {
  static constexpr bool kPrior = true;
  using Prior = f32x4;
  __device__ __forceinline__ f32x4 combine(f32x4 v, const Prior &p) const { return v + p; }
};

template <typename T>
struct EpiQkv : PlainPrior {
  T *q;
  T *kc;
  T *vc;
  const float *bias;
  const RowMap *map;
  int d_model, head_dim, n_heads, n_tokens;
  // 32-bit element offsets: the host limits every buffer to < 2^31 elements.
  // A row's offset in q and in a K/V cache layer, computed once per row when
  // the tile stages its row records, so the stores add instead of multiply.
  struct Row {
    uint32_t q_off;   // r * d_model
    uint32_t kv_off;  // (b * n_heads * n_tokens + tok) * head_dim
  };
  struct Col {
    T *base;       // q, or the K or V cache of the layer
    uint32_t off;  // column offset: c0 for q, h*n_tokens*head_dim + d for K/V
    bool is_q;
  };
  __device__ __forceinline__ Row row(int r) const {
    const RowMap m = map[r];
    return Row{(uint32_t)(r * d_model), (uint32_t)((m.b * n_heads * n_tokens + m.tok) * head_dim)};
  }
  // Which of q, K and V a column belongs to is decided once per wavefront:
  // a wavefront has a span of 16 (fp32), 32, 64 or 128 columns aligned to its
  // width, and d_model is a multiple of 256, so no span crosses from one of
  // the three into the next.  The choice is then uniform (scalar) and the
  // stores take no divergent branches.
  __device__ __forceinline__ Col col(int c0) const {
    const int which = __builtin_amdgcn_readfirstlane(c0 < d_model ? 0 : c0 < 2 * d_model ? 1 : 2);
    if (which == 0) return Col{q, (uint32_t)c0, true};
    const int c = c0 - which * d_model;
    const int h = c / head_dim, d = c - h * head_dim;
    return Col{which == 1 ? kc : vc, (uint32_t)(h * n_tokens * head_dim + d), false};
  }
  __device__ __forceinline__ f32x4 bias4(int c0) const { return load_bias4(bias, c0); }
  __device__ __forceinline__ void store(const Row &m, int, const Col &c, f32x4 v) const {
    store4(c.base + (c.is_q ? m.q_off : m.kv_off) + c.off, v);
  }
};

// TAG only distinguishes the output projection (0) from fc2 (1) as kernel
// symbols, so per-kernel profiles can tell them apart.
template <int TAG>
struct EpiResid : AddPrior {
  float *x;
  const float *bias;
  const RowMap *map;
  int n;
  using Row = int32_t;  // element offset of the residual-stream row (< 2^31)
  using Col = int32_t;
  __device__ __forceinline__ Row row(int r) const { return map[r].x_row * n; }
  __device__ __forceinline__ Col col(int c0) const { return c0; }
  __device__ __forceinline__ f32x4 bias4(int c0) const { return load_bias4(bias, c0); }
  __device__ __forceinline__ f32x4 prior(const Row &xr, const Col &c) const {
    return *reinterpret_cast<const f32x4 *>(x + (uint32_t)(xr + c));
  }
  __device__ __forceinline__ void store(const Row &xr, int, const Col &c, f32x4 v) const {
    *reinterpret_cast<f32x4 *>(x + (uint32_t)(xr + c)) = v;
  }
};

template <typename T>
struct EpiGelu : PlainPrior {
  T *h;
  const float *bias;
  int n;
  using Row = int32_t;
  using Col = int32_t;
  __device__ __forceinline__ Row row(int r) const { return r; }
  __device__ __forceinline__ Col col(int c0) const { return c0; }
  __device__ __forceinline__ f32x4 bias4(int c0) const { return load_bias4(bias, c0); }
  __device__ __forceinline__ void store(const Row &, int r, const Col &c, f32x4 v) const {
    f32x4 g = {gelu_erf(v[0]), gelu_erf(v[1]), gelu_erf(v[2]), gelu_erf(v[3])};
    store4(h + (uint32_t)(r * n + c), g);
  }
};

// Plain epilogue of the sampler's GEMMs: out[r][c] = act(C + bias) stored
// row-major as T (ld = n), act the identity or SiLU.
template <typename T, bool SILU>
struct EpiPlain : PlainPrior {
  T *out;
  const float *bias;
  int n;
  using Row = int32_t;  // element offset of the output row (< 2^31, host-checked)
  using Col = int32_t;
  __device__ __forceinline__ Row row(int r) const { return r * n; }
  __device__ __forceinline__ Col col(int c0) const { return c0; }
  __device__ __forceinline__ f32x4 bias4(int c0) const { return load_bias4(bias, c0); }
  __device__ __forceinline__ void store(const Row &ro, int, const Col &c, f32x4 v) const {
    if constexpr (SILU) v = f32x4{silu(v[0]), silu(v[1]), silu(v[2]), silu(v[3])};
    store4(out + (uint32_t)(ro + c), v);
  }
};

// Second product of a sampler block: the gated residual h[r][c] += gate[r][c]
// (C + bias), h float32 (ld = n), the gate a slice of the modulation buffer
// (ld = mod_ld).
template <typename T>
struct EpiGate {
  static constexpr bool kPrior = true;
  struct Prior {
    f32x4 h;
    T g __attribute__((ext_vector_type(4)));
  };
  float *h;
  const float *bias;
  const T *gate;
  int n, mod_ld;
  using Row = int2;  // element offsets of the row in h and in the modulations (< 2^31)
  using Col = int32_t;
  __device__ __forceinline__ Row row(int r) const { return Row{r * n, r * mod_ld}; }
  __device__ __forceinline__ Col col(int c0) const { return c0; }
  __device__ __forceinline__ f32x4 bias4(int c0) const { return load_bias4(bias, c0); }
  __device__ __forceinline__ Prior prior(const Row &ro, const Col &c) const {
    Prior p;
    p.h = *reinterpret_cast<const f32x4 *>(h + (uint32_t)(ro.x + c));
    p.g = *reinterpret_cast<const decltype(p.g) *>(gate + (uint32_t)(ro.y + c));
    return p;
  }
  __device__ __forceinline__ f32x4 combine(f32x4 v, const Prior &p) const {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = fmaf((float)p.g[e], v[e], p.h[e]);
    return v;
  }
  __device__ __forceinline__ void store(const Row &ro, int, const Col &c, f32x4 v) const {
    *reinterpret_cast<f32x4 *>(h + (uint32_t)(ro.x + c)) = v;
  }
};

// Decoder embedding of the encoder rows (Eq. 2): encoder row r of image
// b = r / n_enc holds buffer token i = r % n_enc (i < n_buf) or the known
// image token known[b][i - n_buf]; its result goes to that token's sequence
// position j in the float32 decoder input x [batch][n_tokens][n], plus the
// decoder's positional embedding pe[j].
struct EpiEmbed : AddPrior {
  float *x;
  const float *bias;
  const float *pe;
  const int32_t *known;
  int n, n_enc, n_buf, n_known, n_tokens;
  struct Row {
    int32_t x_off;   // (b * n_tokens + j) * n
    int32_t pe_off;  // j * n
  };
  using Col = int32_t;
  __device__ __forceinline__ Row row(int r) const {
    const int b = r / n_enc, i = r - b * n_enc;
    const int j = i < n_buf ? i : n_buf + known[b * n_known + (i - n_buf)];
    return Row{(b * n_tokens + j) * n, j * n};
  }
  __device__ __forceinline__ Col col(int c0) const { return c0; }
  __device__ __forceinline__ f32x4 bias4(int c0) const { return load_bias4(bias, c0); }
  __device__ __forceinline__ f32x4 prior(const Row &ro, const Col &c) const {
    return *reinterpret_cast<const f32x4 *>(pe + (uint32_t)(ro.pe_off + c));
  }
  __device__ __forceinline__ void store(const Row &ro, int, const Col &c, f32x4 v) const {
    *reinterpret_cast<f32x4 *>(x + (uint32_t)(ro.x_off + c)) = v;
  }
};

// Empty uses that pin loaded values to this point: without them the compiler
// sinks the loads into the row-guarded store blocks, one wait per block.
__device__ __forceinline__ void keep(const f32x4 &v) { asm volatile("" ::"v"(v)); }
template <class P>
__device__ __forceinline__ auto keep(const P &p) -> decltype((void)p.h, (void)p.g) {
  asm volatile("" ::"v"(p.h), "v"(p.g));
}

// ------------------------------------------------------------------ bf16 MFMA
//
// The MFMA A operand is a 32-row slice of W (output columns) and the B
// operand a 32-row slice of the activations (output rows), so each 32x32
// accumulator holds a block of C^T: lane l owns output row (l & 31) and, in
// register r, output column (r / 4) * 8 + (l / 32) * 4 + r % 4 -- four
// consecutive columns per group of four registers, which the epilogue stores
// together.

// Grouped tile order: GROUP consecutive tile rows sweep all tile columns
// together, so concurrently running workgroups share A rows and W columns.
template <int GROUP = 8>
__device__ __forceinline__ void tile_coords(int id, int tiles_m, int tiles_n, int &tm, int &tn) {
  const int per_group = GROUP * tiles_n;
  const int g = id / per_group;
  const int first_m = g * GROUP;
  const int gm = min(tiles_m - first_m, GROUP);
  const int in = id - g * per_group;
  tm = first_m + in % gm;
  tn = in / gm;
}

// ------------------------------------------------------------------ 256x256 tile
//
// For projections where every token is active: a 256x256x64 workgroup tile
// on four wavefronts of 128x128 (16 accumulators each, which live in the
// accumulation registers).  Operands go from global memory straight into LDS
// (global_load_lds_dwordx4: no staging registers, no LDS write instructions)
// as 32 KB stages of 256 rows x 64 k, 128-byte rows whose 16-byte chunks are
// permuted by an XOR with the row pair index, so the 16 rows one fragment
// read touches per chunk hit 16 distinct bank groups.  The activation rows,
// streamed from memory once per column tile, get three stages and are loaded
// two k-tiles ahead of use; the weight rows, shared by every tile and served
// from L2, get two and are loaded one k-tile ahead: all of the CU's 160 KB.
// Every MFMA is issued in a fixed slot with at most one memory operation
// beside it (sched_barrier): the eight fragment reads of the next k16 step,
// the sixteen loads of a k-tile and the barrier are spread over the 64 MFMAs
// of a k-tile.
namespace big {

constexpr int kStage = 32768;  // bytes per operand stage: 256 rows x 64 k
constexpr int kAStages = 3, kWStages = 2;
constexpr int kWBase = kAStages * kStage;               // weight stages start at 96 KB
constexpr int kSmem = (kAStages + kWStages) * kStage;   // 160 KB

struct Frag {
  bf16x8 x[4];  // activation rows (MFMA B operand)
  bf16x8 w[4];  // weight rows (MFMA A operand)
};

__device__ __forceinline__ void pin() { __builtin_amdgcn_sched_barrier(0); }

__device__ __forceinline__ int swz(int r, int kc) { return kc ^ ((r >> 1) & 7); }

// Load instruction q (0..31 per operand and k-tile, 8 per wavefront) moves
// 1 KB: rows 8q..8q+7 of the operand's 256-row block; lane l writes LDS bytes
// [16 l, 16 l + 16) of it, i.e. row 8q + l / 8 at physical chunk l % 8, which
// holds logical chunk swz(row, l % 8).  `stage` is the LDS byte address of the
// stage (wave-uniform, so M0 is set from a scalar register).  Activation rows
// past M repeat row M - 1 (their results are never stored).
__device__ __forceinline__ void load_lds(unsigned stage, int q, const bf16 *src, int rows, int K,
                                         int r0, int k0, int lane) {
  const int r = q * 8 + (lane >> 3), pc = lane & 7;
  const bf16 *g = src + (size_t)min(r0 + r, rows - 1) * K + k0 + swz(r, pc) * 8;
  asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off"
               :
               : "v"(g), "s"(__builtin_amdgcn_readfirstlane(stage + q * 1024))
               : "memory", "m0");
}

// Fragment r of k16 step s, in the order the MFMAs need them: x0 w0 x1 x2 x3 w1 w2 w3.
__device__ __forceinline__ void read_frag(Frag &f, int r, const unsigned char *sa,
                                          const unsigned char *sw, int s, int wm, int wn,
                                          int lane) {
  const bool is_x = (r == 0 || r == 2 || r == 3 || r == 4);
  const int idx = r <= 1 ? 0 : (r <= 4 ? r - 1 : r - 4);
  const int kc = s * 2 + (lane >> 5);
  if (is_x) {
    const int row = wm * 128 + idx * 32 + (lane & 31);
    f.x[idx] = *reinterpret_cast<const bf16x8 *>(sa + row * 128 + swz(row, kc) * 16);
  } else {
    const int row = wn * 128 + idx * 32 + (lane & 31);
    f.w[idx] = *reinterpret_cast<const bf16x8 *>(sw + row * 128 + swz(row, kc) * 16);
  }
}

__device__ __forceinline__ void mfma(f32x16 (&acc)[4][4], const Frag &f, int q) {
  const int j = q >> 2, i = q & 3;
  acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.w[j], f.x[i], acc[j][i], 0, 0, 0);
}

// Own loads landed in LDS (all, or all but the last VM issued), own LDS reads
// done, then the workgroup barrier.
template <int VM>
__device__ __forceinline__ void barrier_vm() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(VM) : "memory");
}
__device__ __forceinline__ void barrier() { barrier_vm<0>(); }

}  // namespace big

// Write-back through LDS (free once the main loop is done).  In the
// accumulator layout a store instruction would write 16 bytes into each of
// 32 rows; instead each wavefront writes one 32-row block of its accumulators
// to LDS as fp32 and reads it back row-major, so one store instruction covers
// whole row segments (two rows of 128 columns, or four of 64).  Per-row
// addressing data of the tile were staged in LDS by the caller; residual
// priors of the next batch of rows are loaded before this batch's stores.
namespace big {
constexpr int kWbStride = 132;  // floats per staged row (128 + 4: no bank conflicts)
static_assert(4 * 32 * kWbStride * 4 <= kWBase, "staged write-back fits the activation stages");
}  // namespace big

// One wavefront's TM 32-row blocks of TN * 32 columns (accumulators acc[j][i]:
// column block j, row block i) starting at output row row0 and column col0.
// Each block goes through the wavefront's staging area `st` (32 rows of
// TN * 32 + 4 floats) and is read back with TN * 8 lanes per row, so lane l
// owns columns 4 (l % (8 TN)) .. + 3 of rows l / (8 TN) + (64 / (8 TN)) k.
// `rows` are the row records of rows row0.. (in LDS), `b` the bias of this
// lane's four columns.  Residual priors are loaded PB rows at a time, each
// batch before the stores of the previous one.
template <int TN, int TM, int PB, class Epi>
__device__ __forceinline__ void write_back_staged(const f32x16 (&acc)[TN][TM], const Epi &epi,
                                                  int row0, int col0, int M, int lane, float *st,
                                                  const typename Epi::Row *rows, f32x4 b) {
  constexpr int LPR = TN * 8;      // lanes per output row
  constexpr int RPP = 64 / LPR;    // rows per store instruction
  constexpr int KP = 32 / RPP;     // store instructions per 32-row block
  constexpr int STR = TN * 32 + 4; // staged row stride (floats): no bank conflicts
  static_assert(KP % PB == 0, "prior batches");
  constexpr int NB = KP / PB;      // batches per 32-row block
  const int c4 = (lane % LPR) * 4, rsub = lane / LPR, half = lane >> 5;
  const typename Epi::Col col = epi.col(col0 + c4);
  typename Epi::Prior pr[2][PB];  // unused by epilogues without a prior
  // batch u: block u / NB, rows rsub + RPP k for k in [(u % NB) PB, + PB)
  auto load_priors = [&](int u, typename Epi::Prior (&dst)[PB]) {
    const int i = u / NB, k0 = (u % NB) * PB;
#pragma unroll
    for (int k = 0; k < PB; ++k)
      if constexpr (Epi::kPrior) dst[k] = epi.prior(rows[i * 32 + rsub + RPP * (k0 + k)], col);
  };
  if constexpr (Epi::kPrior) load_priors(0, pr[0]);
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    // block row i of the accumulators -> LDS rows 0..31 of this wavefront
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<f32x4 *>(st + (lane & 31) * STR + j * 32 + g * 8 + half * 4) =
            f32x4{acc[j][i][4 * g + 0], acc[j][i][4 * g + 1], acc[j][i][4 * g + 2],
                  acc[j][i][4 * g + 3]};
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    const int rbase = row0 + i * 32;
    const bool full = rbase + 32 <= M;  // the whole block exists: no per-row guard
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int u = i * NB + nb;
      f32x4 v[PB];
#pragma unroll
      for (int k = 0; k < PB; ++k)
        v[k] = *reinterpret_cast<const f32x4 *>(st + (rsub + RPP * (nb * PB + k)) * STR + c4);
      if constexpr (Epi::kPrior) {
        if (u + 1 < TM * NB) load_priors(u + 1, pr[(u + 1) & 1]);
#pragma unroll
        for (int k = 0; k < PB; ++k) keep(pr[u & 1][k]);
      }
      auto value = [&](int k) -> f32x4 { return epi.combine(v[k] + b, pr[u & 1][k]); };
      if (full) {
#pragma unroll
        for (int k = 0; k < PB; ++k) {
          const int r = rsub + RPP * (nb * PB + k);
          epi.store(rows[i * 32 + r], rbase + r, col, value(k));
        }
      } else {
#pragma unroll
        for (int k = 0; k < PB; ++k) {
          const int r = rsub + RPP * (nb * PB + k);
          if (rbase + r < M) epi.store(rows[i * 32 + r], rbase + r, col, value(k));
        }
      }
    }
    // this block's reads of the staging rows are done before the next block
    // overwrites them
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  }
}

template <class Epi>
__global__ __launch_bounds__(256, 1) void gemm_bf16_big_kernel(const bf16 *A, const bf16 *W, int M,
                                                               int N, int K, Epi epi) {
  using namespace big;
  // activation stages at [0, 96K), weight stages at [96K, 160K); after the
  // main loop the write-back stages rows in [0, 66K) and keeps the tile's
  // biases and row records in the weight stage the last k-tile left free
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kSmem];
  static_assert(1024 + 256 * sizeof(typename Epi::Row) <= kStage, "row records fit one stage");
  const int tiles_m = (M + 255) / 256, tiles_n = N / 256;
  int tm, tn;
  tile_coords(xcd_remap(blockIdx.x, gridDim.x), tiles_m, tiles_n, tm, tn);
  const int m0 = tm * 256, n0 = tn * 256;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: scalar address math
  const int wm = wave >> 1, wn = wave & 1;
  const int q0 = wave * 8;  // this wavefront's load instructions q0 .. q0 + 7 of each operand
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)smem;
  f32x16 acc[4][4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[j][i] = f32x16{};
  const int nk = K / 64;
  auto load_a = [&](int sa, int kt, int p) {
    load_lds(lds0 + sa * kStage, q0 + p, A, M, K, m0, kt * 64, lane);
  };
  auto load_w = [&](int kt, int p) {
    load_lds(lds0 + kWBase + (kt & 1) * kStage, q0 + p, W, N, K, n0, kt * 64, lane);
  };

  // The write-back's bias (threads < 64, four columns each) and row record
  // (one row per thread), loaded first and kept in registers: they reach LDS
  // only after the main loop, so no wait on them holds up the pipeline.
  const typename Epi::Row rec = epi.row(min(m0 + tid, M - 1));
  const f32x4 bias = tid < 64 ? epi.bias4(n0 + tid * 4) : f32x4{};
  // k-tiles 0 and 1 of both operands, then wait for k-tile 0 only
#pragma unroll
  for (int p = 0; p < 8; ++p) load_a(0, 0, p);
#pragma unroll
  for (int p = 0; p < 8; ++p) load_w(0, p);
  if (nk > 1) {
#pragma unroll
    for (int p = 0; p < 8; ++p) load_a(1, 1, p);
#pragma unroll
    for (int p = 0; p < 8; ++p) load_w(1, p);
    barrier_vm<16>();
  } else {
    barrier();
  }
  Frag fa, fb;
#pragma unroll
  for (int r = 0; r < 8; ++r) read_frag(fa, r, smem, smem + kWBase, 0, wm, wn, lane);

  // activation stage of k-tiles kt, kt + 1, kt + 2 (kt mod 3, ...)
  int sa0 = 0, sa1 = 1, sa2 = 2;
  for (int kt = 0; kt + 1 < nk; ++kt) {
    const unsigned char *ac = smem + sa0 * kStage, *wc = smem + kWBase + (kt & 1) * kStage;
    const unsigned char *an = smem + sa1 * kStage, *wnx = smem + kWBase + ((kt + 1) & 1) * kStage;
    const bool a2 = kt + 2 < nk;  // k-tile kt+2 exists: its activation rows go out now
    // k16 steps 0..2: fragments of the next step; the second half of the
    // weight rows of k-tile kt+1 (the first went out at the end of k-tile
    // kt-1; k-tile 1 was loaded whole in the prologue), then the activation
    // rows of k-tile kt+2 into the stage k-tile kt-1 left
#pragma unroll
    for (int st = 0; st < 3; ++st) {
      Frag &fc = (st & 1) ? fb : fa;
      Frag &fn = (st & 1) ? fa : fb;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        mfma(acc, fc, q);
        if (q < 8) read_frag(fn, q, ac, wc, st + 1, wm, wn, lane);
        else if (st == 0 && q < 12 && kt > 0) load_w(kt + 1, 4 + (q - 8));
        else if (st == 0 && q >= 12 && a2) load_a(sa2, kt + 2, q - 12);
        else if (st == 1 && q < 12 && a2) load_a(sa2, kt + 2, 4 + (q - 8));
        pin();
      }
    }
    // k16 step 3: barrier (k-tile kt+1 complete -- only the activation loads
    // of k-tile kt+2 may still be in flight -- and every wavefront done with
    // k-tile kt), first fragments of k-tile kt+1, first half of the weight
    // rows of k-tile kt+2 into the weight stage of k-tile kt
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      mfma(acc, fb, q);
      pin();
    }
    if (a2) barrier_vm<8>();
    else barrier();
    pin();
#pragma unroll
    for (int q = 4; q < 12; ++q) {
      mfma(acc, fb, q);
      read_frag(fa, q - 4, an, wnx, 0, wm, wn, lane);
      pin();
    }
#pragma unroll
    for (int q = 12; q < 16; ++q) {
      mfma(acc, fb, q);
      if (a2) load_w(kt + 2, q - 12);
      pin();
    }
    const int t = sa0;
    sa0 = sa1;
    sa1 = sa2;
    sa2 = t;
  }
  {  // last k-tile: no loads in flight
    const unsigned char *ac = smem + sa0 * kStage, *wc = smem + kWBase + ((nk - 1) & 1) * kStage;
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      Frag &fc = (st & 1) ? fb : fa;
      Frag &fn = (st & 1) ? fa : fb;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        mfma(acc, fc, q);
        if (st < 3 && q < 8) read_frag(fn, q, ac, wc, st + 1, wm, wn, lane);
        pin();
      }
    }
  }
  // the write-back's biases and row records into the weight stage that the
  // last k-tile does not read (no wavefront reads it after the last
  // k-tile's barrier); then every wavefront is done with the stages before
  // they hold the write-back's staging rows
  unsigned char *side = smem + kWBase + (nk & 1) * kStage;
  if (tid < 64) *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(side) + tid * 4) = bias;
  reinterpret_cast<typename Epi::Row *>(side + 1024)[tid] = rec;
  barrier();
  const f32x4 b = *reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(side) +
                                                    wn * 128 + (lane & 31) * 4);
  write_back_staged<4, 4, 16>(acc, epi, m0 + wm * 128, n0 + wn * 128, M, lane,
                           reinterpret_cast<float *>(smem) + wave * 32 * kWbStride,
                           reinterpret_cast<const typename Epi::Row *>(side + 1024) + wm * 128, b);
}

// ------------------------------------------------------------------ 256x256 tile, eight wavefronts
//
// The 256x256x64 tile of gemm_bf16_big_kernel (same LDS stages, swizzle,
// direct-to-LDS loads and stage schedule) on eight wavefronts of 128x64 (8
// accumulator blocks, 128 accumulation registers each), two per SIMD: while
// one wavefront of a SIMD waits on a fragment read, a barrier or its
// write-back's LDS round trip, the other can issue MFMAs.  Per k16 step a
// wavefront reads 6 fragments for 8 MFMAs (4 activation and 2 weight
// fragments), 1.5 times the LDS reads per MFMA of the 128x128 wavefront tile.
namespace big8 {

struct Frag {
  bf16x8 x[4];  // activation rows (MFMA B operand)
  bf16x8 w[2];  // weight rows (MFMA A operand)
};

// Fragment r of k16 step s, in the order the MFMAs need them: x0 w0 x1 x2 x3 w1.
__device__ __forceinline__ void read_frag(Frag &f, int r, const unsigned char *sa,
                                          const unsigned char *sw, int s, int wm, int wn,
                                          int lane) {
  const int kc = s * 2 + (lane >> 5);
  if (r == 1 || r == 5) {
    const int idx = r == 1 ? 0 : 1;
    const int row = wn * 64 + idx * 32 + (lane & 31);
    f.w[idx] = *reinterpret_cast<const bf16x8 *>(sw + row * 128 + big::swz(row, kc) * 16);
  } else {
    const int idx = r == 0 ? 0 : r - 1;
    const int row = wm * 128 + idx * 32 + (lane & 31);
    f.x[idx] = *reinterpret_cast<const bf16x8 *>(sa + row * 128 + big::swz(row, kc) * 16);
  }
}

__device__ __forceinline__ void mfma(f32x16 (&acc)[2][4], const Frag &f, int q) {
  const int j = q >> 2, i = q & 3;
  acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.w[j], f.x[i], acc[j][i], 0, 0, 0);
}

}  // namespace big8

template <class Epi>
__global__ __launch_bounds__(512, 1) void gemm_bf16_big8_kernel(const bf16 *A, const bf16 *W,
                                                                int M, int N, int K, Epi epi) {
  using namespace big;
  // LDS as in gemm_bf16_big_kernel; the write-back stages 8 x 32 rows of 68
  // floats in [0, 70 KB)
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kSmem];
  static_assert(1024 + 256 * sizeof(typename Epi::Row) <= kStage, "row records fit one stage");
  static_assert(8 * 32 * 68 * 4 <= kWBase, "staged write-back fits the activation stages");
  const int tiles_m = (M + 255) / 256, tiles_n = N / 256;
  int tm, tn;
  tile_coords(xcd_remap(blockIdx.x, gridDim.x), tiles_m, tiles_n, tm, tn);
  const int m0 = tm * 256, n0 = tn * 256;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const int q0 = wave * 4;  // this wavefront's load instructions q0 .. q0 + 3 of each operand
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)smem;
  f32x16 acc[2][4];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[j][i] = f32x16{};
  const int nk = K / 64;
  auto load_a = [&](int sa, int kt, int p) {
    load_lds(lds0 + sa * kStage, q0 + p, A, M, K, m0, kt * 64, lane);
  };
  auto load_w = [&](int kt, int p) {
    load_lds(lds0 + kWBase + (kt & 1) * kStage, q0 + p, W, N, K, n0, kt * 64, lane);
  };

  const typename Epi::Row rec = epi.row(min(m0 + (tid & 255), M - 1));
  const f32x4 bias = tid < 64 ? epi.bias4(n0 + tid * 4) : f32x4{};
  // k-tiles 0 and 1 of both operands, then wait for k-tile 0 only
#pragma unroll
  for (int p = 0; p < 4; ++p) load_a(0, 0, p);
#pragma unroll
  for (int p = 0; p < 4; ++p) load_w(0, p);
  if (nk > 1) {
#pragma unroll
    for (int p = 0; p < 4; ++p) load_a(1, 1, p);
#pragma unroll
    for (int p = 0; p < 4; ++p) load_w(1, p);
    barrier_vm<8>();
  } else {
    barrier();
  }
  big8::Frag fa, fb;
#pragma unroll
  for (int r = 0; r < 6; ++r) big8::read_frag(fa, r, smem, smem + kWBase, 0, wm, wn, lane);

  int sa0 = 0, sa1 = 1, sa2 = 2;
  for (int kt = 0; kt + 1 < nk; ++kt) {
    const unsigned char *ac = smem + sa0 * kStage, *wc = smem + kWBase + (kt & 1) * kStage;
    const unsigned char *an = smem + sa1 * kStage, *wnx = smem + kWBase + ((kt + 1) & 1) * kStage;
    const bool a2 = kt + 2 < nk;
    // k16 steps 0..2: the fragments of the next step, then two loads: the
    // second half of the weight rows of k-tile kt+1 (step 0; k-tile 1 was
    // loaded whole in the prologue), the activation rows of k-tile kt+2 into
    // the stage k-tile kt-1 left (steps 1 and 2)
#pragma unroll
    for (int st = 0; st < 3; ++st) {
      big8::Frag &fc = (st & 1) ? fb : fa;
      big8::Frag &fn = (st & 1) ? fa : fb;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        big8::mfma(acc, fc, q);
        if (q < 6) big8::read_frag(fn, q, ac, wc, st + 1, wm, wn, lane);
        else if (st == 0 && kt > 0) load_w(kt + 1, 2 + (q - 6));
        else if (st > 0 && a2) load_a(sa2, kt + 2, (st - 1) * 2 + (q - 6));
        pin();
      }
    }
    // k16 step 3: barrier (k-tile kt+1 complete -- only the activation loads
    // of k-tile kt+2 may still be in flight -- and every wavefront done with
    // k-tile kt), the first fragments of k-tile kt+1, the first half of the
    // weight rows of k-tile kt+2 into the weight stage of k-tile kt
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      big8::mfma(acc, fb, q);
      pin();
    }
    if (a2) barrier_vm<4>();
    else barrier();
    pin();
#pragma unroll
    for (int q = 2; q < 8; ++q) {
      big8::mfma(acc, fb, q);
      big8::read_frag(fa, q - 2, an, wnx, 0, wm, wn, lane);
      if (q >= 6 && a2) load_w(kt + 2, q - 6);
      pin();
    }
    const int t = sa0;
    sa0 = sa1;
    sa1 = sa2;
    sa2 = t;
  }
  {  // last k-tile: no loads in flight
    const unsigned char *ac = smem + sa0 * kStage, *wc = smem + kWBase + ((nk - 1) & 1) * kStage;
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      big8::Frag &fc = (st & 1) ? fb : fa;
      big8::Frag &fn = (st & 1) ? fa : fb;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        big8::mfma(acc, fc, q);
        if (st < 3 && q < 6) big8::read_frag(fn, q, ac, wc, st + 1, wm, wn, lane);
        pin();
      }
    }
  }
  unsigned char *side = smem + kWBase + (nk & 1) * kStage;
  if (tid < 64) *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(side) + tid * 4) = bias;
  if (tid < 256) reinterpret_cast<typename Epi::Row *>(side + 1024)[tid] = rec;
  barrier();
  const f32x4 b = *reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(side) +
                                                    wn * 64 + (lane & 15) * 4);
  write_back_staged<2, 4, 4>(acc, epi, m0 + wm * 128, n0 + wn * 64, M, lane,
                             reinterpret_cast<float *>(smem) + wave * 32 * 68,
                             reinterpret_cast<const typename Epi::Row *>(side + 1024) + wm * 128, b);
}

// ------------------------------------------------------------------ 320x256 tile, eight wavefronts
//
// A 320x256x64 workgroup tile for products over whole images of 320 tokens:
// one tile row is one image, so a range of b images has b tile rows and a
// product with N = 1024 runs b * 4 tiles -- exactly one wave of 256 compute
// units for a 64-image range, where 256x256 tiles make 320 (1.25 waves) --
// and N = 3072 / 4096 three / four whole waves.  Eight wavefronts of 160x64
// (2 x 5 accumulator blocks, 160 accumulation registers each; two wavefronts
// share a SIMD), the 256x256 tile's 128-byte swizzled rows and direct-to-LDS
// loads, two 40 KB activation stages and two 32 KB weight stages (144 KB).
// A k-tile's activation rows go out right after the barrier that frees their
// stage, one k-tile ahead of use; its weight rows, which the L2 serves, beside
// the first MFMAs of the next k-tile.  Per k16 step a wavefront reads 7 fragments for 10
// MFMAs (5 activation, 2 weight).  Accumulation is the same chain of k16
// steps in ascending order as every other tile, so results are bitwise
// those of the 256x256 tile.
namespace t320 {

constexpr int kBM = 320;
constexpr int kAStage = kBM * 128;      // 40 KB: 320 rows x 64 k
constexpr int kWStage = 256 * 128;      // 32 KB
constexpr int kWBase = 2 * kAStage;     // weight stages start at 80 KB
constexpr int kSmem = kWBase + 2 * kWStage;  // 144 KB
constexpr int kALoads = kBM / 8 / 8;    // 1 KB load instructions per wavefront per k-tile: 5
constexpr int kWLoads = 256 / 8 / 8;    // 4
constexpr int kLoads = kALoads + kWLoads;
constexpr int kWbStride = 68;           // floats per staged row (64 + 4)
static_assert(8 * 32 * kWbStride * 4 <= kWBase, "staged write-back fits the activation stages");

// One set of fragments, refilled as the MFMAs of a k16 step release them.
struct Frag {
  bf16x8 x[5];  // activation rows (MFMA B operand)
  bf16x8 w[2];  // weight rows (MFMA A operand)
};

// Fragment r (0..4: activation row block r; 5, 6: weight row block r - 5) of
// k16 step s from a stage pair.
__device__ __forceinline__ void read_frag(Frag &f, int r, const unsigned char *sa,
                                          const unsigned char *sw, int s, int wm, int wn,
                                          int lane) {
  const int kc = s * 2 + (lane >> 5);
  if (r >= 5) {
    const int row = wn * 64 + (r - 5) * 32 + (lane & 31);
    f.w[r - 5] = *reinterpret_cast<const bf16x8 *>(sw + row * 128 + big::swz(row, kc) * 16);
  } else {
    const int row = wm * 160 + r * 32 + (lane & 31);
    f.x[r] = *reinterpret_cast<const bf16x8 *>(sa + row * 128 + big::swz(row, kc) * 16);
  }
}

// MFMA q of a k16 step: column block q / 5, row block q % 5.
__device__ __forceinline__ void mfma(f32x16 (&acc)[2][5], const Frag &f, int q) {
  const int j = q / 5, i = q % 5;
  acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.w[j], f.x[i], acc[j][i], 0, 0, 0);
}

// 1 KB of an operand into LDS at `lds` (wave-uniform): the scalar base is the
// operand at the k-tile's first column, `off` the lane's byte offset from it
// (32-bit: the host keeps every operand below 2^31 elements).
__device__ __forceinline__ void load_lds(unsigned lds, const bf16 *base, uint32_t off) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(off), "s"(base), "s"(__builtin_amdgcn_readfirstlane(lds))
               : "memory", "m0");
}

}  // namespace t320

template <class Epi>
__global__ __launch_bounds__(512, 1) void gemm_bf16_t320_kernel(const bf16 *A, const bf16 *W,
                                                                 int M, int N, int K, Epi epi) {
  using namespace t320;
  // activation stages at [0, 80K), weight stages at [80K, 144K); after the
  // main loop the write-back stages rows in [0, 68K) and keeps the tile's
  // biases and row records in the weight stage the last k-tile left free
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kSmem];
  static_assert(1024 + kBM * sizeof(typename Epi::Row) <= kWStage, "row records fit one stage");
  const int tiles_m = (M + kBM - 1) / kBM, tiles_n = N / 256;
  int tm, tn;
  // groups of 4 tile rows: an XCD's 32 concurrent tiles cover 4 rows x 8
  // columns (QKV 117 -> 114.5 us per range against groups of 8, with about
  // the same L2 fetch bytes)
  tile_coords<4>(xcd_remap(blockIdx.x, gridDim.x), tiles_m, tiles_n, tm, tn);
  const int m0 = tm * kBM, n0 = tn * 256;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)smem;
  f32x16 acc[2][5];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < 5; ++i) acc[j][i] = f32x16{};
  const int nk = K / 64;
  // This wavefront's load p of every k-tile: p < 5 moves activation rows
  // 8 q .. 8 q + 7 (q = 5 wave + p of the tile's 40 blocks), p >= 5 weight
  // rows (q = 4 wave + p - 5 of 32); lane l writes row 8 q + l / 8 at
  // physical chunk l % 8, which holds logical chunk swz(row, l % 8).
  // Activation rows past M repeat row M - 1 (their results are never stored).
  uint32_t off[kLoads];
#pragma unroll
  for (int p = 0; p < kLoads; ++p) {
    const bool is_a = p < kALoads;
    const int q = is_a ? wave * kALoads + p : wave * kWLoads + (p - kALoads);
    const int r = q * 8 + (lane >> 3);
    const int row = is_a ? min(m0 + r, M - 1) : n0 + r;
    off[p] = (uint32_t)(row * K + big::swz(r, lane & 7) * 8) * 2u;
  }
  auto load = [&](int kt, int p) {
    const int s = kt & 1;
    if (p < kALoads)
      load_lds(lds0 + s * kAStage + (wave * kALoads + p) * 1024, A + kt * 64, off[p]);
    else
      load_lds(lds0 + kWBase + s * kWStage + (wave * kWLoads + p - kALoads) * 1024, W + kt * 64,
               off[p]);
  };

  const typename Epi::Row rec = epi.row(min(m0 + min(tid, kBM - 1), M - 1));
  const f32x4 bias = tid < 64 ? epi.bias4(n0 + tid * 4) : f32x4{};
  // k-tiles 0 and 1, then wait for k-tile 0 only
#pragma unroll
  for (int p = 0; p < kLoads; ++p) load(0, p);
  if (nk > 1) {
#pragma unroll
    for (int p = 0; p < kLoads; ++p) load(1, p);
    big::barrier_vm<kLoads>();
  } else {
    big::barrier();
  }
  // Per k16 step: MFMA q uses weight block q / 5 and activation block q % 5.
  // The step's own x4 and w1 are read beside MFMAs 0 and 1 (their previous
  // values are last used by MFMA 9 of the step before); beside MFMAs 5..9
  // the next step's w0, x0, x1, x2, x3 replace the ones MFMAs 4..8 used last.
  Frag f;
  read_frag(f, 5, smem, smem + kWBase, 0, wm, wn, lane);
#pragma unroll
  for (int r = 0; r < 4; ++r) read_frag(f, r, smem, smem + kWBase, 0, wm, wn, lane);
  constexpr int kNext[5] = {5, 0, 1, 2, 3};  // fragment read beside MFMA 5 + i

  for (int kt = 0; kt + 1 < nk; ++kt) {
    const int c = kt & 1, n = c ^ 1;
    const unsigned char *ac = smem + c * kAStage, *wc = smem + kWBase + c * kWStage;
    const unsigned char *an = smem + n * kAStage, *wnx = smem + kWBase + n * kWStage;
    const bool more = kt + 2 < nk;  // k-tile kt+2 exists
#pragma unroll
    for (int st = 0; st < 4; ++st) {
#pragma unroll
      for (int q = 0; q < 10; ++q) {
        t320::mfma(acc, f, q);
        if (q == 0) read_frag(f, 4, ac, wc, st, wm, wn, lane);
        if (q == 1) read_frag(f, 6, ac, wc, st, wm, wn, lane);
        // loads 5..8 of k-tile kt+1 (loads 0..4 went out in the step 3 of
        // k-tile kt-1; k-tile 1 was loaded whole in the prologue)
        if (kt > 0 && st == 0 && q >= 2 && q <= 4) load(kt + 1, kALoads + q - 2);
        if (kt > 0 && st == 1 && q == 2) load(kt + 1, kLoads - 1);
        // step 3: barrier (k-tile kt+1 landed, every wavefront done with
        // k-tile kt), then the next k-tile's first fragments and loads 0..4
        // of k-tile kt+2 into the stages k-tile kt leaves
        if (st == 3 && q == 4) big::barrier();
        if (q >= 5) {
          if (st < 3) read_frag(f, kNext[q - 5], ac, wc, st + 1, wm, wn, lane);
          else read_frag(f, kNext[q - 5], an, wnx, 0, wm, wn, lane);
          if (st == 3 && more) load(kt + 2, q - 5);
        }
        big::pin();
      }
    }
  }
  {  // last k-tile: no loads in flight
    const int c = (nk - 1) & 1;
    const unsigned char *ac = smem + c * kAStage, *wc = smem + kWBase + c * kWStage;
#pragma unroll
    for (int st = 0; st < 4; ++st) {
#pragma unroll
      for (int q = 0; q < 10; ++q) {
        t320::mfma(acc, f, q);
        if (q == 0) read_frag(f, 4, ac, wc, st, wm, wn, lane);
        if (q == 1) read_frag(f, 6, ac, wc, st, wm, wn, lane);
        if (st < 3 && q >= 5) read_frag(f, kNext[q - 5], ac, wc, st + 1, wm, wn, lane);
        big::pin();
      }
    }
  }
  unsigned char *side = smem + kWBase + (nk & 1) * kWStage;
  if (tid < 64) *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(side) + tid * 4) = bias;
  if (tid < kBM) reinterpret_cast<typename Epi::Row *>(side + 1024)[tid] = rec;
  big::barrier();
  const f32x4 b = *reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(side) +
                                                    wn * 64 + (lane & 15) * 4);
  write_back_staged<2, 5, 4>(acc, epi, m0 + wm * 160, n0 + wn * 64, M, lane,
                             reinterpret_cast<float *>(smem) + wave * 32 * kWbStride,
                             reinterpret_cast<const typename Epi::Row *>(side + 1024) + wm * 160, b);
}

// ------------------------------------------------------------------ 64 TM x 128 tiles
//
// For products that leave 256x256 tiles a partial wave (the narrow products of
// cache-aware layers, N = d_model on a few thousand active rows; every product
// of a small batch): tiles of 64 TM x 128 x 64 on four wavefronts of 32 TM x 64
// (2 TM accumulator blocks), one workgroup per CU.  Operand stages use the
// 256x256 tile's 128-byte rows, XOR swizzle and direct-to-LDS loads with a
// scalar base.  Alone, the loads of a 128x128 tile take 0.65 and its fragment
// reads and MFMAs 0.7 of the time that a loop issuing them in bursts took, so
// the loop spreads all three: beside each MFMA at most one or two memory
// operations, fragments read two k16 steps before use (four register sets),
// a k-tile's loads over the whole of the k-tile before, and one barrier per
// k-tile that waits for the next k-tile's loads only (the stage it frees was
// read a k-tile earlier).
// No split of K: every output is one accumulation over all of K in
// ascending k16 steps, as in every other tile, so the result does not depend
// on which tile a shape gets.
namespace mid {

constexpr int kBN = 128, kBK = 64;

template <int TM>
struct Shape {
  static constexpr int kBM = 64 * TM;
  static constexpr int kWOff = kBM * kBK * 2;              // weight rows after the activation rows
  static constexpr int kStage = (kBM + kBN) * kBK * 2;
  static constexpr int kALoads = 2 * TM, kLoads = kALoads + 4;  // 1 KB each, per wavefront
};

template <int TM>
struct Frag {
  bf16x8 x[TM];  // activation rows (MFMA B operand)
  bf16x8 w[2];   // weight rows (MFMA A operand)
};

// Fragment r of k16 step s of a stage, in the order the MFMAs need them: w0,
// x0 .. x(TM-1), w1.
template <int TM>
__device__ __forceinline__ void read_frag(Frag<TM> &f, int r, const unsigned char *stage, int s,
                                          int wm, int wn, int lane) {
  const int kc = s * 2 + (lane >> 5);
  if (r == 0 || r == TM + 1) {
    const int j = r == 0 ? 0 : 1;
    const int row = wn * 64 + j * 32 + (lane & 31);
    f.w[j] = *reinterpret_cast<const bf16x8 *>(stage + Shape<TM>::kWOff + row * 128 +
                                               big::swz(row, kc) * 16);
  } else {
    const int row = wm * 32 * TM + (r - 1) * 32 + (lane & 31);
    f.x[r - 1] = *reinterpret_cast<const bf16x8 *>(stage + row * 128 + big::swz(row, kc) * 16);
  }
}

// At most n (<= NMAX) of this wavefront's k-tiles of L loads in flight, then
// the workgroup barrier.
template <int L, int NMAX>
__device__ __forceinline__ void barrier_tiles(int n) {
  if constexpr (NMAX > 0) {
    if (n < NMAX) {
      barrier_tiles<L, NMAX - 1>(n);
      return;
    }
  }
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(L * NMAX) : "memory");
}

}  // namespace mid

template <class Epi, int TM, int NS>
__global__ __launch_bounds__(256, 1) void gemm_bf16_mid_kernel(const bf16 *A, const bf16 *W, int M,
                                                               int N, int K, Epi epi) {
  using namespace mid;
  using big::pin;
  using Row = typename Epi::Row;
  using S = Shape<TM>;
  static_assert(NS >= 3 && S::kLoads * (NS - 1) <= 63, "stages; vmcnt holds 63");
  // after the main loop the write-back stages 4 x 32 rows of 68 floats and
  // keeps the tile's row records behind them
  __shared__ __attribute__((aligned(1024))) unsigned char smem[NS * S::kStage];
  constexpr int kRowsOff = 4 * 32 * 68 * 4;
  static_assert(kRowsOff + S::kBM * sizeof(Row) <= NS * S::kStage, "row records fit the stages");
  const int tiles_m = (M + S::kBM - 1) / S::kBM, tiles_n = N / kBN;
  int tm, tn;
  tile_coords(xcd_remap(blockIdx.x, gridDim.x), tiles_m, tiles_n, tm, tn);
  const int m0 = tm * S::kBM, n0 = tn * kBN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)smem;
  const unsigned char *smem_u = smem;
  f32x16 acc[2][TM];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < TM; ++i) acc[j][i] = f32x16{};
  const int nk = K / kBK;
  // Load p of every k-tile: p < kALoads moves activation rows 8 q .. 8 q + 7
  // (q = kALoads wave + p), the rest weight rows; lane l writes row 8 q + l / 8
  // at physical chunk l % 8, which holds logical chunk swz(row, l % 8).
  // Activation rows past M repeat row M - 1 (their results are never stored).
  uint32_t off[S::kLoads];
#pragma unroll
  for (int p = 0; p < S::kLoads; ++p) {
    const bool is_a = p < S::kALoads;
    const int q = is_a ? wave * S::kALoads + p : wave * 4 + (p - S::kALoads);
    const int r = q * 8 + (lane >> 3);
    const int row = is_a ? min(m0 + r, M - 1) : n0 + r;
    off[p] = ((uint32_t)row * (uint32_t)K + (uint32_t)(big::swz(r, lane & 7) * 8)) * 2u;
  }
  auto load = [&](int st, int t, int p) {
    const unsigned sb = lds0 + (unsigned)st * S::kStage;
    if (p < S::kALoads)
      t320::load_lds(sb + (wave * S::kALoads + p) * 1024, A + t * kBK, off[p]);
    else
      t320::load_lds(sb + S::kWOff + (wave * 4 + p - S::kALoads) * 1024, W + t * kBK, off[p]);
  };

  // the write-back's row record and this lane's bias, kept in registers until
  // after the main loop
  Row rec[(S::kBM + 255) / 256];
#pragma unroll
  for (int u = 0; u < (S::kBM + 255) / 256; ++u)
    rec[u] = epi.row(min(m0 + min(tid + 256 * u, S::kBM - 1), M - 1));
  const f32x4 bias = epi.bias4(n0 + wn * 64 + (lane & 15) * 4);

  // k-tiles 0 .. NS-2 in flight, then wait for k-tile 0
#pragma unroll
  for (int t = 0; t < NS - 1; ++t)
    if (t < nk) {
#pragma unroll
      for (int p = 0; p < S::kLoads; ++p) load(t, t, p);
    }
  barrier_tiles<S::kLoads, NS - 2>(min(NS - 1, nk) - 1);
  Frag<TM> f[4];
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int r = 0; r < TM + 2; ++r) read_frag<TM>(f[s], r, smem_u, s, wm, wn, lane);

  constexpr int MF = 2 * TM;  // MFMAs per k16 step
  int cur = 0, nxt = 1, prv = NS - 1;  // stages of k-tiles t, t + 1, t - 1
  for (int t = 0; t < nk; ++t) {
    const unsigned char *sc = smem_u + cur * S::kStage, *sn = smem_u + nxt * S::kStage;
    const bool more = t + 1 < nk, ld = t + NS - 1 < nk;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      // k-tile t+1 landed before its fragments are read; of the k-tiles issued
      // so far, t + 2 .. t + NS - 2 may still be on their way
      if (s == 2 && more) {
        barrier_tiles<S::kLoads, NS - 3>(min(NS - 3, nk - 2 - t));
        pin();
      }
#pragma unroll
      for (int q = 0; q < MF; ++q) {
        const int j = q / TM, i = q % TM;
        acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[s].w[j], f[s].x[i], acc[j][i], 0, 0, 0);
        // fragments of two steps on, TM + 2 over the step's MFMAs
#pragma unroll
        for (int r = q * (TM + 2) / MF; r < (q + 1) * (TM + 2) / MF; ++r) {
          if (s < 2) read_frag<TM>(f[s + 2], r, sc, s + 2, wm, wn, lane);
          else if (more) read_frag<TM>(f[s - 2], r, sn, s - 2, wm, wn, lane);
        }
        // k-tile t + NS - 1 into the stage of k-tile t - 1, which every
        // wavefront has read before the barrier: steps 2 and 3
        if (s >= 2 && ld) {
          const int u = (s - 2) * MF + q;
#pragma unroll
          for (int p = u * S::kLoads / (2 * MF); p < (u + 1) * S::kLoads / (2 * MF); ++p)
            load(prv, t + NS - 1, p);
        }
        pin();
      }
    }
    prv = cur;
    cur = nxt;
    nxt = nxt + 1 == NS ? 0 : nxt + 1;
  }
  // every wavefront is done with the stages before the row records and the
  // staged rows overwrite them
  big::barrier_vm<0>();
  Row *rows_lds = reinterpret_cast<Row *>(smem + kRowsOff);
#pragma unroll
  for (int u = 0; u < (S::kBM + 255) / 256; ++u)
    if (tid + 256 * u < S::kBM) rows_lds[tid + 256 * u] = rec[u];
  big::barrier_vm<0>();
  write_back_staged<2, TM, 8>(acc, epi, m0 + wm * 32 * TM, n0 + wn * 64, M, lane,
                              reinterpret_cast<float *>(smem) + wave * 32 * 68,
                              rows_lds + wm * 32 * TM, bias);
}

// ------------------------------------------------------------------ 64x128 tile
//
// For products of several hundred rows that larger tiles would not spread over
// the chip (the sampler's block products on 512 rows): a 64x128x128 tile on
// four wavefronts of 32x64 (2 accumulator blocks).  With so little work per
// workgroup its time is the serial chain of k-tiles (barrier, LDS round trip,
// dependent MFMAs), not bandwidth, so the k-tile is long: three 48 KB stages
// of 256-byte rows (16-byte chunks XOR-permuted by the row's low four bits,
// so 16 rows read at one chunk hit 16 distinct bank groups), one barrier per
// 128 of K, the next k16 step's fragments read while the current one's MFMAs
// run, and the loads of k-tile t+3 issued once every wavefront is done with
// k-tile t.
namespace small {

constexpr int kBM = 64, kBN = 128, kBK = 128;
constexpr int kRow = kBK * 2;                  // 256-byte rows
constexpr int kWOff = kBM * kRow;              // weight rows start 16 KB into a stage
constexpr int kStage = (kBM + kBN) * kRow;     // 48 KB
constexpr int kLoads = kStage / 1024 / 4;      // load instructions per wavefront per k-tile
static_assert(kLoads == 12, "load count per wavefront");

__device__ __forceinline__ int swz(int r, int c) { return c ^ (r & 15); }

struct Frag {
  bf16x8 x;     // activation rows (MFMA B operand)
  bf16x8 w[2];  // weight rows (MFMA A operand)
};

// Load instruction q (0..47 per k-tile) moves 1 KB = four 256-byte rows:
// q < 16 carries activation rows 4q..4q+3, q >= 16 weight rows 4(q-16)..;
// lane l writes LDS bytes [16 l, 16 l + 16): row 4 q' + l / 16 at physical
// chunk l % 16.
__device__ __forceinline__ void load_lds(unsigned stage, int q, const bf16 *A, const bf16 *W,
                                         int M, int K, int m0, int n0, int k0, int lane) {
  const int rr = lane >> 4, pc = lane & 15;
  const bf16 *g;
  if (q < 16) {
    const int r = q * 4 + rr;
    g = A + (size_t)min(m0 + r, M - 1) * K + k0 + swz(r, pc) * 8;
  } else {
    const int r = (q - 16) * 4 + rr;
    g = W + (size_t)(n0 + r) * K + k0 + swz(r, pc) * 8;
  }
  asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off"
               :
               : "v"(g), "s"(__builtin_amdgcn_readfirstlane(stage + q * 1024))
               : "memory", "m0");
}

// Fragments of k16 step s (0..7) of a stage.
__device__ __forceinline__ void read_frags(Frag &f, const unsigned char *stage, int s, int wm,
                                           int wn, int lane) {
  const int c = 2 * s + (lane >> 5);
  const int xr = wm * 32 + (lane & 31);
  f.x = *reinterpret_cast<const bf16x8 *>(stage + xr * kRow + swz(xr, c) * 16);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int wr = wn * 64 + j * 32 + (lane & 31);
    f.w[j] = *reinterpret_cast<const bf16x8 *>(stage + kWOff + wr * kRow + swz(wr, c) * 16);
  }
}

__device__ __forceinline__ void mfma(f32x16 (&acc)[2][1], const Frag &f) {
#pragma unroll
  for (int j = 0; j < 2; ++j)
    acc[j][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.w[j], f.x, acc[j][0], 0, 0, 0);
}

}  // namespace small

// One tile of an M x N x K product; `smem` holds three stages, `rows` kBM row records.
template <class Epi>
__device__ __forceinline__ void small_tile(const bf16 *A, const bf16 *W, int M, int N, int K,
                                           const Epi &epi, int id, unsigned char *smem,
                                           typename Epi::Row *rows_lds) {
  using namespace small;
  using big::barrier_vm;
  using big::pin;
  using Row = typename Epi::Row;
  constexpr int kStr = 2 * 32 + 4;  // staged write-back row (floats)
  static_assert(4 * 32 * kStr * 4 <= 3 * kStage, "staged write-back fits the stages");
  const int tiles_m = (M + kBM - 1) / kBM, tiles_n = N / kBN;
  int tm, tn;
  tile_coords(id, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * kBM, n0 = tn * kBN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int q0 = wave * kLoads;
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)smem;
  const unsigned char *smem_u = smem;
  f32x16 acc[2][1] = {{f32x16{}}, {f32x16{}}};
  const int nk = K / kBK;
  auto load_tile = [&](unsigned st, int t) {
#pragma unroll
    for (int p = 0; p < kLoads; ++p) load_lds(st, q0 + p, A, W, M, K, m0, n0, t * kBK, lane);
  };

  // the write-back's row record (threads < 64) and this lane's bias, kept in
  // registers until after the main loop
  Row rec{};
  if (tid < kBM) rec = epi.row(min(m0 + tid, M - 1));
  const f32x4 bias = epi.bias4(n0 + wn * 64 + (lane & 15) * 4);

  // k-tiles 0, 1 and 2 (as far as they exist)
  unsigned s0 = lds0, s1 = lds0 + kStage, s2 = lds0 + 2 * kStage;
  load_tile(s0, 0);
  if (nk > 1) load_tile(s1, 1);
  if (nk > 2) load_tile(s2, 2);
  if (nk > 2) barrier_vm<2 * kLoads>();
  else if (nk > 1) barrier_vm<kLoads>();
  else barrier_vm<0>();
  Frag f[2];
  read_frags(f[0], smem_u + (s0 - lds0), 0, wm, wn, lane);

  for (int t = 0; t < nk; ++t) {
    // s0: k-tile t (f[0] holds its step-0 fragments); s1, s2: k-tiles t+1, t+2
    const unsigned char *sc = smem_u + (s0 - lds0);
#pragma unroll
    for (int st = 0; st < 7; ++st) {
      read_frags(f[(st + 1) & 1], sc, st + 1, wm, wn, lane);
      mfma(acc, f[st & 1]);
      pin();
    }
    if (t + 1 < nk) {
      // k-tile t+1 complete (k-tile t+2 may still be in flight) and k-tile t
      // read by every wavefront
      if (t + 2 < nk) barrier_vm<kLoads>();
      else barrier_vm<0>();
      read_frags(f[0], smem_u + (s1 - lds0), 0, wm, wn, lane);
    }
    mfma(acc, f[1]);
    if (t + 3 < nk) load_tile(s0, t + 3);  // into the stage k-tile t left
    const unsigned s_old = s0;
    s0 = s1;
    s1 = s2;
    s2 = s_old;
  }
  if (tid < kBM) rows_lds[tid] = rec;
  barrier_vm<0>();
  write_back_staged<2, 1, 8>(acc, epi, m0 + wm * 32, n0 + wn * 64, M, lane,
                             reinterpret_cast<float *>(smem) + wave * 32 * kStr,
                             rows_lds + wm * 32, bias);
}

// With side products (see HeadSides) the tiles of the main product come first.
template <class Epi, bool SIDES>
__global__ __launch_bounds__(256) void gemm_bf16_small_kernel(const bf16 *A, const bf16 *W, int M,
                                                              int N, int K, Epi epi,
                                                              HeadSides sides) {
  using namespace small;
  using Plain = EpiPlain<bf16, false>;
  constexpr size_t kRec = sizeof(typename Epi::Row) > sizeof(Plain::Row) ? sizeof(typename Epi::Row)
                                                                          : sizeof(Plain::Row);
  __shared__ __attribute__((aligned(1024))) unsigned char smem[3 * kStage];
  __shared__ __attribute__((aligned(16))) unsigned char rows[kBM * kRec];
  int id = xcd_remap(blockIdx.x, gridDim.x);
  if constexpr (SIDES) {
    const int tiles_m = (M + kBM - 1) / kBM;
    const int main_tiles = tiles_m * (N / kBN);
    if (id >= main_tiles) {
      id -= main_tiles;
      const int first = tiles_m * (sides.s[0].n / kBN);
      const HeadSide j = id < first ? sides.s[0] : sides.s[1];
      const Plain pe{{}, static_cast<bf16 *>(j.out), j.bias, sides.ld};
      small_tile(static_cast<const bf16 *>(j.a), static_cast<const bf16 *>(j.w), M, j.n, K, pe,
                 id < first ? id : id - first, smem, reinterpret_cast<Plain::Row *>(rows));
      return;
    }
  }
  small_tile(A, W, M, N, K, epi, id, smem, reinterpret_cast<typename Epi::Row *>(rows));
}

// ------------------------------------------------------------------ 32 and 64 rows x 32 and 64 columns
//
// For products of a few hundred rows, whose 64x128 tiles leave most of the
// chip idle while each walks all of K alone, bound by what one CU loads
// (about 60 to 85 GB/s where the weights come from the memory-side cache): a
// tile of BM x BN x 128 keeps that walk in one workgroup -- every output is
// still one accumulation over ascending k16 steps -- but loads (BM + BN) rows
// instead of 192, on more CUs.  One 32x32 block per wavefront; tiles of fewer
// than four blocks leave the other wavefronts to loading.  The loop is that of
// the 64 TM x 128 tiles on the 256-byte rows of the 64x128 tile: fragments
// read four k16 steps ahead, NS stages with NS - 1 k-tiles in flight, one
// barrier per k-tile.
// One tile of an M x N x K product; `smem` holds the NS stages.
template <class Epi, int BM, int BN, int NS>
__device__ __forceinline__ void tiny_tile(const bf16 *A, const bf16 *W, int M, int N, int K,
                                          const Epi &epi, int id, unsigned char *smem) {
  using big::pin;
  using small::kBK;
  using small::kRow;
  using Row = typename Epi::Row;
  constexpr int kWOff = BM * kRow;
  constexpr int kStage = (BM + BN) * kRow;
  constexpr int kALoads = BM / 16, kLoads = (BM + BN) / 16;  // 1 KB each, per wavefront
  constexpr int kBlocksN = BN / 32, kBlocks = BM / 32 * kBlocksN;
  constexpr int kSteps = kBK / 16, PD = 4;  // k16 steps, fragments read PD of them ahead
  constexpr int kStr = 32 + 4;              // staged write-back row (floats)
  constexpr int kRowsOff = kBlocks * 32 * kStr * 4;
  static_assert(NS >= 3 && kLoads * (NS - 1) <= 63, "stages; vmcnt holds 63");
  static_assert(kRowsOff + BM * sizeof(Row) <= NS * kStage, "row records fit the stages");
  const int tiles_m = (M + BM - 1) / BM, tiles_n = N / BN;
  int tm, tn;
  tile_coords(id, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool computes = wave < kBlocks;
  const int wm = computes ? wave / kBlocksN : 0, wn = computes ? wave % kBlocksN : 0;
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)smem;
  f32x16 acc[1][1] = {{f32x16{}}};
  const int nk = K / kBK;
  // Load p of every k-tile: p < kALoads moves activation rows 4 q .. 4 q + 3
  // (q = kALoads wave + p), the rest weight rows; lane l writes row 4 q + l / 16
  // at physical chunk l % 16.  Activation rows past M repeat row M - 1.
  uint32_t off[kLoads];
#pragma unroll
  for (int p = 0; p < kLoads; ++p) {
    const bool is_a = p < kALoads;
    const int q = is_a ? wave * kALoads + p : wave * (kLoads - kALoads) + (p - kALoads);
    const int r = q * 4 + (lane >> 4);
    const int row = is_a ? min(m0 + r, M - 1) : n0 + r;
    off[p] = ((uint32_t)row * (uint32_t)K + (uint32_t)(small::swz(r, lane & 15) * 8)) * 2u;
  }
  auto load = [&](int st, int t, int p) {
    const unsigned sb = lds0 + (unsigned)st * kStage;
    if (p < kALoads)
      t320::load_lds(sb + (wave * kALoads + p) * 1024, A + t * kBK, off[p]);
    else
      t320::load_lds(sb + kWOff + (wave * (kLoads - kALoads) + p - kALoads) * 1024, W + t * kBK,
                     off[p]);
  };
  struct Frag {
    bf16x8 x, w;
  } f[kSteps];
  const int xr = wm * 32 + (lane & 31), wr = wn * 32 + (lane & 31);
  auto read = [&](int st, int s) {
    const unsigned char *b = smem + st * kStage;
    const int c = 2 * s + (lane >> 5);
    f[s].x = *reinterpret_cast<const bf16x8 *>(b + xr * kRow + small::swz(xr, c) * 16);
    f[s].w = *reinterpret_cast<const bf16x8 *>(b + kWOff + wr * kRow + small::swz(wr, c) * 16);
  };

  // the write-back's row record and this lane's bias, kept in registers until
  // after the main loop
  Row rec{};
  if (tid < BM) rec = epi.row(min(m0 + tid, M - 1));
  const f32x4 bias = epi.bias4(n0 + wn * 32 + (lane & 7) * 4);

  // k-tiles 0 .. NS-2 in flight, then wait for k-tile 0
#pragma unroll
  for (int t = 0; t < NS - 1; ++t)
    if (t < nk) {
#pragma unroll
      for (int p = 0; p < kLoads; ++p) load(t, t, p);
    }
  mid::barrier_tiles<kLoads, NS - 2>(min(NS - 1, nk) - 1);
  if (computes) {
#pragma unroll
    for (int s = 0; s < PD; ++s) read(0, s);
  }
  int cur = 0, nxt = 1, prv = NS - 1;  // stages of k-tiles t, t + 1, t - 1
  for (int t = 0; t < nk; ++t) {
    const bool more = t + 1 < nk;
    auto steps = [&](int s0, int s1, bool rd, int stage) {
#pragma unroll
      for (int s = s0; s < s1; ++s) {
        acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[s].w, f[s].x, acc[0][0], 0, 0, 0);
        if (rd) read(stage, (s + PD) % kSteps);
        pin();
      }
    };
    if (computes) steps(0, kSteps - PD, true, cur);
    if (more) {
      // k-tile t+1 landed; those of t + 2 .. t + NS - 2 may still be in flight
      mid::barrier_tiles<kLoads, NS - 3>(min(NS - 3, nk - 2 - t));
      pin();
      // into the stage of k-tile t - 1, which every wavefront has read
      if (t + NS - 1 < nk) {
#pragma unroll
        for (int p = 0; p < kLoads; ++p) load(prv, t + NS - 1, p);
      }
    }
    if (computes) steps(kSteps - PD, kSteps, more, nxt);
    prv = cur;
    cur = nxt;
    nxt = nxt + 1 == NS ? 0 : nxt + 1;
  }
  // every wavefront is done with the stages before the row records and the
  // staged rows overwrite them
  big::barrier_vm<0>();
  Row *rows_lds = reinterpret_cast<Row *>(smem + kRowsOff);
  if (tid < BM) rows_lds[tid] = rec;
  big::barrier_vm<0>();
  if (computes)
    write_back_staged<1, 1, 4>(acc, epi, m0 + wm * 32, n0 + wn * 32, M, lane,
                               reinterpret_cast<float *>(smem) + wave * 32 * kStr,
                               rows_lds + wm * 32, bias);
}

// With side products (see HeadSides) the tiles of the main product come first.
template <class Epi, bool SIDES, int BM, int BN, int NS>
__global__ __launch_bounds__(256, 1) void gemm_bf16_tiny_kernel(const bf16 *A, const bf16 *W, int M,
                                                                int N, int K, Epi epi,
                                                                HeadSides sides) {
  using Plain = EpiPlain<bf16, false>;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[NS * (BM + BN) * small::kRow];
  int id = xcd_remap(blockIdx.x, gridDim.x);
  if constexpr (SIDES) {
    const int tiles_m = (M + BM - 1) / BM;
    const int main_tiles = tiles_m * (N / BN);
    if (id >= main_tiles) {
      id -= main_tiles;
      const int first = tiles_m * (sides.s[0].n / BN);
      const HeadSide j = id < first ? sides.s[0] : sides.s[1];
      const Plain pe{{}, static_cast<bf16 *>(j.out), j.bias, sides.ld};
      tiny_tile<Plain, BM, BN, NS>(static_cast<const bf16 *>(j.a), static_cast<const bf16 *>(j.w),
                                   M, j.n, K, pe, id < first ? id : id - first, smem);
      return;
    }
  }
  tiny_tile<Epi, BM, BN, NS>(A, W, M, N, K, epi, id, smem);
}

// ------------------------------------------------------------------ few rows
//
// The sampler's products on up to 48 rows (a few images' generating tokens):
// such a product is its weights streamed once, and its time the
// latency of one workgroup's walk over K (the 64x128 tile gave 5 rows x 1280
// x 1280 ten workgroups and 9.4 us).  A workgroup takes 16 columns.  Its eight
// wavefronts bring both operands into LDS, a stage of 256 k at a time with all
// NS stages in flight from the start (K = 1280 in one go), laid out as the
// MFMAs read them; wavefront i then multiplies the 16 rows of block i, one
// ascending sum over K, reading the next stage beside the MFMAs of the present
// one.  That is the order of every tile (the matrix instructions add their
// products one by one in ascending k, whatever their shape), so a row's result
// does not depend on how many rows share its call.  With K split over the
// wavefronts and their partial tiles added it did; 15 steps of 4 blocks of
// width 1280 then took 735 us with 5 rows, 1003 with 24 and 1136 with 33, and
// take 773, 972 and 1063.
namespace rows16 {

constexpr int kWaves = 8;
constexpr int kBN = 16;
constexpr int kSteps = 8;              // steps of 32 k per stage, one per wavefront
constexpr int kPart = kSteps * 1024;   // bytes of a stage per 16 rows or columns

// Stages in flight: five take K = 1280 whole; with three row blocks only four
// fit the CU's LDS.  (Two and three blocks on three stages, which lets two
// workgroups share a CU: 7% slower at width 1280, 3% faster to 25% slower above.)
__host__ __device__ constexpr int stages(int mb) { return mb < 3 ? 5 : 4; }

// The activations of a block's first product are the modulated norm of h,
// a = LN(h) (1 + scale) + shift.  With few rows (head_norm_fits) every workgroup
// forms them itself instead of a launch before it doing so: the rows' float32
// values are a few dozen KB that the L2 holds, and a launch costs as much as the
// whole product.
struct NormIn {
  const float *h;  // [M][K]; NULL: the activations are given
  const bf16 *shift, *scale;  // row stride mod_ld
  int mod_ld;
  float eps;
};
constexpr int kNormElems = 28 * 1024;  // M (K + 8) of them in LDS at most (56 KB)

// Rows wave, wave + 8 of the activations into `lds` (row stride K + 8: the 16
// rows of a fragment read start on distinct bank groups).
__device__ __forceinline__ void norm_rows(const NormIn &in, int M, int K, bf16 *lds, int wave,
                                          int lane) {
  constexpr int NV = 16;  // K <= 4096: float4 chunks per lane
  const int nv = K / 256;
  const float inv_w = 1.0f / (float)K;
  for (int r = wave; r < M; r += kWaves) {
    const f32x4 *hr = reinterpret_cast<const f32x4 *>(in.h + (size_t)r * K);
    const bf16 *sh = in.shift + (size_t)r * in.mod_ld, *sc = in.scale + (size_t)r * in.mod_ld;
    f32x4 v[NV], t = f32x4{};
    bf16x4 a[NV], b[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k)
      if (k < nv) {
        v[k] = hr[lane + 64 * k];
        a[k] = *reinterpret_cast<const bf16x4 *>(sc + 4 * (lane + 64 * k));
        b[k] = *reinterpret_cast<const bf16x4 *>(sh + 4 * (lane + 64 * k));
      }
    big::pin();
#pragma unroll
    for (int k = 0; k < NV; ++k)
      if (k < nv) t += v[k];
    const float mean = norm_mean(norm_sum4(t[0], t[1], t[2], t[3]), inv_w);
    t = f32x4{};
#pragma unroll
    for (int k = 0; k < NV; ++k)
      if (k < nv) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[k][e] = norm_centre(v[k][e], mean);
          t[e] = fmaf(v[k][e], v[k][e], t[e]);
        }
      }
    const float rstd = norm_rstd(norm_sum4(t[0], t[1], t[2], t[3]), inv_w, in.eps);
#pragma unroll
    for (int k = 0; k < NV; ++k)
      if (k < nv) {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          o[e] = (bf16)norm_mod(v[k][e], rstd, (float)a[k][e], (float)b[k][e]);
        *reinterpret_cast<bf16x4 *>(lds + (size_t)r * (K + 8) + 4 * (lane + 64 * k)) = o;
      }
  }
}

// Bytes of LDS: the stages in flight of the weights and MB row blocks, or
// (NORM) of the weights, then the whole activations.
inline uint32_t smem_bytes(int mb, bool norm, int m, int k) {
  const int ns = std::min(stages(mb), k / (32 * kSteps));
  const int plain = ns * (1 + mb) * kPart, with = ns * kPart + m * (k + 8) * 2;
  return (uint32_t)(norm ? std::max(plain, with) : plain);  // (side products are plain)
}

// The 16 columns from n0 of the whole M <= MB * 16 rows, K a multiple of a
// stage.  NORM (MB = 1): the
// activations come from `in`.
template <class Epi, int MB, bool NORM>
__device__ __forceinline__ void tile(const bf16 *A, const bf16 *W, int M, int K, const Epi &epi,
                                     int n0, unsigned char *smem, const NormIn &in) {
  static_assert(!NORM || MB == 1, "one row block");
  constexpr int NS = stages(MB), L = NORM ? 1 : 1 + MB, kStage = L * kPart;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)smem;
  const int nst = K / (32 * kSteps);
  const int kl = (lane >> 4) * 8;  // MFMA operands: row or column lane % 16, k kl .. kl + 7

  // what the results are combined with, on its way before the operands
  const int row = wave * 16 + (lane & 15), c0 = n0 + (lane >> 4) * 4;
  typename Epi::Col col{};
  typename Epi::Row rec{};
  typename Epi::Prior pr{};
  f32x4 bias{};
  if (wave < MB) {
    col = epi.col(c0);
    rec = epi.row(min(row, M - 1));
    bias = epi.bias4(c0);
    if constexpr (Epi::kPrior) pr = epi.prior(rec, col);
  }

  // Step `wave` of stage t, in slot t % NS: lane l's 16 bytes of the weights,
  // then of each row block, at 16 l.  Rows past M repeat row M - 1 (not stored).
  uint32_t off[L];
#pragma unroll
  for (int i = 0; i < L; ++i)
    off[i] = (uint32_t)((i == 0 ? lane & 15 : min((i - 1) * 16 + (lane & 15), M - 1)) * K + kl) * 2u;
  auto load = [&](int t) {
    const unsigned at = lds0 + (unsigned)(t % NS) * kStage + wave * 1024;
    const int k0 = (t * kSteps + wave) * 32;
#pragma unroll
    for (int i = 0; i < L; ++i)
      t320::load_lds(at + i * kPart, (i == 0 ? W + (size_t)n0 * K : A) + k0, off[i]);
  };
#pragma unroll
  for (int t = 0; t < NS; ++t)
    if (t < nst) load(t);
  bf16 *acts = reinterpret_cast<bf16 *>(smem + min(NS, nst) * kStage);  // NORM
  if constexpr (NORM) {
    norm_rows(in, M, K, acts, wave, lane);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  }
  bf16x8 w[kSteps], x[kSteps];
  const bf16 *ap = acts + (size_t)min(lane & 15, M - 1) * (K + 8) + kl;
  auto read = [&](int t, int s) {
    const unsigned char *sp = smem + (t % NS) * kStage + s * 1024 + lane * 16;
    w[s] = *reinterpret_cast<const bf16x8 *>(sp);
    if constexpr (NORM) x[s] = *reinterpret_cast<const bf16x8 *>(ap + (t * kSteps + s) * 32);
    else x[s] = *reinterpret_cast<const bf16x8 *>(sp + (1 + wave) * kPart);
  };
  f32x4 acc{};
  // stage 0 landed; the others issued may still be on their way
  mid::barrier_tiles<L, NS - 1>(min(nst, NS) - 1);
  if (wave < MB) {
#pragma unroll
    for (int s = 0; s < kSteps; ++s) read(0, s);
  }
  for (int t = 0; t + 1 < nst; ++t) {
    // stage t + 1 landed.  Issued after it: min(nst, NS) - 2 stages at first,
    // then up to NS - 3, as slots come free one at a time -- stage t - 1's now,
    // which was read, and its MFMAs issued, before this barrier.
    mid::barrier_tiles<L, NS - 2>(t == 0 ? min(nst, NS) - 2 : min(nst - 2 - t, NS - 3));
    big::pin();
    if (t > 0 && t - 1 + NS < nst) load(t - 1 + NS);
    if (wave < MB) {
#pragma unroll
      for (int s = 0; s < kSteps; ++s) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[s], x[s], acc, 0, 0, 0);
        read(t + 1, s);
        big::pin();
      }
    }
  }
  if (wave < MB) {
#pragma unroll
    for (int s = 0; s < kSteps; ++s)
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[s], x[s], acc, 0, 0, 0);
  }
  if (wave < MB && row < M) epi.store(rec, row, col, epi.combine(acc + bias, pr));
}

}  // namespace rows16

template <class Epi, int MB, bool SIDES, bool NORM>
__global__ __launch_bounds__(512) void gemm_bf16_rows_kernel(const bf16 *A, const bf16 *W, int M,
                                                             int N, int K, Epi epi,
                                                             HeadSides sides,
                                                             rows16::NormIn in) {
  using namespace rows16;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_rows[];
  int id = blockIdx.x;
  if constexpr (SIDES) {
    const int main_tiles = N / kBN;
    if (id >= main_tiles) {
      id -= main_tiles;
      const int first = sides.s[0].n / kBN;
      const HeadSide j = id < first ? sides.s[0] : sides.s[1];
      const EpiPlain<bf16, false> pe{{}, static_cast<bf16 *>(j.out), j.bias, sides.ld};
      tile<EpiPlain<bf16, false>, MB, false>(
          static_cast<const bf16 *>(j.a), static_cast<const bf16 *>(j.w), M, K, pe,
          (id < first ? id : id - first) * kBN, smem_rows, in);
      return;
    }
  }
  tile<Epi, MB, NORM>(A, W, M, K, epi, id * kBN, smem_rows, in);
}

// Tile choice by estimated time.  Every tile runs one workgroup per CU, so a
// product takes ceil(tiles / CUs) rounds of c0 + (K / 64) c1 us: c0 the launch,
// first loads and write-back, c1 a 64-deep k-tile, both fitted to products of
// 16 to 5120 rows at the model widths (N = D, 3D, 4D, K = D, 4D for D = 768,
// 1024, 1280; within about 20% of every measured time except where the whole
// chip is busy and its clock drops, which moves all tiles alike).  Half of the
// time that the tiles would take spread evenly over the chip is added, which
// settles near ties for the tile that takes less of the chip.  A call that is one
// of several image ranges shares the chip with them (`shared`): there the time of
// two such products side by side is added instead (a full and a cache-aware step
// as two ranges in us, by the single call's rule / this one: 64 images, D = 768,
// 8 layers 4943 / 4681, 16 images 1821 / 1730; 32 images, D = 1280, 4 layers
// 3234 / 3025; 64 images, D = 1024, 8 layers 7050 / 6770, 8 images 1682 / 1732).
// Measured against the best of the tiles used before (320, 256 and 128 rows x
// 256 columns, 128 x 128, 64 x 128), one box: 4352 x 1024 x 4096: 71 -> 51 us (192
// x 128), 1280 x 4096 x 1024: 24.5 -> 18.8, 3600 x 1280 x 5120: 90 -> 64, 2432 x
// 3072 x 1024: 23.9 -> 21.4 (256 x 128).  The tiles of at most 64 x 64 against 64 x
// 128: 150 x 768 x 3072: 19.5 -> 10.0 (32 x 32), 150 x 768 x 768: 7.9 -> 4.8,
// 300 x 1024 x 4096: 24.6 -> 14.5 (32 x 64), 1280 x 768 x 3072: 20.5 -> 15.1
// (64 x 64); 16 rows x 1280 x 5120: 29.0 -> 14.4 (32 x 32).
int gemm_tile_kind(DType dt, int32_t m, int32_t n, int32_t k, bool shared) {
  if (dt != DType::BF16 || m <= 0) return GEMM_TILE_128;
  struct Tile {
    int kind, rows, cols;
    double c0, c1;
  };
  static constexpr Tile kTiles[] = {
      {GEMM_TILE_320, 320, 256, 10.5, 1.20}, {GEMM_TILE_256, 256, 256, 9.5, 1.10},
      {GEMM_TILE_256x128, 256, 128, 6.5, 0.80}, {GEMM_TILE_192x128, 192, 128, 5.5, 0.60},
      {GEMM_TILE_128, 128, 128, 4.5, 0.45}, {GEMM_TILE_64x128, 64, 128, 3.6, 0.345},
      {GEMM_TILE_64x64, 64, 64, 3.0, 0.217}, {GEMM_TILE_32x64, 32, 64, 2.95, 0.174},
      {GEMM_TILE_32x32, 32, 32, 3.1, 0.1425},
  };
  const int cus = device_cu_count();
  const bool small_off = (int64_t)n * k < (1LL << 31);  // 32-bit operand offsets
  int best = -1;
  double best_t = 0.0;
  for (const Tile &t : kTiles) {
    if (t.rows <= 64 && k % small::kBK != 0) continue;
    if (!small_off && t.kind != GEMM_TILE_256 && t.kind != GEMM_TILE_64x128) continue;
    const int64_t tiles = (int64_t)((m + t.rows - 1) / t.rows) * (n / t.cols);
    const double one = t.c0 + (k / 64) * t.c1;
    const int64_t alone = (tiles + cus - 1) / cus, two = (2 * tiles + cus - 1) / cus;
    const double time = shared ? (double)(alone + two) * one
                               : (double)alone * one + 0.5 * tiles * one / cus;
    if (best < 0 || time < best_t) {
      best = t.kind;
      best_t = time;
    }
  }
  return best;
}

// Up to three blocks of 16 rows, as long as the launch's workgroups (16 of its
// n columns each, side products among them) are resident at once: two per CU
// with one row block (80 KB of LDS; up to 96 KB with the norm of more than 8
// rows inside, at widths of 1536 and more), one with two or three.  A sampling step in
// us, this kernel / tiles: width 1280, 3 and 8 blocks: 5 rows 42 / 59 and 91 /
// 142, 16 rows 49 / 61 and 114 / 147, 32 rows 53 / 62 and 127 / 151, 48 rows
// 60 / 62 and 146 / 151; width 1536, 17 rows: 8 blocks (253 workgroups) 124 /
// 162, 3 blocks (288) 66 / 67, 33 rows 81 / 67; width 2048, 3 blocks (384): 16
// rows 82 / 82, 17 rows 92 / 82; width 4096 (768): 1 row 173 / 163, 16 rows
// 206 / 166, 40 rows 314 / 183.  A time embedding whose length is no whole
// number of stages takes a tile.  (Both give the same bits.)
bool gemm_few_rows(DType dt, int32_t m, int32_t n, int32_t k) {
  return dt == DType::BF16 && m <= 48 && k % (32 * rows16::kSteps) == 0 &&
         n / rows16::kBN <= device_cu_count() * (m <= 16 ? 2 : 1);
}

// The few-row kernel with the side products' tiles after the main ones.
template <class Epi, bool SIDES>
static void run_rows(const bf16 *A, const bf16 *W, int m, int n, int k, const Epi &epi,
                     const HeadSides &sides, hipStream_t s) {
  const int grid = (n + (SIDES ? sides.s[0].n + sides.s[1].n : 0)) / rows16::kBN;
  const rows16::NormIn none{};
#define R_(MB)                                                                             \
  launch_kernel(gemm_bf16_rows_kernel<Epi, MB, SIDES, false>, grid, 512,                   \
                rows16::smem_bytes(MB, false, m, k), s, A, W, m, n, k, epi, sides, none)
  if (m <= 16) R_(1);
  else if (m <= 32) R_(2);
  else R_(3);
#undef R_
}

template <class Epi, int BM, int BN, int NS>
static void run_tiny(const bf16 *A, const bf16 *W, int m, int n, int k, const Epi &epi,
                     hipStream_t s) {
  launch_kernel(gemm_bf16_tiny_kernel<Epi, false, BM, BN, NS>, ((m + BM - 1) / BM) * (n / BN), 256,
                0, s, A, W, m, n, k, epi, HeadSides{});
}

template <class Epi, int TM, int NS>
static void run_mid(const bf16 *A, const bf16 *W, int m, int n, int k, const Epi &epi,
                    hipStream_t s) {
  constexpr int kBM = mid::Shape<TM>::kBM;
  launch_kernel(gemm_bf16_mid_kernel<Epi, TM, NS>, ((m + kBM - 1) / kBM) * (n / mid::kBN), 256, 0,
                s, A, W, m, n, k, epi);
}

// N a multiple of 256 and K of 64 (the host limits d_model and d_mlp to
// multiples of 256).
template <class Epi>
static hipError_t run_bf16(const void *a, const void *w, int m, int n, int k, const Epi &epi,
                           hipStream_t s, bool shared = false) {
  if (m == 0) return hipSuccess;
  if (n % 256 != 0 || k % 64 != 0) return hipErrorInvalidValue;
  const bf16 *A = static_cast<const bf16 *>(a), *W = static_cast<const bf16 *>(w);
  switch (gemm_tile_kind(DType::BF16, m, n, k, shared)) {
    case GEMM_TILE_256:
      // eight wavefronts where the write-back is a large share of a tile
      // (K < 2048: fc1, QKV, the output projection), four where the main
      // loop dominates and the fewer LDS reads per MFMA win (fc2)
      if (k < 2048)
        launch_kernel(gemm_bf16_big8_kernel<Epi>, ((m + 255) / 256) * (n / 256), 512, 0, s, A, W,
                      m, n, k, epi);
      else
        launch_kernel(gemm_bf16_big_kernel<Epi>, ((m + 255) / 256) * (n / 256), 256, 0, s, A, W,
                      m, n, k, epi);
      break;
    case GEMM_TILE_320:
      launch_kernel(gemm_bf16_t320_kernel<Epi>, ((m + t320::kBM - 1) / t320::kBM) * (n / 256), 512,
                    0, s, A, W, m, n, k, epi);
      break;
    case GEMM_TILE_64x128:
      launch_kernel(gemm_bf16_small_kernel<Epi, false>,
                    ((m + small::kBM - 1) / small::kBM) * (n / small::kBN), 256, 0, s, A, W, m, n,
                    k, epi, HeadSides{});
      break;
    case GEMM_TILE_64x64: run_tiny<Epi, 64, 64, 5>(A, W, m, n, k, epi, s); break;
    case GEMM_TILE_32x64: run_tiny<Epi, 32, 64, 6>(A, W, m, n, k, epi, s); break;
    case GEMM_TILE_32x32: run_tiny<Epi, 32, 32, 8>(A, W, m, n, k, epi, s); break;
    case GEMM_TILE_192x128: run_mid<Epi, 3, 4>(A, W, m, n, k, epi, s); break;
    case GEMM_TILE_256x128: run_mid<Epi, 4, 3>(A, W, m, n, k, epi, s); break;
    default: run_mid<Epi, 2, 4>(A, W, m, n, k, epi, s); break;
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------ fp32 (v_mfma_f32)
//
// fp32 products run on the fp32 matrix instructions (exact fp32 multiplies and
// accumulation, twice the rate of the vector FMA).  Lanes load four
// consecutive k of a row as one 16-byte read and spend them in four MFMAs:
// both operands then carry the same permutation of k, which a dot product
// does not see.
//
// Two kernels:
//  - f32_tile: a 64x64x32 tile of four 32x32 wavefronts, operands straight
//    from global memory into the 128-byte swizzled LDS rows of the bf16 tiles
//    (32 floats per row), four stages;
//  - f32_skinny: for products whose 64x64 tiles would not give every compute
//    unit one.  These are bound by the latency of one workgroup's walk over K
//    (a 64x64 FMA tile with two barriers per 16 of K took 182 us for 32 rows x
//    768 x 3072 on 12 compute units), so a workgroup takes 16 columns and up
//    to 64 rows, its 16 wavefronts split K, load both operands directly into
//    the MFMA registers (64-byte row segments, every load of a wavefront
//    independent of the others) and sum their partial tiles through LDS in
//    wavefront order.
// Which of them runs depends on M, and an image's rows must not depend on the
// images that share its call.  So both add up an output in one order, which
// depends on K alone: 16 slices of K, each from zero and added to the sum of
// those before it; inside a slice 16 k at a time, element e of the four
// 16-byte chunks in turn for e = 0 .. 3.  (The matrix instructions add their
// products one by one in ascending k, so 32x32x2 on chunk pairs (0, 1), (2, 3)
// continues the sum as 16x16x4 on all four does.)
namespace f32 {

constexpr int kWaves = 16;  // K slices; the skinny kernel has a wavefront for each

__device__ __forceinline__ f32x4 mfma4(const f32x4 &w, const f32x4 &x, f32x4 acc) {
#pragma unroll
  for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[e], x[e], acc, 0, 0, 0);
  return acc;
}

}  // namespace f32

// C^T blocks of 16 columns x MB * 16 rows: lane l holds column group l / 16
// (four consecutive columns) of row l % 16 of each block.
template <class Epi, int MB>
__global__ __launch_bounds__(1024) void gemm_f32_skinny_kernel(const float *__restrict__ A,
                                                               const float *__restrict__ W, int M,
                                                               int N, int K, Epi epi) {
  using namespace f32;
  __shared__ f32x4 part[kWaves][MB][64];
  const int tiles_n = N / 16;
  const int n0 = (blockIdx.x % tiles_n) * 16, m0 = (blockIdx.x / tiles_n) * (MB * 16);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // steps of 16 k; wavefront w takes steps [w S / 16, (w + 1) S / 16)
  const int steps = K / 16;
  const int s0 = wave * steps / kWaves, s1 = (wave + 1) * steps / kWaves;
  const int kl = (lane >> 4) * 4;
  const float *wp = W + (size_t)(n0 + (lane & 15)) * K + kl;
  const float *xp[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
    xp[i] = A + (size_t)min(m0 + i * 16 + (lane & 15), M - 1) * K + kl;
  f32x4 acc[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) acc[i] = f32x4{};
  constexpr int U = MB >= 4 ? 3 : 4;  // steps whose loads are in flight together
  int s = s0;
  for (; s + U <= s1; s += U) {
    f32x4 w[U], x[U][MB];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      w[u] = *reinterpret_cast<const f32x4 *>(wp + (s + u) * 16);
#pragma unroll
      for (int i = 0; i < MB; ++i)
        x[u][i] = *reinterpret_cast<const f32x4 *>(xp[i] + (s + u) * 16);
    }
    big::pin();  // every load before the first MFMA's wait
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < MB; ++i) acc[i] = mfma4(w[u], x[u][i], acc[i]);
  }
  for (; s < s1; ++s) {
    const f32x4 w = *reinterpret_cast<const f32x4 *>(wp + s * 16);
#pragma unroll
    for (int i = 0; i < MB; ++i)
      acc[i] = mfma4(w, *reinterpret_cast<const f32x4 *>(xp[i] + s * 16), acc[i]);
  }
#pragma unroll
  for (int i = 0; i < MB; ++i) part[wave][i][lane] = acc[i];
  __syncthreads();
  if (wave >= MB) return;
  f32x4 v = part[0][wave][lane];
#pragma unroll
  for (int g = 1; g < kWaves; ++g) v += part[g][wave][lane];
  const int row = m0 + wave * 16 + (lane & 15), c0 = n0 + kl;
  // the column's destination is uniform over the wavefront: computed by all
  // lanes, before the row guard
  const typename Epi::Col c = epi.col(c0);
  if (row >= M) return;
  const typename Epi::Row r = epi.row(row);
  v += epi.bias4(c0);
  if constexpr (Epi::kPrior) v = epi.combine(v, epi.prior(r, c));
  epi.store(r, row, c, v);
}

// A 64x64x32 tile (K a multiple of 256: whole steps in every slice).
template <class Epi>
__global__ __launch_bounds__(256, 2) void gemm_f32_tile_kernel(const float *A, const float *W, int M,
                                                            int N, int K, Epi epi) {
  using Row = typename Epi::Row;
  constexpr int T = 64, NS = 4;
  constexpr int kWOff = T * 128, kStage = 2 * T * 128;  // 8 KB per operand
  constexpr int kStr = 36;                              // staged write-back row (floats)
  __shared__ __attribute__((aligned(1024))) unsigned char smem[NS * kStage];
  __shared__ __attribute__((aligned(16))) Row rows_lds[T];
  static_assert(4 * 32 * kStr * 4 <= NS * kStage, "staged write-back fits the stages");
  const int tiles_m = (M + T - 1) / T, tiles_n = N / T;
  int tm, tn;
  tile_coords(xcd_remap(blockIdx.x, gridDim.x), tiles_m, tiles_n, tm, tn);
  const int m0 = tm * T, n0 = tn * T;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)smem;
  const int nk = K / 32;
  // a k-tile of 32 floats (two steps of 16) is 64 16-bit elements to the loader
  const bf16 *A2 = reinterpret_cast<const bf16 *>(A), *W2 = reinterpret_cast<const bf16 *>(W);
  auto load_tile = [&](int t) {
    const unsigned sb = lds0 + (unsigned)(t % NS) * kStage;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      big::load_lds(sb, wave * 2 + p, A2, M, 2 * K, m0, t * 64, lane);
      big::load_lds(sb + kWOff, wave * 2 + p, W2, N, 2 * K, n0, t * 64, lane);
    }
  };
  Row rec{};
  if (tid < T) rec = epi.row(min(m0 + tid, M - 1));
  const f32x4 bias = epi.bias4(n0 + wn * 32 + (lane & 7) * 4);
  const int rx = wm * 32 + (lane & 31), rw = wn * 32 + (lane & 31);
#pragma unroll
  for (int t = 0; t < NS - 1; ++t)
    if (t < nk) load_tile(t);
  // This half's chunks of the pairs (0, 1) and (2, 3) of a step, read one step
  // ahead.
  struct Frag {
    f32x4 x[2], w[2];
  };
  const int steps = K / 16;
  auto read = [&](int s) {
    if ((s & 1) == 0) {
      // k-tile t landed (issued so far: up to t + NS - 2, four loads each) and
      // every wavefront done with k-tile t - 1, whose stage takes t + NS - 1
      const int t = s >> 1, ahead = min(NS - 2, nk - 1 - t);
      if (ahead >= 2) big::barrier_vm<8>();
      else if (ahead == 1) big::barrier_vm<4>();
      else big::barrier_vm<0>();
      if (t + NS - 1 < nk) load_tile(t + NS - 1);
    }
    const unsigned char *sc = smem + ((s >> 1) % NS) * kStage;
    Frag f;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int kc = (s & 1) * 4 + u * 2 + (lane >> 5);
      f.x[u] = *reinterpret_cast<const f32x4 *>(sc + rx * 128 + big::swz(rx, kc) * 16);
      f.w[u] = *reinterpret_cast<const f32x4 *>(sc + kWOff + rw * 128 + big::swz(rw, kc) * 16);
    }
    return f;
  };
  // One slice into `c`.  Two accumulators take the slices in turn, so that the
  // one before, `done`, is added to the sum beside the MFMAs of this one: a
  // layer of 2480 rows at D = 768 takes 476 us, with a single accumulator (read,
  // added and cleared between two slices) 504, in one sum over all of K 447.
  // Two wavefronts per SIMD as the launch bound keep the accumulators in VGPRs,
  // which the additions can read.  The sum starts at -0, which leaves the first
  // slice's bits alone.
  f32x16 acc[2], sum[1][1];
#pragma unroll
  for (int e = 0; e < 16; ++e) sum[0][0][e] = acc[1][e] = -0.0f;
  int s = 0;
  Frag f = read(0);
  auto step = [&](f32x16 &c, const f32x16 &c0) {
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(f.w[0][0], f.x[0][0], c0, 0, 0, 0);
    big::pin();
    const Frag next = read(min(++s, steps - 1));  // (the last is odd: read again, no barrier)
    big::pin();
#pragma unroll
    for (int i = 1; i < 8; ++i)
      c = __builtin_amdgcn_mfma_f32_32x32x2f32(f.w[i & 1][i >> 1], f.x[i & 1][i >> 1], c, 0, 0, 0);
    f = next;
  };
  auto slice = [&](f32x16 &c, const f32x16 &done) {
    step(c, f32x16{});
    sum[0][0] += done;
    for (int j = 1; j < steps / f32::kWaves; ++j) step(c, c);
  };
#pragma unroll 1
  for (int g = 0; g < f32::kWaves; g += 2) {
    slice(acc[0], acc[1]);
    slice(acc[1], acc[0]);
  }
  sum[0][0] += acc[1];
  if (tid < T) rows_lds[tid] = rec;
  big::barrier_vm<0>();
  write_back_staged<1, 1, 4>(sum, epi, m0 + wm * 32, n0 + wn * 32, M, lane,
                             reinterpret_cast<float *>(smem) + wave * 32 * kStr, rows_lds + wm * 32,
                             bias);
}

template <class Epi>
static hipError_t run_f32(const void *a, const void *w, int m, int n, int k, const Epi &epi,
                          hipStream_t s) {
  if (m == 0) return hipSuccess;
  if (n % 64 != 0 || k % 32 != 0) return hipErrorInvalidValue;
  const float *A = static_cast<const float *>(a), *W = static_cast<const float *>(w);
  const long tiles = (long)((m + 63) / 64) * (n / 64);
  // 64x64 tiles once every compute unit has one (and K is the model's: a time
  // embedding's may be any multiple of 64); else the skinny kernel, with as
  // few rows per workgroup as cover a small M
  if (tiles >= device_cu_count() && k % 256 == 0)
    launch_kernel(gemm_f32_tile_kernel<Epi>, (unsigned)tiles, 256, 0, s, A, W, m, n, k, epi);
  else if (m <= 16)
    launch_kernel(gemm_f32_skinny_kernel<Epi, 1>, n / 16, 1024, 0, s, A, W, m, n, k, epi);
  else if (m <= 32)
    launch_kernel(gemm_f32_skinny_kernel<Epi, 2>, n / 16, 1024, 0, s, A, W, m, n, k, epi);
  else
    launch_kernel(gemm_f32_skinny_kernel<Epi, 4>, (n / 16) * ((m + 63) / 64), 1024, 0, s, A, W, m,
                  n, k, epi);
  return hipGetLastError();
}

// ------------------------------------------------------------------ launchers

hipError_t launch_gemm_qkv(DType dt, const void *a, const void *w, const float *bias, int32_t m,
                           int32_t n, int32_t k, const RowMap *map, QkvOut o, bool shared,
                           hipStream_t s) {
  if (dt == DType::F32) {
    EpiQkv<float> e{{}, static_cast<float *>(o.q), static_cast<float *>(o.k_cache),
                    static_cast<float *>(o.v_cache), bias, map, o.d_model, o.head_dim,
                    o.n_heads, o.n_tokens};
    return run_f32(a, w, m, n, k, e, s);
  }
  EpiQkv<bf16> e{{}, static_cast<bf16 *>(o.q), static_cast<bf16 *>(o.k_cache),
                 static_cast<bf16 *>(o.v_cache), bias, map, o.d_model, o.head_dim, o.n_heads,
                 o.n_tokens};
  return run_bf16(a, w, m, n, k, e, s, shared);
}

hipError_t launch_gemm_resid(DType dt, const void *a, const void *w, const float *bias, int32_t m,
                             int32_t n, int32_t k, const RowMap *map, float *x, int32_t tag,
                             bool shared, hipStream_t s) {
  if (tag == 0) {
    EpiResid<0> e{{}, x, bias, map, n};
    return dt == DType::F32 ? run_f32(a, w, m, n, k, e, s) : run_bf16(a, w, m, n, k, e, s, shared);
  }
  EpiResid<1> e{{}, x, bias, map, n};
  return dt == DType::F32 ? run_f32(a, w, m, n, k, e, s) : run_bf16(a, w, m, n, k, e, s, shared);
}

hipError_t launch_gemm_gelu(DType dt, const void *a, const void *w, const float *bias, int32_t m,
                            int32_t n, int32_t k, void *h, bool shared, hipStream_t s) {
  if (dt == DType::F32) {
    EpiGelu<float> e{{}, static_cast<float *>(h), bias, n};
    return run_f32(a, w, m, n, k, e, s);
  }
  EpiGelu<bf16> e{{}, static_cast<bf16 *>(h), bias, n};
  return run_bf16(a, w, m, n, k, e, s, shared);
}

}  // namespace marche

namespace marche {

// A bf16 sampler product without side products.
template <class Epi>
static hipError_t run_plain(const void *a, const void *w, int m, int n, int k, const Epi &epi,
                            hipStream_t s) {
  if (m == 0 || !gemm_few_rows(DType::BF16, m, n, k)) return run_bf16(a, w, m, n, k, epi, s);
  if (n % 256 != 0) return hipErrorInvalidValue;
  run_rows<Epi, false>(static_cast<const bf16 *>(a), static_cast<const bf16 *>(w), m, n, k, epi,
                       HeadSides{}, s);
  return hipGetLastError();
}

hipError_t launch_gemm_plain(DType dt, const void *a, const void *w, const float *bias, int32_t m,
                             int32_t n, int32_t k, void *out, DType out_dt, bool silu_act,
                             int32_t ld, hipStream_t s) {
  if (dt == DType::F32) {
    if (out_dt != DType::F32) return hipErrorInvalidValue;
    if (silu_act) return run_f32(a, w, m, n, k, EpiPlain<float, true>{{}, static_cast<float *>(out), bias, ld}, s);
    return run_f32(a, w, m, n, k, EpiPlain<float, false>{{}, static_cast<float *>(out), bias, ld}, s);
  }
  if (out_dt == DType::F32) {
    if (silu_act) return hipErrorInvalidValue;
    return run_plain(a, w, m, n, k, EpiPlain<float, false>{{}, static_cast<float *>(out), bias, ld}, s);
  }
  if (silu_act) return run_plain(a, w, m, n, k, EpiPlain<bf16, true>{{}, static_cast<bf16 *>(out), bias, ld}, s);
  return run_plain(a, w, m, n, k, EpiPlain<bf16, false>{{}, static_cast<bf16 *>(out), bias, ld}, s);
}

int head_side_tiles(DType dt, int32_t m, int32_t width) {
  if (dt != DType::BF16 || m <= 0) return 0;
  const int tiles_m = (m + small::kBM - 1) / small::kBM;
  return std::max(0, device_cu_count() / tiles_m - width / small::kBN);
}

// Tile of a sampler block's product of `width` columns with side products of
// n_side columns on more rows than the few-row kernel takes: the smallest
// whose tiles all run at once, one per CU, else 64 x 128 (50 steps of 8 blocks
// of width 1280 with 64 x 128 always and by this rule: 96 rows 10.5 and 8.1 ms,
// 128 rows 10.5 and 7.7, 256 rows 10.7 and 8.5).
int head_tile_kind(int32_t m, int32_t width, int32_t n_side) {
  if (n_side == 0) return gemm_tile_kind(DType::BF16, m, width, width);
  const int cols = (width + n_side) / 64;
  if ((m + 31) / 32 * cols <= device_cu_count()) return GEMM_TILE_32x64;
  if ((m + 63) / 64 * cols <= device_cu_count()) return GEMM_TILE_64x64;
  return GEMM_TILE_64x128;
}

template <class Epi, int BM, int BN, int NS>
static void run_tiny_sides(const bf16 *A, const bf16 *W, int m, int width, const Epi &epi,
                           const HeadSides &sides, int n_side, hipStream_t s) {
  launch_kernel(gemm_bf16_tiny_kernel<Epi, true, BM, BN, NS>,
                ((m + BM - 1) / BM) * ((width + n_side) / BN), 256, 0, s, A, W, m, width, width, epi,
                sides);
}

template <class Epi>
static hipError_t run_head(const void *a, const void *w, int m, int width, const Epi &epi,
                           const HeadSides &sides, hipStream_t s) {
  const bf16 *A = static_cast<const bf16 *>(a), *W = static_cast<const bf16 *>(w);
  const int n_side = sides.s[0].n + sides.s[1].n;
  if (n_side == 0) return run_plain(a, w, m, width, width, epi, s);
  if (width % 256 != 0 || sides.s[0].n % small::kBN != 0 || sides.s[1].n % small::kBN != 0)
    return hipErrorInvalidValue;
  if (gemm_few_rows(DType::BF16, m, width + n_side, width)) {
    run_rows<Epi, true>(A, W, m, width, width, epi, sides, s);
    return hipGetLastError();
  }
  switch (head_tile_kind(m, width, n_side)) {
    case GEMM_TILE_32x64: run_tiny_sides<Epi, 32, 64, 6>(A, W, m, width, epi, sides, n_side, s); break;
    case GEMM_TILE_64x64: run_tiny_sides<Epi, 64, 64, 5>(A, W, m, width, epi, sides, n_side, s); break;
    default:
      launch_kernel(gemm_bf16_small_kernel<Epi, true>,
                    ((m + small::kBM - 1) / small::kBM) * ((width + n_side) / small::kBN), 256, 0,
                    s, A, W, m, width, width, epi, sides);
  }
  return hipGetLastError();
}

hipError_t launch_head_gemm_silu(DType dt, const void *a, const void *w, const float *bias,
                                 int32_t m, int32_t width, void *y, const HeadSides &sides,
                                 hipStream_t s) {
  if (dt == DType::F32)
    return run_f32(a, w, m, width, width,
                   EpiPlain<float, true>{{}, static_cast<float *>(y), bias, width}, s);
  return run_head(a, w, m, width, EpiPlain<bf16, true>{{}, static_cast<bf16 *>(y), bias, width},
                  sides, s);
}

// One row per wavefront (8), or two at widths where the products are long enough
// to hide the second, as far as they fit the LDS.  15 sampling steps of 8 blocks
// in us, norm inside / a launch of its own: 8 rows: width 256 855 / 949, 1280
// 1442 / 1520, 2048 2567 / 2804; 16 rows: width 256 1012 / 982, 1024 1559 / 1486,
// 1280 1697 / 1612; 12 rows: width 1536 1739 / 1723 (3 blocks 820 / 855), 2048
// 2730 / 2933.
bool head_norm_fits(DType dt, int32_t m, int32_t width) {
  return dt == DType::BF16 && m >= 1 && m <= (width < 1536 ? 8 : 16) &&
         (int64_t)m * (width + 8) <= rows16::kNormElems;
}

hipError_t launch_head_gemm_norm_silu(const float *h, const void *mod, int32_t mod_ld,
                                      int32_t shift_off, int32_t scale_off, float eps,
                                      const void *w, const float *bias, int32_t m, int32_t width,
                                      void *y, const HeadSides &sides, hipStream_t s) {
  if (!head_norm_fits(DType::BF16, m, width) || width % 256 != 0 || width > 4096 ||
      sides.s[0].n % 16 != 0 || sides.s[1].n % 16 != 0)
    return hipErrorInvalidValue;
  const bf16 *W = static_cast<const bf16 *>(w), *mo = static_cast<const bf16 *>(mod);
  const EpiPlain<bf16, true> epi{{}, static_cast<bf16 *>(y), bias, width};
  const rows16::NormIn in{h, mo + shift_off, mo + scale_off, mod_ld, eps};
  launch_kernel(gemm_bf16_rows_kernel<EpiPlain<bf16, true>, 1, true, true>,
                (width + sides.s[0].n + sides.s[1].n) / rows16::kBN, 512,
                rows16::smem_bytes(1, true, m, width), s, nullptr, W, m, width, width, epi, sides, in);
  return hipGetLastError();
}

hipError_t launch_head_gemm_gate(DType dt, const void *a, const void *w, const float *bias,
                                 int32_t m, int32_t width, float *h, const void *gate,
                                 int32_t mod_ld, const HeadSides &sides, hipStream_t s) {
  if (dt == DType::F32)
    return run_f32(a, w, m, width, width,
                   EpiGate<float>{h, bias, static_cast<const float *>(gate), width, mod_ld}, s);
  return run_head(a, w, m, width,
                  EpiGate<bf16>{h, bias, static_cast<const bf16 *>(gate), width, mod_ld}, sides, s);
}

hipError_t launch_gemm_embed(DType dt, const void *a, const void *w, const float *bias, int32_t m,
                             int32_t n, int32_t k, float *x, const float *pe, const int32_t *known,
                             int32_t n_enc, int32_t n_buf, int32_t n_known, int32_t n_tokens,
                             hipStream_t s) {
  EpiEmbed e{{}, x, bias, pe, known, n, n_enc, n_buf, n_known, n_tokens};
  return dt == DType::F32 ? run_f32(a, w, m, n, k, e, s) : run_bf16(a, w, m, n, k, e, s);
}

}  // namespace marche
