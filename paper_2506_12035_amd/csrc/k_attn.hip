// Cache-aware bidirectional attention (Algorithm 1 / Section 4.1) and the
// attention-mass score pass of the selection layer (Section 4.2).
//
// Because the fresh K/V of the active tokens were already written into the
// layer's cache by the QKV epilogue, the active segment K_A and the cached
// segment K_C are one resident buffer [b][h][N][d_h]: the online-softmax
// merge of the two segments (Appendix A) becomes the kernel's own loop over
// key tiles, with a running maximum and a rescaled running sum, and no K/V is
// ever concatenated or copied.
//
// bf16 kernels (gfx950 MFMA, v_mfma_f32_32x32x16_bf16): one workgroup per
// (image, head, chunk of active queries), one wavefront per 32 queries:
//   - S^T = K Q^T is formed so that lane l owns query (l & 31): the row
//     maximum and sum need one cross-half exchange, and the accumulator
//     rescale is a per-lane scalar;
//   - O^T = V^T P^T: P stays in registers (converted to bf16); the operand V^T
//     comes from a transposing LDS read, or (resident kernel) from tiles stored
//     transposed with the keys of every 16-key group permuted to match the
//     accumulator layout of S^T.
// Softmax runs in the log2 domain with fp32 statistics.  Three kernels:
// attn_resident_kernel (full layers, every key of a head in LDS),
// attn_reg_kernel (head width 64, whole key tiles) and attn_gen_kernel (any
// other shape, among them the two segments of Appendix B's comparison as
// separate buffers in one online-softmax pass: Appendix A's merge without
// concatenation).
#include <algorithm>
#include <type_traits>

#include "device_common.h"

namespace marche {

constexpr int TK = 64;  // keys per tile

// Position of key k (0..15) inside its 16-key group in the transposed V tile.
// S^T's accumulator gives lane half hf the keys {4hf..4hf+3, 8+4hf..8+4hf+3}
// of each 16-key group; this places exactly those at positions 8hf..8hf+7.
__device__ __forceinline__ int vperm16(int k) {
  return (k & 3) | (((k >> 3) & 1) << 2) | (((k >> 2) & 1) << 3);
}

// Element offsets inside one tile's K and V^T blocks.  Padded layout: rows of
// DH + 8 (K) and TK + 8 (V^T) elements.  Swizzled layout (DH = 64 only): rows
// of 64 elements whose 16-byte chunks are permuted by an XOR with the row
// pair index, so 16 consecutive rows read at one chunk hit distinct banks
// without padding (8 KB per tile for K and for V^T).
template <int DH, bool SWZ>
__device__ __forceinline__ int k_off(int key, int d) {
  if constexpr (SWZ) return key * 64 + ((((d >> 3) ^ (key >> 1)) & 7) << 3) + (d & 7);
  else return key * (DH + 8) + d;
}
template <int DH, bool SWZ>
__device__ __forceinline__ int vt_off(int row, int pos) {
  if constexpr (SWZ) return row * 64 + ((((pos >> 3) ^ (row >> 1)) & 7) << 3) + (pos & 7);
  else return row * (TK + 8) + pos;
}

// One 64-key tile of the online softmax for one wavefront's 32 queries.
// ks: the tile's K rows in LDS; vt: its transposed V (keys of each 16-key
// group permuted by vperm16); t0: the tile's first key within a segment of
// ns keys, MASK set when the tile runs past the segment's end.  Updates the
// running maximum, sum and the O^T accumulators in the log2 domain (sl2 =
// log2(e) / sqrt(d_h) > 0).  The maximum is taken over the raw logits: as
// rounding a product by a positive constant is monotone, fl(max * sl2) is
// the maximum of the scaled logits exactly, and the scale then folds into
// the exponent's argument as one FMA per logit.
template <int DH, bool SWZ = false, bool MASK = false>
__device__ __forceinline__ void attn_tile(const bf16 *ks, const bf16 *vt, const bf16x8 (&qf)[DH / 16],
                                          f32x16 (&acc)[(DH + 31) / 32], float &m_run, float &l_run,
                                          int t0, int ns, float sl2, int lane) {
  static_assert(!SWZ || DH == 64, "swizzled tiles hold 64-element rows");
  constexpr int QS = DH / 16, ODB = (DH + 31) / 32;
  // S^T for two 32-key blocks: lane -> query (lane & 31),
  // register r -> key (r / 4) * 8 + (lane / 32) * 4 + r % 4 of the block.
  f32x16 s[2];
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    s[kb] = f32x16{};
#pragma unroll
    for (int st = 0; st < QS; ++st) {
      const bf16x8 ka = *reinterpret_cast<const bf16x8 *>(
          &ks[k_off<DH, SWZ>(kb * 32 + (lane & 31), st * 16 + (lane >> 5) * 8)]);
      s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qf[st], s[kb], 0, 0, 0);
    }
  }
  float mx = -INFINITY;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if constexpr (MASK) {
        const int key = t0 + kb * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        if (key >= ns) s[kb][r] = -INFINITY;
      }
      mx = fmaxf(mx, s[kb][r]);
    }
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
  const float m_new = fmaxf(m_run, mx * sl2);
  const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
  float psum = 0.f;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float p = __builtin_amdgcn_exp2f(fmaf(s[kb][r], sl2, -m_new));
      s[kb][r] = p;
      psum += p;
    }
  l_run = l_run * alpha + psum;
  m_run = m_new;
#pragma unroll
  for (int d = 0; d < ODB; ++d) acc[d] *= alpha;

  // O^T += V^T P^T over the 64 keys of the tile, 16 keys per MFMA.
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      bf16x8 pb;
#pragma unroll
      for (int e = 0; e < 8; ++e) pb[e] = (bf16)s[kb][8 * u + e];
#pragma unroll
      for (int d = 0; d < ODB; ++d) {
        const bf16x8 va = *reinterpret_cast<const bf16x8 *>(
            &vt[vt_off<DH, SWZ>(d * 32 + (lane & 31), kb * 32 + 16 * u + (lane >> 5) * 8)]);
        acc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb, acc[d], 0, 0, 0);
      }
    }
}

// ------------------------------------------------------------ cache-aware kernel, head width 64
//
// Cache-aware layers at head width 64 with every key tile whole (N a multiple
// of 64): one workgroup per (image, head, chunk of QB*32 active queries), one
// wavefront per 32 queries over all keys.  Key tiles (64 keys of K and of V,
// 16 KB) go global -> registers -> one of two LDS slots, row-major: no
// transposition on the way.  The MFMA operand V^T (32 head dims x 16 keys per
// lane group) comes from the transposing LDS read of gfx950 (ds_read_tr16_b64:
// within 16 lanes, lane 4e + q names row e and four consecutive columns
// 4q..4q+3 of a 4 x 16 block, and lane i receives column i of the four rows).
// K and V tiles permute the 16-byte chunks of a row by an XOR with the
// bit-reversed row-pair index, so a K fragment read (16 rows at one chunk)
// and a V^T read (4 rows x 4 chunks per 32 lanes) each touch every bank group
// once.  Only registers stage the next tile, so a workgroup needs 32 KB of
// LDS and five fit on a compute unit: at MAR-L sizes every (image, head) of a
// call is resident at once, each with one tile in flight.
namespace strm {

constexpr int kSlotBytes = 16384;  // 64 keys x 64 dims x 2 bytes, K then V

// Chunk permutation of row r: the row-pair index (r >> 1) & 7, bit-reversed.
__device__ __forceinline__ int swz(int r) {
  const int x = (r >> 1) & 7;
  return ((x & 1) << 2) | (x & 2) | (x >> 2);
}

typedef short s16x4 __attribute__((ext_vector_type(4)));

// Transposing read of four consecutive keys for this lane's head dim (see above).
__device__ __forceinline__ s16x4 read_tr(const unsigned char *p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (s16x4 __attribute__((address_space(3))) *)(
          (__attribute__((address_space(3))) unsigned char *)(uintptr_t)p));
}

// One 64-key tile of the online softmax for this wavefront's 32 queries
// (lane -> query lane & 31), in the log2 domain, as attn_tile does for the
// transposed-V layouts: S^T = K Q^T, running max over the raw logits, the
// scale folded into the exponent, O^T += V^T P^T.
__device__ __forceinline__ void tile(const unsigned char *slot, const bf16x8 (&qf)[4],
                                     f32x16 (&acc)[2], float &m_run, float &l_run, float sl2,
                                     int lane) {
  const unsigned char *kt = slot, *vt = slot + 8192;
  f32x16 s[2];
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    s[kb] = f32x16{};
    const int row = kb * 32 + (lane & 31);
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      const int c = st * 2 + (lane >> 5);
      const bf16x8 ka = *reinterpret_cast<const bf16x8 *>(kt + row * 128 + ((c ^ swz(row)) << 4));
      s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qf[st], s[kb], 0, 0, 0);
    }
  }
  float mx = -INFINITY;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kb][r]);
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
  const float m_new = fmaxf(m_run, mx * sl2);
  const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
  float psum = 0.f;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float p = __builtin_amdgcn_exp2f(fmaf(s[kb][r], sl2, -m_new));
      s[kb][r] = p;
      psum += p;
    }
  l_run = l_run * alpha + psum;
  m_run = m_new;
  acc[0] *= alpha;
  acc[1] *= alpha;

  // V^T operand rows: lane group g = lane / 16 reads rows kbase + e (e = its
  // source lane's (lane & 15) / 4) at head dims d0 + 4 (lane & 3) .. + 3
  const int g = lane >> 4, e = (lane & 15) >> 2, q = lane & 3;
  const int hf = lane >> 5;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      // P^T: lane half hf holds keys 16u + 4hf + 0..3 and 16u + 8 + 4hf + 0..3
      // of the 32-key block in s[kb][8u .. 8u + 7]
      bf16x8 pb;
#pragma unroll
      for (int j = 0; j < 8; ++j) pb[j] = (bf16)s[kb][8 * u + j];
#pragma unroll
      for (int db = 0; db < 2; ++db) {
        const int c = db * 4 + (g & 1) * 2 + (q >> 1);  // logical 16-byte chunk
        s16x4 lo, hi;
        {
          const int row = kb * 32 + u * 16 + 4 * hf + e;
          lo = read_tr(vt + row * 128 + ((c ^ swz(row)) << 4) + (q & 1) * 8);
        }
        {
          const int row = kb * 32 + u * 16 + 8 + 4 * hf + e;
          hi = read_tr(vt + row * 128 + ((c ^ swz(row)) << 4) + (q & 1) * 8);
        }
        const s16x4 v8[2] = {lo, hi};
        const bf16x8 va = *reinterpret_cast<const bf16x8 *>(v8);
        acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb, acc[db], 0, 0, 0);
      }
    }
}

}  // namespace strm

// SCORES (the selection layer, Section 4.2): the workgroup of query chunk 0,
// which holds the image's generating rows (its first n_gen[b] <= 16 QB rows),
// then writes the attention mass each key receives from them,
// a.scores[b][h][j].  Its wavefronts put the final row maximum and
// normaliser of those rows in LDS and stream the K tiles once more; wavefront
// w takes key block w % 2 of each tile for generating block w / 2: S = Q K^T
// (one lane per key), the probabilities with the final statistics, summed
// over the block's rows; the blocks' sums are added in block order.
template <int QB, bool SCORES = false>
__global__ __launch_bounds__(QB * 64) void attn_reg_kernel(AttnArgs a, int chunks) {
  using namespace strm;
  constexpr int NT = QB * 64;
  constexpr int CPL = 1024 / NT;  // 16-byte chunks per lane per tile (K and V)
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * kSlotBytes];

  const int id = xcd_remap(blockIdx.x, gridDim.x);
  const int bh = id / chunks, chunk = id - bh * chunks;
  const int b = bh / a.n_heads, h = bh - b * a.n_heads;
  const int r0 = a.a_off ? a.a_off[b] : b * a.a_max;
  const int na = a.a_off ? a.a_off[b + 1] - r0 : a.a_max;
  const int q0 = chunk * QB * 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int N = a.n_tokens, D = a.d_model, nt = N / TK;
  if (q0 >= na) {  // uniform over the workgroup
    if (SCORES && chunk == 0)  // no active row: no key receives any mass
      for (int j = tid; j < N; j += NT) a.scores[(size_t)bh * N + j] = 0.f;
    return;
  }
  const bf16 *kg = static_cast<const bf16 *>(a.k_cache) + (size_t)bh * N * 64;
  const bf16 *vg = static_cast<const bf16 *>(a.v_cache) + (size_t)bh * N * 64;

  const int qi = q0 + wave * 32 + (lane & 31);
  const bf16 *qrow = static_cast<const bf16 *>(a.q) + (size_t)(r0 + min(qi, na - 1)) * D + h * 64;
  bf16x8 qf[4];
#pragma unroll
  for (int s = 0; s < 4; ++s)
    qf[s] = *reinterpret_cast<const bf16x8 *>(qrow + s * 16 + (lane >> 5) * 8);

  // Chunk j of a tile (j = i * NT + tid): matrix j / 512 (K, V), row (j % 512)
  // / 8, logical chunk j % 8; coalesced in global memory, permuted in LDS.
  // Every load is unconditional (a tile index past the last repeats the last
  // tile, which the L2 still holds), so the waits the compiler places count
  // exactly the loads issued after the ones a store needs.
  u32x4 rt[CPL];
  auto gload = [&](u32x4 (&r)[CPL], int t) {
    const size_t off = (size_t)min(t, nt - 1) * TK * 64;
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      const int j = i * NT + tid;
      r[i] = *reinterpret_cast<const u32x4 *>((j < 512 ? kg : vg) + off + (j & 511) * 8);
    }
  };
  auto sstore = [&](const u32x4 (&r)[CPL], int buf) {
    unsigned char *slot = smem + buf * kSlotBytes;
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      const int j = i * NT + tid;
      const int row = (j & 511) >> 3, c = j & 7;
      *reinterpret_cast<u32x4 *>(slot + (j >> 9) * 8192 + row * 128 + ((c ^ swz(row)) << 4)) = r[i];
    }
  };

  const float sl2 = 1.4426950408889634f / 8.0f;  // log2(e) / sqrt(64)
  float m_run = -INFINITY, l_run = 0.f;
  f32x16 acc[2] = {f32x16{}, f32x16{}};
  gload(rt, 0);
  sstore(rt, 0);
  __syncthreads();
  // Tile t is in LDS slot t & 1 and the registers are free again: they take
  // tile t + 1 while tile t computes, then it goes into the other slot.  The
  // loop is unrolled by two so that each step's slot is a constant (its LDS
  // offsets fold into the reads' immediates).  The scheduling barriers keep
  // the stores of the next tile (and the waits for its loads) behind the
  // whole tile step, which would otherwise start them, and wait, in the
  // middle of it.
  // A wavefront whose 32 queries all lie past the active set (the last query
  // chunk of a long sequence) keeps loading, storing and meeting the
  // barriers but skips the tile step, leaving its SIMD to the others.
  const bool live = q0 + wave * 32 < na;  // uniform over the wavefront
  auto step = [&](int t, auto slot) {
    constexpr int SL = decltype(slot)::value;
    gload(rt, t + 1);
    __builtin_amdgcn_sched_barrier(0);
    if (live) tile(smem + SL * kSlotBytes, qf, acc, m_run, l_run, sl2, lane);
    __builtin_amdgcn_sched_barrier(0);
    sstore(rt, SL ^ 1);
    __syncthreads();
  };
  int t = 0;
  for (; t + 2 <= nt; t += 2) {
    step(t, std::integral_constant<int, 0>{});
    step(t + 1, std::integral_constant<int, 1>{});
  }
  if (t < nt) step(t, std::integral_constant<int, 0>{});

  const float inv = 1.0f / (l_run + __shfl_xor(l_run, 32, 64));
  if (qi < na) {
    bf16 *orow = static_cast<bf16 *>(a.o) + (size_t)(r0 + qi) * D + h * 64;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        const int dh0 = db * 32 + gq * 8 + (lane >> 5) * 4;
        bf16x4 pk = {(bf16)(acc[db][4 * gq + 0] * inv), (bf16)(acc[db][4 * gq + 1] * inv),
                     (bf16)(acc[db][4 * gq + 2] * inv), (bf16)(acc[db][4 * gq + 3] * inv)};
        *reinterpret_cast<bf16x4 *>(orow + dh0) = pk;
      }
  }
  if constexpr (SCORES) {
    if (chunk != 0) return;  // uniform over the workgroup
    constexpr int CPK = 512 / NT;  // K chunks per lane per tile
    const int n_gen = a.n_gen[b];
    const int gb_n = (n_gen + 31) / 32;
    // LDS: K tiles in the K halves of the two slots; the blocks' per-key sums
    // in slot 0's V half; the statistics in slot 1's V half
    float *part = reinterpret_cast<float *>(smem + 8192);
    float *st_mx = reinterpret_cast<float *>(smem + kSlotBytes + 8192);
    float *st_iv = st_mx + QB * 32;
    // (the main loop ended on a barrier: no wavefront reads the slots again)
    if (lane < 32) {
      const int row = wave * 32 + lane;            // query qi of this lane
      st_mx[row] = qi < n_gen ? m_run : INFINITY;  // rows past n_gen: probability 0
      st_iv[row] = qi < n_gen ? inv : 0.f;
    }
    const int kb = wave & 1, gb = wave >> 1, hf = lane >> 5;
    const bool active = gb < gb_n;
    bf16x8 qg[4];
    {
      const int row = r0 + min(gb * 32 + (lane & 31), na - 1);
      const bf16 *qr = static_cast<const bf16 *>(a.q) + (size_t)row * D + h * 64;
#pragma unroll
      for (int s2 = 0; s2 < 4; ++s2)
        qg[s2] = *reinterpret_cast<const bf16x8 *>(qr + s2 * 16 + hf * 8);
    }
    u32x4 rk[CPK];
    auto kload = [&](int tk) {
      const size_t off = (size_t)min(tk, nt - 1) * TK * 64;
#pragma unroll
      for (int i = 0; i < CPK; ++i)
        rk[i] = *reinterpret_cast<const u32x4 *>(kg + off + (i * NT + tid) * 8);
    };
    auto kstore = [&](int buf) {
      unsigned char *slot = smem + buf * kSlotBytes;
#pragma unroll
      for (int i = 0; i < CPK; ++i) {
        const int j = i * NT + tid, row = j >> 3, c = j & 7;
        *reinterpret_cast<u32x4 *>(slot + row * 128 + ((c ^ swz(row)) << 4)) = rk[i];
      }
    };
    __syncthreads();  // the statistics are in LDS
    f32x4 mx[4], iv[4];  // rows gb*32 + 8 g + 4 hf + 0..3 of the accumulator
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int r = min(gb, QB - 1) * 32 + 8 * g + 4 * hf;
      mx[g] = *reinterpret_cast<const f32x4 *>(st_mx + r);
      iv[g] = *reinterpret_cast<const f32x4 *>(st_iv + r);
    }
    kload(0);
    kstore(0);
    __syncthreads();
    for (int tk = 0; tk < nt; ++tk) {
      kload(tk + 1);
      __builtin_amdgcn_sched_barrier(0);
      if (active) {
        const unsigned char *kt = smem + (tk & 1) * kSlotBytes;
        const int row = kb * 32 + (lane & 31);
        f32x16 sc = f32x16{};
#pragma unroll
        for (int st = 0; st < 4; ++st) {
          const int c = st * 2 + hf;
          const bf16x8 ka =
              *reinterpret_cast<const bf16x8 *>(kt + row * 128 + ((c ^ swz(row)) << 4));
          sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qg[st], ka, sc, 0, 0, 0);
        }
        float p = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r)
          p += __builtin_amdgcn_exp2f(fmaf(sc[r], sl2, -mx[r >> 2][r & 3])) * iv[r >> 2][r & 3];
        p += __shfl_xor(p, 32, 64);
        if (lane < 32) part[gb * 64 + kb * 32 + lane] = p;
      }
      __syncthreads();
      if (wave == 0) {
        float tot = 0.f;
        for (int g2 = 0; g2 < gb_n; ++g2) tot += part[g2 * 64 + lane];
        a.scores[(size_t)bh * N + tk * TK + lane] = tot;
      }
      __builtin_amdgcn_sched_barrier(0);
      kstore((tk + 1) & 1);
      __syncthreads();
    }
  }
}

// ------------------------------------------------------------ general streaming kernel
//
// Every other shape: head width 80, key counts that are no multiple of a tile,
// two key segments, and calls with too few (image, head) pairs to fill the
// chip.  The tile step and LDS layout follow attn_reg_kernel (row-major K and
// V, V^T from the transposing LDS read); in addition
//  - key tiles of the first segment are followed by those of the second, and a
//    segment's last tile may be partial (ALIGNED: none is, and no masked tile
//    step is compiled);
//  - KS groups of QB wavefronts share a workgroup: group g takes the key tiles
//    t = g mod KS with LDS slots of its own, and the groups' (maximum, sum,
//    output) are merged in group order at the end.  With few workgroups a
//    compute unit then walks KS tiles at a time instead of one;
//  - stats (optional) receives each row's final maximum (log2 domain) and
//    1 / sum, which the stand-alone score pass reads.
// Head width 80: K rows of 176 and V rows of 192 bytes, so that the 16 rows of
// a K fragment read and the 4 rows of a V^T read start on distinct bank
// groups without a permutation; the V^T rows past 80 are whatever the padding
// holds and only reach output rows that are never stored.
namespace gen {

template <int DH>
struct Lay {
  static constexpr bool SWZ = DH == 64;
  static constexpr int CPR = DH / 8;                 // 16-byte chunks per row
  static constexpr int KSTR = SWZ ? 128 : 176;       // bytes per K row
  static constexpr int VSTR = SWZ ? 128 : 192;       // bytes per V row
  static constexpr int VOFF = TK * KSTR;
  static constexpr int SLOT = TK * (KSTR + VSTR);
  static constexpr int ODB = (DH + 31) / 32;
  __device__ __forceinline__ static int k_at(int row, int c) {
    return row * KSTR + ((SWZ ? c ^ strm::swz(row) : c) << 4);
  }
  __device__ __forceinline__ static int v_at(int row, int c) {
    return VOFF + row * VSTR + ((SWZ ? c ^ strm::swz(row) : c) << 4);
  }
};

// One tile of the online softmax (as strm::tile) of which the first `left`
// keys exist (uniform).  PART: the state covers a part of the keys only, whose
// logits may all be -inf (infinite keys) while others' are not: a maximum of
// -inf then scales nothing instead of making the state NaN.
template <int DH, bool ALIGNED, bool PART>
__device__ __forceinline__ void tile(const unsigned char *slot, const bf16x8 (&qf)[DH / 16],
                                     f32x16 (&acc)[Lay<DH>::ODB], float &m_run, float &l_run,
                                     float sl2, int left, int lane) {
  using L = Lay<DH>;
  f32x16 s[2];
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    s[kb] = f32x16{};
    const int row = kb * 32 + (lane & 31);
#pragma unroll
    for (int st = 0; st < DH / 16; ++st) {
      const bf16x8 ka =
          *reinterpret_cast<const bf16x8 *>(slot + L::k_at(row, st * 2 + (lane >> 5)));
      s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qf[st], s[kb], 0, 0, 0);
    }
  }
  if constexpr (!ALIGNED) {
    if (left < TK) {
      asm volatile("");  // keeps the branch: if-converted, every tile would pay for the mask
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (kb * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3) >= left) s[kb][r] = -INFINITY;
    }
  }
  float mx = -INFINITY;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kb][r]);
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
  const float m_new = fmaxf(m_run, mx * sl2);
  const float m_ref = PART && m_new == -INFINITY ? 0.f : m_new;
  const float alpha = __builtin_amdgcn_exp2f(m_run - m_ref);
  float psum = 0.f;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float p = __builtin_amdgcn_exp2f(fmaf(s[kb][r], sl2, -m_ref));
      s[kb][r] = p;
      psum += p;
    }
  l_run = l_run * alpha + psum;
  m_run = m_new;
#pragma unroll
  for (int d = 0; d < L::ODB; ++d) acc[d] *= alpha;
  const int g = lane >> 4, e = (lane & 15) >> 2, q = lane & 3, hf = lane >> 5;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      bf16x8 pb;
#pragma unroll
      for (int j = 0; j < 8; ++j) pb[j] = (bf16)s[kb][8 * u + j];
#pragma unroll
      for (int db = 0; db < L::ODB; ++db) {
        const int c = db * 4 + (g & 1) * 2 + (q >> 1);
        const int row = kb * 32 + u * 16 + 4 * hf + e;
        const strm::s16x4 v8[2] = {strm::read_tr(slot + L::v_at(row, c) + (q & 1) * 8),
                                   strm::read_tr(slot + L::v_at(row + 8, c) + (q & 1) * 8)};
        const bf16x8 va = *reinterpret_cast<const bf16x8 *>(v8);
        acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb, acc[db], 0, 0, 0);
      }
    }
}

}  // namespace gen

template <int DH, int QB, int KS, bool SEG2, bool ALIGNED>
__global__ __launch_bounds__(QB *KS * 64) void attn_gen_kernel(AttnArgs a, int chunks) {
  using L = gen::Lay<DH>;
  constexpr int GT = QB * 64;                        // threads of a key group
  constexpr int MPL = 512 / GT;                      // chunks 0..7 of 64 rows: per lane
  constexpr int TAIL = DH == 80 ? 256 : 0;           // chunks 8 and 9 of K's and V's rows
  constexpr int TPL = TAIL / GT;
  static_assert(512 % GT == 0 && TAIL % GT == 0, "whole chunks per lane");
  constexpr int kMerge = KS > 1 ? (KS - 1) * QB * (L::ODB * 16 + 2) * 256 : 0;
  // A group of one wavefront needs no second slot (nor barriers): its LDS
  // operations are in order, so it overwrites a tile once it has read it, and
  // twice as many workgroups fit.
  constexpr int SLOTS = QB == 1 ? 1 : 2;
  constexpr int kTiles = SLOTS * KS * L::SLOT;
  constexpr int kSmem = kTiles > kMerge ? kTiles : kMerge;
  auto group_sync = [] {
    if constexpr (QB == 1) __builtin_amdgcn_wave_barrier();
    else __syncthreads();
  };
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kSmem];

  const int id = xcd_remap(blockIdx.x, gridDim.x);
  const int bh = id / chunks, chunk = id - bh * chunks;
  const int b = bh / a.n_heads, h = bh - b * a.n_heads;
  const int r0 = a.a_off ? a.a_off[b] : b * a.a_max;
  const int na = a.a_off ? a.a_off[b + 1] - r0 : a.a_max;
  const int q0 = chunk * QB * 32;
  if (q0 >= na) return;  // uniform over the workgroup

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave / QB, qb = wave - grp * QB;
  const int gt = qb * 64 + lane;
  const int N1 = a.n_tokens, N2 = SEG2 ? a.n2 : 0, D = a.d_model;
  const bf16 *kg = static_cast<const bf16 *>(a.k_cache) + (size_t)bh * N1 * DH;
  const bf16 *vg = static_cast<const bf16 *>(a.v_cache) + (size_t)bh * N1 * DH;
  const bf16 *kg2 = SEG2 ? static_cast<const bf16 *>(a.k2) + (size_t)bh * N2 * DH : kg;
  const bf16 *vg2 = SEG2 ? static_cast<const bf16 *>(a.v2) + (size_t)bh * N2 * DH : vg;
  const int nt1 = (N1 + TK - 1) / TK, nt = nt1 + (N2 + TK - 1) / TK;
  // rows of tile t that exist (>= 1), and its first row in K and V
  auto tile_of = [&](int t, const bf16 *&kb, const bf16 *&vb) {
    const bool s1 = !SEG2 || t < nt1;
    const int t0 = (s1 ? t : t - nt1) * TK;
    kb = (s1 ? kg : kg2) + (size_t)t0 * DH;
    vb = (s1 ? vg : vg2) + (size_t)t0 * DH;
    return (s1 ? N1 : N2) - t0;
  };

  const int qi = q0 + qb * 32 + (lane & 31);
  const bf16 *qrow = static_cast<const bf16 *>(a.q) + (size_t)(r0 + min(qi, na - 1)) * D + h * DH;
  bf16x8 qf[DH / 16];
#pragma unroll
  for (int s = 0; s < DH / 16; ++s)
    qf[s] = *reinterpret_cast<const bf16x8 *>(qrow + s * 16 + (lane >> 5) * 8);

  // Lane gt moves chunk gt % 8 of rows gt / 8 + (GT / 8) i of K and V and, at
  // head width 80, tail chunks 8 + gt % 2 (rows of K, then of V).  Loads are
  // unconditional: rows past a segment's end repeat its last one.
  u32x4 rk[MPL], rv[MPL], rtl[TPL ? TPL : 1];
  auto gload = [&](int t) {
    const bf16 *kb, *vb;
    const int last = tile_of(min(t, nt - 1), kb, vb) - 1;
#pragma unroll
    for (int i = 0; i < MPL; ++i) {
      const int row = (gt >> 3) + i * (GT / 8);
      const uint32_t off = (uint32_t)((ALIGNED ? row : min(row, last)) * DH + (gt & 7) * 8);
      rk[i] = *reinterpret_cast<const u32x4 *>(kb + off);
      rv[i] = *reinterpret_cast<const u32x4 *>(vb + off);
    }
#pragma unroll
    for (int i = 0; i < TPL; ++i) {
      const int j = i * GT + gt, row = (j & 127) >> 1;
      const uint32_t off = (uint32_t)((ALIGNED ? row : min(row, last)) * DH + 64 + (j & 1) * 8);
      rtl[i] = *reinterpret_cast<const u32x4 *>((j < 128 ? kb : vb) + off);
    }
  };
  auto sstore = [&](unsigned char *slot) {
#pragma unroll
    for (int i = 0; i < MPL; ++i) {
      const int row = (gt >> 3) + i * (GT / 8);
      *reinterpret_cast<u32x4 *>(slot + L::k_at(row, gt & 7)) = rk[i];
      *reinterpret_cast<u32x4 *>(slot + L::v_at(row, gt & 7)) = rv[i];
    }
#pragma unroll
    for (int i = 0; i < TPL; ++i) {
      const int j = i * GT + gt, row = (j & 127) >> 1, c = 8 + (j & 1);
      *reinterpret_cast<u32x4 *>(slot + (j < 128 ? L::k_at(row, c) : L::v_at(row, c))) = rtl[i];
    }
  };

  const float sl2 = 1.4426950408889634f / sqrtf((float)DH);  // log2(e) / sqrt(d_h)
  float m_run = -INFINITY, l_run = 0.f;
  f32x16 acc[L::ODB];
#pragma unroll
  for (int d = 0; d < L::ODB; ++d) acc[d] = f32x16{};
  // a wavefront whose queries all lie past the active set only moves tiles
  const bool live = q0 + qb * 32 < na;
  unsigned char *slots = smem + grp * SLOTS * L::SLOT;
  gload(grp);
  sstore(slots);
  group_sync();
  const int rounds = (nt + KS - 1) / KS;
#pragma unroll 1
  for (int it = 0; it < rounds; ++it) {
    const int t = it * KS + grp;
    gload(t + KS);
    __builtin_amdgcn_sched_barrier(0);
    const unsigned char *sp = slots + (it & (SLOTS - 1)) * L::SLOT;
    if (live && t < nt) {
      const bf16 *kb, *vb;
      const int left = ALIGNED ? TK : tile_of(t, kb, vb);
      gen::tile<DH, ALIGNED, (KS > 1)>(sp, qf, acc, m_run, l_run, sl2, left, lane);
    }
    __builtin_amdgcn_sched_barrier(0);
    sstore(slots + ((it + 1) & (SLOTS - 1)) * L::SLOT);
    group_sync();
  }

  l_run += __shfl_xor(l_run, 32, 64);
  if constexpr (KS > 1) {
    if constexpr (QB == 1) __syncthreads();  // every group is done with its slot
    constexpr int REC = (L::ODB * 16 + 2) * 64;  // floats per wavefront
    float *rec = reinterpret_cast<float *>(smem) + ((grp - 1) * QB + qb) * REC + lane;
    if (grp > 0) {
      rec[0] = m_run;
      rec[64] = l_run;
#pragma unroll
      for (int d = 0; d < L::ODB; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) rec[(2 + d * 16 + r) * 64] = acc[d][r];
    }
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int g2 = 0; g2 < KS - 1; ++g2) {
      const float *o2 = reinterpret_cast<const float *>(smem) + (g2 * QB + qb) * REC + lane;
      const float m2 = o2[0], m_new = fmaxf(m_run, m2);
      const float a1 = __builtin_amdgcn_exp2f(m_run - m_new);
      const float a2 = __builtin_amdgcn_exp2f(m2 - m_new);
      l_run = l_run * a1 + o2[64] * a2;
      m_run = m_new;
#pragma unroll
      for (int d = 0; d < L::ODB; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          acc[d][r] = acc[d][r] * a1 + o2[(2 + d * 16 + r) * 64] * a2;
    }
  }
  const float inv = 1.0f / l_run;
  if (qi < na) {
    bf16 *orow = static_cast<bf16 *>(a.o) + (size_t)(r0 + qi) * D + h * DH;
#pragma unroll
    for (int d = 0; d < L::ODB; ++d)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int dh0 = d * 32 + g * 8 + (lane >> 5) * 4;
        if (dh0 < DH) {
          bf16x4 pk = {(bf16)(acc[d][4 * g + 0] * inv), (bf16)(acc[d][4 * g + 1] * inv),
                       (bf16)(acc[d][4 * g + 2] * inv), (bf16)(acc[d][4 * g + 3] * inv)};
          *reinterpret_cast<bf16x4 *>(orow + dh0) = pk;
        }
      }
    if (a.stats && lane < 32) {
      float *st = a.stats + ((size_t)(r0 + qi) * a.n_heads + h) * 2;
      st[0] = m_run;
      st[1] = inv;
    }
  }
}

// Every query of an image in one workgroup and every key resident in LDS
// (layers where all N <= NTL * 64 tokens are active): one workgroup per
// (image, head); wavefront w owns the NQB 32-query blocks w, w + NW, ...  All
// K/V tiles are loaded at once (registers, then LDS: one memory latency per
// workgroup instead of one per tile) and read once per (image, head), after
// which each wavefront runs the online softmax over the resident tiles with
// no further loads or barriers.  With SWZ (head width 64) the tiles take
// 80 KB, so two workgroups share a CU and one's loads overlap the other's
// arithmetic.
//
// SCORES (the selection layer, Section 4.2): the kernel also writes the
// attention mass each key receives from the image's generating rows (its
// first n_gen[b] active rows), a.scores[b][h][j] = sum over those rows i of
// softmax_j(q_i . k_j / sqrt(d_h)), from the K tiles it holds.  Each
// wavefront keeps the final row maximum and normaliser of its generating
// rows; once every wavefront is done with the V tiles, those go to LDS in
// their place, and the wavefronts split the key tiles: for each key, S = Q
// K^T over the generating rows (one lane per key), the probabilities with
// the final statistics, summed over the rows in a fixed order.
template <int DH, int NW, int NTL, int NQB, bool SWZ, bool SCORES = false>
__global__ __launch_bounds__(NW * 64) void attn_resident_kernel(AttnArgs a) {
  constexpr int NT = NW * 64;
  constexpr int ODB = (DH + 31) / 32;
  constexpr int DHV = ODB * 32;
  constexpr int KT = SWZ ? TK * 64 : TK * (DH + 8);     // elements per K tile
  constexpr int VT = SWZ ? DHV * 64 : DHV * (TK + 8);   // elements per V^T tile
  constexpr int CPR = DH / 8;
  constexpr int TCH = TK * CPR;
  constexpr int LPT = (TCH + NT - 1) / NT;
  constexpr int VPCH = TCH / 2;
  constexpr int LPV = (VPCH + NT - 1) / NT;
  constexpr int QS = DH / 16;
  __shared__ __attribute__((aligned(16))) bf16 Ks[NTL][KT];
  __shared__ __attribute__((aligned(16))) bf16 Vt[NTL][VT];

  const int bh = xcd_remap(blockIdx.x, gridDim.x);
  const int b = bh / a.n_heads, h = bh - b * a.n_heads;
  const int r0 = a.a_off ? a.a_off[b] : b * a.a_max;
  const int na = a.a_off ? a.a_off[b + 1] - r0 : a.a_max;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int N = a.n_tokens, D = a.d_model;
  const int ntiles = (N + TK - 1) / TK;  // <= NTL (host-checked)
  const bf16 *kg = static_cast<const bf16 *>(a.k_cache) + (size_t)(b * a.n_heads + h) * N * DH;
  const bf16 *vg = static_cast<const bf16 *>(a.v_cache) + (size_t)(b * a.n_heads + h) * N * DH;

  if constexpr (DHV > DH) {  // V^T rows past DH (padding to a multiple of 32) hold zeros
    for (int i = tid; i < NTL * (DHV - DH) * (TK + 8); i += NT) {
      const int t = i / ((DHV - DH) * (TK + 8)), rem = i % ((DHV - DH) * (TK + 8));
      Vt[t][DH * (TK + 8) + rem] = (bf16)0.0f;
    }
  }
  // this wavefront's queries of every block it computes, issued first so
  // that their latency hides behind the K/V loads instead of stalling the
  // start of each block
  bf16x8 qall[NQB][QS];
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    const int wq0 = (qb * NW + wave) * 32;
    if (wq0 < na) {
      const int qi = wq0 + (lane & 31);
      const bf16 *qrow =
          static_cast<const bf16 *>(a.q) + (size_t)(r0 + min(qi, na - 1)) * D + h * DH;
#pragma unroll
      for (int st = 0; st < QS; ++st)
        qall[qb][st] = *reinterpret_cast<const bf16x8 *>(qrow + st * 16 + (lane >> 5) * 8);
    }
  }
  // all tiles' loads, then all LDS writes
  u32x4 rk[NTL][LPT], rv0[NTL][LPV], rv1[NTL][LPV];
#pragma unroll
  for (int t = 0; t < NTL; ++t) {
    if (t >= ntiles) break;
    const int t0 = t * TK;
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      const int c = i * NT + tid;
      if (c < TCH) {
        const int key = min(t0 + c / CPR, N - 1), d = (c % CPR) * 8;
        rk[t][i] = *reinterpret_cast<const u32x4 *>(kg + (size_t)key * DH + d);
      }
    }
#pragma unroll
    for (int i = 0; i < LPV; ++i) {
      const int c = i * NT + tid;
      if (c < VPCH) {
        const int kp = c / CPR, d = (c % CPR) * 8;
        const int k0 = min(t0 + 2 * kp, N - 1), k1 = min(t0 + 2 * kp + 1, N - 1);
        rv0[t][i] = *reinterpret_cast<const u32x4 *>(vg + (size_t)k0 * DH + d);
        rv1[t][i] = *reinterpret_cast<const u32x4 *>(vg + (size_t)k1 * DH + d);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < NTL; ++t) {
    if (t >= ntiles) break;
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      const int c = i * NT + tid;
      if (c < TCH) {
        const int key = c / CPR, d = (c % CPR) * 8;
        *reinterpret_cast<u32x4 *>(&Ks[t][k_off<DH, SWZ>(key, d)]) = rk[t][i];
      }
    }
#pragma unroll
    for (int i = 0; i < LPV; ++i) {
      const int c = i * NT + tid;
      if (c < VPCH) {
        const int kp = c / CPR, d = (c % CPR) * 8;
        const int pos = ((2 * kp) & ~15) | vperm16((2 * kp) & 15);  // even: a 32-bit pair
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const unsigned w0 = rv0[t][i][e >> 1], w1 = rv1[t][i][e >> 1];
          const unsigned lo = (e & 1) ? (w0 >> 16) : (w0 & 0xFFFFu);
          const unsigned hi = (e & 1) ? (w1 & 0xFFFF0000u) : (w1 << 16);
          *reinterpret_cast<unsigned *>(&Vt[t][vt_off<DH, SWZ>(d + e, pos)]) = lo | hi;
        }
      }
    }
  }
  __syncthreads();

  const float sl2 = 1.4426950408889634f / sqrtf((float)DH);
  const int n_gen = SCORES ? a.n_gen[b] : 0;
  // final statistics of this wavefront's blocks (generating rows only)
  float st_m[NQB], st_inv[NQB];
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    st_m[qb] = INFINITY;
    st_inv[qb] = 0.f;
  }
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    const int wq0 = (qb * NW + wave) * 32;
    if (wq0 >= na) break;  // uniform over the wavefront; no barrier inside the loop
    const int qi = wq0 + (lane & 31);
    const bf16x8 (&qf)[QS] = qall[qb];
    float m_run = -INFINITY, l_run = 0.f;
    f32x16 acc[ODB];
#pragma unroll
    for (int d = 0; d < ODB; ++d) acc[d] = f32x16{};
    for (int t = 0; t < N / TK; ++t)
      attn_tile<DH, SWZ>(Ks[t], Vt[t], qf, acc, m_run, l_run, t * TK, N, sl2, lane);
    if (N % TK)
      attn_tile<DH, SWZ, true>(Ks[N / TK], Vt[N / TK], qf, acc, m_run, l_run, (N / TK) * TK, N,
                               sl2, lane);

    const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    const float inv = 1.0f / l_tot;
    if (SCORES && qi < n_gen) {
      st_m[qb] = m_run;
      st_inv[qb] = inv;
    }
    if (qi < na) {
      bf16 *orow = static_cast<bf16 *>(a.o) + (size_t)(r0 + qi) * D + h * DH;
#pragma unroll
      for (int d = 0; d < ODB; ++d)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int dh0 = d * 32 + g * 8 + (lane >> 5) * 4;
          if (dh0 < DH) {
            bf16x4 pk = {(bf16)(acc[d][4 * g + 0] * inv), (bf16)(acc[d][4 * g + 1] * inv),
                         (bf16)(acc[d][4 * g + 2] * inv), (bf16)(acc[d][4 * g + 3] * inv)};
            *reinterpret_cast<bf16x4 *>(orow + dh0) = pk;
          }
        }
    }
  }
  if constexpr (SCORES) {
    // statistics of generating row i at st_mx[i], st_iv[i], in the V tiles'
    // place; rows at or past n_gen read maximum +inf and normaliser 0, so
    // their probabilities are exactly 0
    const int gb_n = (n_gen + 31) / 32;  // blocks with generating rows
    float *st_mx = reinterpret_cast<float *>(&Vt[0][0]);
    float *st_iv = st_mx + NQB * NW * 32;
    static_assert(2 * NQB * NW * 32 * 4 <= (int)sizeof(Vt), "statistics fit the V tiles");
    __syncthreads();  // every wavefront is done with the V tiles
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      const int row = (qb * NW + wave) * 32 + (lane & 31);
      if (lane < 32 && row < gb_n * 32) {
        st_mx[row] = st_m[qb];
        st_iv[row] = st_inv[qb];
      }
    }
    __syncthreads();
    const int hf = lane >> 5;
    for (int t = wave; t < ntiles; t += NW) {
      float sc[2] = {0.f, 0.f};  // keys t*64 + kb*32 + (lane & 31), this lane's half of the rows
      for (int gb = 0; gb < gb_n; ++gb) {
        const int qi = gb * 32 + (lane & 31);
        const bf16 *qrow =
            static_cast<const bf16 *>(a.q) + (size_t)(r0 + min(qi, na - 1)) * D + h * DH;
        bf16x8 qf[QS];
#pragma unroll
        for (int st = 0; st < QS; ++st)
          qf[st] = *reinterpret_cast<const bf16x8 *>(qrow + st * 16 + hf * 8);
        // rows of register r: gb*32 + 8 (r / 4) + 4 hf + r % 4
        f32x4 mx[4], iv[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          mx[g] = *reinterpret_cast<const f32x4 *>(st_mx + gb * 32 + 8 * g + 4 * hf);
          iv[g] = *reinterpret_cast<const f32x4 *>(st_iv + gb * 32 + 8 * g + 4 * hf);
        }
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
          f32x16 s = f32x16{};
#pragma unroll
          for (int st = 0; st < QS; ++st) {
            const bf16x8 ka = *reinterpret_cast<const bf16x8 *>(
                &Ks[t][k_off<DH, SWZ>(kb * 32 + (lane & 31), st * 16 + hf * 8)]);
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[st], ka, s, 0, 0, 0);
          }
          float part = 0.f;
#pragma unroll
          for (int r = 0; r < 16; ++r)
            part += __builtin_amdgcn_exp2f(fmaf(s[r], sl2, -mx[r >> 2][r & 3])) * iv[r >> 2][r & 3];
          sc[kb] += part;
        }
      }
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const float tot = sc[kb] + __shfl_xor(sc[kb], 32, 64);
        const int key = t * TK + kb * 32 + (lane & 31);
        if (lane < 32 && key < N) a.scores[(size_t)bh * N + key] = tot;
      }
    }
  }
}

constexpr int RES_NTL = 5;    // keys resident: 320
constexpr int RES_QMAX = 320; // queries per workgroup
constexpr int RES_QMIN = 128; // queries up to which the streaming kernels are used
constexpr int RES_SCMIN = 64; // the same at a selection layer whose scores they cannot write

// Query blocks per workgroup of the streaming kernel for a_max rows.
static int reg_qb(int32_t a_max) {
  return a_max <= 32 ? 1 : a_max <= 64 ? 2 : a_max <= 128 ? 4 : 8;
}

// The register-staged kernel of head width 64 for one key segment of whole
// tiles (at least three).
bool attn_streams(int32_t head_dim, int32_t n_tokens, bool two_segments) {
  return head_dim == 64 && !two_segments && n_tokens % TK == 0 && n_tokens >= 3 * TK;
}

// Whether that kernel can write the score pass: the generating rows within
// query chunk 0, and one (key block, generating block) pair per wavefront.
static bool streams_scores(int32_t a_max, int32_t n_tokens, int32_t head_dim, int32_t gen_max) {
  return attn_streams(head_dim, n_tokens, false) && 2 * ((gen_max + 31) / 32) <= reg_qb(a_max);
}

// Whether the resident kernel writes the score pass: all queries and keys
// within one workgroup's reach and more than 128 queries in some image, or more
// than 64 where the streaming kernel cannot, because a separate score pass
// costs more than the streaming attention saves there (one layer, scores and
// selection, with it / on the resident kernel, 65 to 128 rows: 4 images, heads
// of 80, 320 keys 88.2 / 82.7 us; 64 images 379 / 372; heads of 64, 229 keys
// 72.7 / 67.3 and 252 / 234).
static bool resident_scores(int32_t a_max, int32_t n_tokens, int32_t head_dim, int32_t gen_max) {
  const int q_min =
      streams_scores(a_max, n_tokens, head_dim, gen_max) ? RES_QMIN : RES_SCMIN;
  return a_max > q_min && a_max <= RES_QMAX && n_tokens <= RES_NTL * TK;
}

// Host choice of the resident kernel: more than 128 active queries in some
// image (below that one streaming workgroup of four wavefronts covers an
// (image, head), reads each K/V element once as well and skips wavefronts
// without queries: 64 images x 16 heads with 9..71 queries of width 64 took
// 30.7 us on the resident kernel, and the 4-layer call 652 us on it against
// 631), all of them and all keys within one workgroup's reach, one key segment.
// With fewer (image, head) pairs than two workgroups per compute unit the
// streaming kernel spreads a pair's queries over several workgroups instead
// (4 images x 12 heads x 320 tokens, 12 layers of a full and a cache-aware step:
// 1761 us with it, 1655 without); from there on the two are level, and the
// resident one is ahead when another image range runs beside it (two 64-image
// ranges of 16 heads: 12.94 against 13.09 ms for a full and a cache-aware step
// of 8 layers).  Both sum in the same order.
bool attn_resident(const AttnArgs &a) {
  if (a.scores) return resident_scores(a.a_max, a.n_tokens, a.head_dim, a.gen_max);
  return !a.k2 && a.a_max > RES_QMIN && a.a_max <= RES_QMAX && a.n_tokens <= RES_NTL * TK &&
         (int64_t)a.batch * a.n_heads >= 2 * device_cu_count();
}

bool attn_fuses_scores(int32_t a_max, int32_t n_tokens, int32_t head_dim, int32_t gen_max) {
  return resident_scores(a_max, n_tokens, head_dim, gen_max) ||
         streams_scores(a_max, n_tokens, head_dim, gen_max);
}

template <int DH, int QB, int KS, bool SEG2>
static hipError_t run_attn_gen(const AttnArgs &a, hipStream_t s) {
  const int chunks = (a.a_max + QB * 32 - 1) / (QB * 32);
  const int grid = a.batch * a.n_heads * chunks;
  if (a.n_tokens % TK == 0 && (!SEG2 || a.n2 % TK == 0))
    launch_kernel(attn_gen_kernel<DH, QB, KS, SEG2, true>, grid, QB * KS * 64, 0, s, a, chunks);
  else
    launch_kernel(attn_gen_kernel<DH, QB, KS, SEG2, false>, grid, QB * KS * 64, 0, s, a, chunks);
  return hipGetLastError();
}

template <int QB>
static hipError_t run_attn_reg(const AttnArgs &a, hipStream_t s) {
  const int chunks = (a.a_max + QB * 32 - 1) / (QB * 32);
  const int grid = a.batch * a.n_heads * chunks;
  if (a.scores)
    launch_kernel(attn_reg_kernel<QB, true>, grid, QB * 64, 0, s, a, chunks);
  else
    launch_kernel(attn_reg_kernel<QB>, grid, QB * 64, 0, s, a, chunks);
  return hipGetLastError();
}


// Query blocks per workgroup, key groups, and whether attn_reg_kernel runs.
struct AttnShape {
  int qb, ks;
  bool reg;
};

// Launch shape of the streaming kernels.  QB wavefronts of 32 queries per
// workgroup: as many as the largest active set needs, up to four (eight in
// attn_reg_kernel: one pass over K/V per 256 queries).  The stand-alone
// segment attention takes two key groups of at most two query blocks where
// its grid is then no more than one workgroup per compute unit: a workgroup's
// time is its serial walk over the key tiles (16 images x 16 heads of width
// 80, 45 queries x 1548 keys: 33.4 us with one group, 26.4 with two; at 512
// workgroups or more two groups only shrink the number resident: 19.1 against
// 22.2 us at 1024).  A layer step never does: its images' results must not
// depend on how many images share the call, and two groups sum in another
// order.
static AttnShape attn_shape(const AttnArgs &a) {
  const int q = a.a_max <= 32 ? 1 : 2;
  const bool split = !a.a_off && (int64_t)a.batch * a.n_heads *
                                         ((a.a_max + 32 * q - 1) / (32 * q)) <=
                                     device_cu_count();
  if (split) return {q, 2, false};
  if (attn_streams(a.head_dim, a.n_tokens, a.k2 != nullptr) && !a.stats) {
    // eight blocks (fewer passes over K/V) only where that leaves four
    // workgroups per compute unit: a step of 8 layers with 2 x 4 images x 16
    // heads x 1088 queries measured 2602 us with eight and 2546 with four
    const int qb = reg_qb(a.a_max);
    const int64_t wgs8 = (int64_t)a.batch * a.n_heads * ((a.a_max + 255) / 256);
    if (qb == 8 && !a.scores && wgs8 < 4 * device_cu_count() && a.a_max > 256) return {4, 1, true};
    return {qb, 1, true};
  }
  return {std::min(reg_qb(a.a_max), 4), 1, false};
}

int attn_query_blocks(const AttnArgs &a) { return attn_shape(a).qb; }

template <int DH, bool SEG2>
static hipError_t attn_bf16_nw(const AttnArgs &a, hipStream_t s) {
  const AttnShape f = attn_shape(a);
  if constexpr (DH == 64 && !SEG2) {
    if (f.reg) {
      switch (f.qb) {
        case 1: return run_attn_reg<1>(a, s);
        case 2: return run_attn_reg<2>(a, s);
        case 4: return run_attn_reg<4>(a, s);
        default: return run_attn_reg<8>(a, s);
      }
    }
  }
  if (f.qb == 1)
    return f.ks == 2 ? run_attn_gen<DH, 1, 2, SEG2>(a, s) : run_attn_gen<DH, 1, 1, SEG2>(a, s);
  if (f.qb == 2)
    return f.ks == 2 ? run_attn_gen<DH, 2, 2, SEG2>(a, s) : run_attn_gen<DH, 2, 1, SEG2>(a, s);
  return run_attn_gen<DH, 4, 1, SEG2>(a, s);
}

template <int DH>
static hipError_t attn_bf16_dispatch(const AttnArgs &a, hipStream_t s) {
  if (a.k2) return attn_bf16_nw<DH, true>(a, s);
  if (attn_resident(a)) {
    const int grid = a.batch * a.n_heads;
    if constexpr (DH == 64) {  // 80 KB of swizzled tiles: two workgroups per CU
      if (a.scores)
        launch_kernel(attn_resident_kernel<DH, 4, RES_NTL, 3, true, true>, grid, 4 * 64, 0, s, a);
      else
        launch_kernel(attn_resident_kernel<DH, 4, RES_NTL, 3, true>, grid, 4 * 64, 0, s, a);
    } else {
      if (a.scores)
        launch_kernel(attn_resident_kernel<DH, 10, RES_NTL, 1, false, true>, grid, 10 * 64, 0, s,
                      a);
      else
        launch_kernel(attn_resident_kernel<DH, 10, RES_NTL, 1, false>, grid, 10 * 64, 0, s, a);
    }
    return hipGetLastError();
  }
  return attn_bf16_nw<DH, false>(a, s);
}

// ------------------------------------------------------------ concatenation
//
// The baseline of Appendix B: K and V of the active segment and of the cached
// segment copied into one buffer per (image, head), active rows first.  Per
// (image, head) the destination is two contiguous copies, so chunk j (16
// bytes) of the destination block comes from chunk j of the active block
// (j < na * cpr) or chunk j - na * cpr of the cached block.  Each thread moves
// CPT chunks of K and of V, all loads issued before the stores.  Grid:
// (chunks of a destination block / (256 * CPT), image * head).
constexpr int CONCAT_CPT = 4;

__global__ __launch_bounds__(256) void concat_kv_kernel(u32x4 *__restrict__ kd, u32x4 *__restrict__ vd,
                                                        const u32x4 *__restrict__ ka,
                                                        const u32x4 *__restrict__ va,
                                                        const u32x4 *__restrict__ kc,
                                                        const u32x4 *__restrict__ vc, int a_chunks,
                                                        int c_chunks) {
  const int per = a_chunks + c_chunks;
  const size_t bh = blockIdx.y;
  const int j0 = blockIdx.x * 256 * CONCAT_CPT + threadIdx.x;
  u32x4 kv[CONCAT_CPT], vv[CONCAT_CPT];
#pragma unroll
  for (int u = 0; u < CONCAT_CPT; ++u) {
    const int j = j0 + u * 256;
    if (j < per) {
      const bool act = j < a_chunks;
      const size_t src = act ? bh * a_chunks + j : bh * c_chunks + (j - a_chunks);
      kv[u] = act ? ka[src] : kc[src];
      vv[u] = act ? va[src] : vc[src];
    }
  }
#pragma unroll
  for (int u = 0; u < CONCAT_CPT; ++u) {
    const int j = j0 + u * 256;
    if (j < per) {
      kd[bh * per + j] = kv[u];
      vd[bh * per + j] = vv[u];
    }
  }
}

hipError_t launch_concat_kv(DType dt, void *k_dst, void *v_dst, const void *k_a, const void *v_a,
                            const void *k_c, const void *v_c, int32_t bh, int32_t na, int32_t nc,
                            int32_t head_dim, hipStream_t s) {
  const int es = dt == DType::BF16 ? 2 : 4;
  if ((head_dim * es) % 16 != 0 || bh > 65535) return hipErrorInvalidValue;
  const int cpr = head_dim * es / 16;
  const int per = (na + nc) * cpr;
  if (bh == 0 || per == 0) return hipSuccess;
  const dim3 grid((per + 256 * CONCAT_CPT - 1) / (256 * CONCAT_CPT), bh);
  launch_kernel(concat_kv_kernel, grid, 256, 0, s, static_cast<u32x4 *>(k_dst), static_cast<u32x4 *>(v_dst), static_cast<const u32x4 *>(k_a),
      static_cast<const u32x4 *>(v_a), static_cast<const u32x4 *>(k_c),
      static_cast<const u32x4 *>(v_c), na * cpr, nc * cpr);
  return hipGetLastError();
}

// fp32 attention: one workgroup per (image, head, R active rows).  Four lanes
// share a key (each holds DH / 4 dims in 16-byte pieces, so a load instruction
// covers 64 bytes of 16 keys and two shuffles finish a dot product), the
// logits of every key stay in LDS, the softmax runs over them with exact expf,
// and the output is formed with DH / 4 lanes per key, the lane groups' partial
// sums added in group order.  Its time at a few dozen rows is load latency:
// one wavefront per (row, head) walking its keys one by one took 20 us at 32
// rows x 12 heads x 320 keys.  R = 4 where there are enough rows to fill the
// chip (each K/V element read then serves four rows).
// stats (optional): the row's maximum logit and 1 / sum, [row][head][2].
template <int DH, int R>
__global__ __launch_bounds__(256) void attn_f32_kernel(AttnArgs a, int chunks) {
  constexpr int C4 = DH / 16;       // 16-byte pieces per lane of a key
  constexpr int LPD = DH / 4;       // lanes per key when forming the output
  constexpr int G = 256 / LPD;      // keys in flight there: 16 or 12
  extern __shared__ float smem[];
  float *ps = smem;                 // [R][N]
  float *red = ps + R * a.n_tokens; // [4][R], then the output partials [G][R][DH]
  const int bh = blockIdx.x / chunks, chunk = blockIdx.x - bh * chunks;
  const int b = bh / a.n_heads, h = bh - b * a.n_heads;
  const int r0 = a.a_off[b], na = a.a_off[b + 1] - r0;
  const int q0 = chunk * R;
  if (q0 >= na) return;  // uniform over the workgroup
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int N = a.n_tokens, D = a.d_model;
  const float *kg = static_cast<const float *>(a.k_cache) + (size_t)bh * N * DH;
  const float *vg = static_cast<const float *>(a.v_cache) + (size_t)bh * N * DH;
  const float scale = 1.0f / sqrtf((float)DH);
  const int li = lane & 3;
  f32x4 q[R][C4];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const float *qg =
        static_cast<const float *>(a.q) + (size_t)(r0 + min(q0 + r, na - 1)) * D + h * DH;
#pragma unroll
    for (int c = 0; c < C4; ++c) q[r][c] = *reinterpret_cast<const f32x4 *>(qg + c * 16 + li * 4);
  }
  float mx[R];
#pragma unroll
  for (int r = 0; r < R; ++r) mx[r] = -INFINITY;
#pragma unroll 2
  for (int j0 = 0; j0 < N; j0 += 64) {
    const int j = j0 + (tid >> 2);
    const float *kr = kg + (size_t)min(j, N - 1) * DH + li * 4;
    f32x4 k[C4];
#pragma unroll
    for (int c = 0; c < C4; ++c) k[c] = *reinterpret_cast<const f32x4 *>(kr + c * 16);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float d = 0.f;
#pragma unroll
      for (int c = 0; c < C4; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) d = fmaf(q[r][c][e], k[c][e], d);
      d += __shfl_xor(d, 1, 64);
      d += __shfl_xor(d, 2, 64);
      d *= scale;
      if (j < N) {
        if (li == 0) ps[r * N + j] = d;
        mx[r] = fmaxf(mx[r], d);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    mx[r] = wave_max(mx[r]);
    if (lane == 0) red[wave * R + r] = mx[r];
  }
  __syncthreads();
  float sum[R], inv[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    mx[r] = fmaxf(fmaxf(red[r], red[R + r]), fmaxf(red[2 * R + r], red[3 * R + r]));
    sum[r] = 0.f;
    for (int j = tid; j < N; j += 256) {
      const float e = expf(ps[r * N + j] - mx[r]);
      ps[r * N + j] = e;
      sum[r] += e;
    }
    sum[r] = wave_sum(sum[r]);
  }
  __syncthreads();  // the maxima have been read
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (lane == 0) red[wave * R + r] = sum[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r)
    inv[r] = 1.0f / ((red[r] + red[R + r]) + (red[2 * R + r] + red[3 * R + r]));
  if (a.stats && tid < R && q0 + tid < na) {
    float m_r = 0.f, i_r = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (tid == r) { m_r = mx[r]; i_r = inv[r]; }
    float *st = a.stats + ((size_t)(r0 + q0 + tid) * a.n_heads + h) * 2;
    st[0] = m_r;
    st[1] = i_r;
  }
  __syncthreads();  // the sums have been read: red becomes the output partials
  const int g = tid / LPD, dl = (tid - g * LPD) * 4;
  if (g < G) {
    f32x4 acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = f32x4{};
#pragma unroll 4
    for (int j = g; j < N; j += G) {
      const f32x4 v = *reinterpret_cast<const f32x4 *>(vg + (size_t)j * DH + dl);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const float p = ps[r * N + j];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[r][e] = fmaf(p, v[e], acc[r][e]);
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[(g * R + r) * DH + dl + e] = acc[r][e];
  }
  __syncthreads();
  for (int i = tid; i < R * DH; i += 256) {
    const int r = i / DH, d = i - r * DH;
    if (q0 + r >= na) continue;
    float o = 0.f;
#pragma unroll
    for (int gg = 0; gg < G; ++gg) o += red[(gg * R + r) * DH + d];
    float iv = inv[0];
#pragma unroll
    for (int rr = 1; rr < R; ++rr) iv = r == rr ? inv[rr] : iv;
    static_cast<float *>(a.o)[(size_t)(r0 + q0 + r) * D + h * DH + d] = o * iv;
  }
}

template <int DH, int R>
static hipError_t attn_f32_run(const AttnArgs &a, hipStream_t s) {
  const int chunks = (a.a_max + R - 1) / R;
  constexpr int G = 256 / (DH / 4);
  const size_t lds = ((size_t)R * a.n_tokens + G * R * DH) * sizeof(float);
  launch_kernel(attn_f32_kernel<DH, R>, a.batch * a.n_heads * chunks, 256, lds, s, a, chunks);
  return hipGetLastError();
}

template <int DH>
static hipError_t attn_f32_dispatch(const AttnArgs &a, hipStream_t s) {
  // four rows per workgroup once that still leaves two workgroups per compute
  // unit (and their logits fit 32 KB), else one
  if (a.n_tokens <= 2048 && (int64_t)a.a_total * a.n_heads >= 8LL * device_cu_count())
    return attn_f32_run<DH, 4>(a, s);
  return attn_f32_run<DH, 1>(a, s);
}

hipError_t launch_attention(DType dt, const AttnArgs &a, hipStream_t s) {
  if (a.a_total == 0) return hipSuccess;
  if (a.k2 && dt != DType::BF16) return hipErrorInvalidValue;
  if (dt == DType::BF16) {
    if (a.head_dim == 64) return attn_bf16_dispatch<64>(a, s);
    if (a.head_dim == 80) return attn_bf16_dispatch<80>(a, s);
  } else {
    if (a.head_dim == 64) return attn_f32_dispatch<64>(a, s);
    if (a.head_dim == 80) return attn_f32_dispatch<80>(a, s);
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------- score pass
//
// scores[b][h][j] = sum over the generating rows i (the first n_gen[b] active
// rows of image b) of softmax_j(q_i . k_j / sqrt(d_h)) -- the post-softmax
// attention mass each key receives, one head at a time, from the row
// statistics (maximum and 1 / sum over all N keys) that the attention kernel
// left in a.stats.  One workgroup per (image, head, 64 keys), four lanes per
// key; the generating rows are added in order, so the result is
// deterministic.  (With one workgroup per (image, head) finding the
// statistics itself, the pass took 101 us for 12 heads x 320 keys x 16 rows.)
constexpr int SC_ROWS = 16;  // generating rows staged in LDS at a time

template <typename T, int DH>
__global__ __launch_bounds__(256) void attn_scores_kernel(AttnArgs a,
                                                          const int32_t *__restrict__ n_gen,
                                                          float *__restrict__ scores, int key_wgs) {
  constexpr int C4 = DH / 16;
  __shared__ __attribute__((aligned(16))) float qs[SC_ROWS][DH];
  __shared__ float st[SC_ROWS][2];
  const int N = a.n_tokens, D = a.d_model;
  const int bh = blockIdx.x / key_wgs, kw = blockIdx.x - bh * key_wgs;
  const int b = bh / a.n_heads, h = bh - b * a.n_heads;
  const int tid = threadIdx.x, li = tid & 3, j = kw * 64 + (tid >> 2);
  const int g = n_gen[b], r0 = a.a_off[b];
  const T *kr = static_cast<const T *>(a.k_cache) + ((size_t)bh * N + min(j, N - 1)) * DH + li * 4;
  const T *qg = static_cast<const T *>(a.q);
  f32x4 k[C4];
#pragma unroll
  for (int c = 0; c < C4; ++c) {
    if constexpr (sizeof(T) == 4) {
      k[c] = *reinterpret_cast<const f32x4 *>(kr + c * 16);
    } else {
      const bf16x4 v = *reinterpret_cast<const bf16x4 *>(kr + c * 16);
      k[c] = f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
    }
  }
  // the statistics' domain: natural for fp32 (expf), log2 for bf16
  const float scale = (sizeof(T) == 4 ? 1.0f : 1.4426950408889634f) / sqrtf((float)DH);
  float tot = 0.f;
  for (int g0 = 0; g0 < g; g0 += SC_ROWS) {
    const int nr = min(SC_ROWS, g - g0);
    __syncthreads();
    for (int i = tid; i < nr * DH; i += 256) {
      const int r = i / DH, d = i - r * DH;
      qs[r][d] = to_f32(qg[(size_t)(r0 + g0 + r) * D + h * DH + d]);
    }
    if (tid < 2 * nr)
      st[tid >> 1][tid & 1] = a.stats[((size_t)(r0 + g0 + (tid >> 1)) * a.n_heads + h) * 2 + (tid & 1)];
    __syncthreads();
    for (int r = 0; r < nr; ++r) {
      float d = 0.f;
#pragma unroll
      for (int c = 0; c < C4; ++c) {
        const f32x4 q = *reinterpret_cast<const f32x4 *>(&qs[r][c * 16 + li * 4]);
#pragma unroll
        for (int e = 0; e < 4; ++e) d = fmaf(q[e], k[c][e], d);
      }
      d += __shfl_xor(d, 1, 64);
      d += __shfl_xor(d, 2, 64);
      const float p = sizeof(T) == 4 ? expf(d * scale - st[r][0])
                                     : __builtin_amdgcn_exp2f(fmaf(d, scale, -st[r][0]));
      tot += p * st[r][1];
    }
  }
  if (li == 0 && j < N) scores[(size_t)bh * N + j] = tot;
}

template <typename T, int DH>
static hipError_t scores_dispatch(const AttnArgs &a, const int32_t *n_gen, float *scores,
                                  hipStream_t s) {
  const int key_wgs = (a.n_tokens + 63) / 64;
  launch_kernel(attn_scores_kernel<T, DH>, a.batch * a.n_heads * key_wgs, 256, 0, s, a, n_gen,
                scores, key_wgs);
  return hipGetLastError();
}

hipError_t launch_attn_scores(DType dt, const AttnArgs &a, const int32_t *n_gen, float *scores,
                              hipStream_t s) {
  if (a.batch == 0) return hipSuccess;
  if (!a.stats) return hipErrorInvalidValue;
  if (dt == DType::BF16) {
    if (a.head_dim == 64) return scores_dispatch<bf16, 64>(a, n_gen, scores, s);
    if (a.head_dim == 80) return scores_dispatch<bf16, 80>(a, n_gen, scores, s);
  } else {
    if (a.head_dim == 64) return scores_dispatch<float, 64>(a, n_gen, scores, s);
    if (a.head_dim == 80) return scores_dispatch<float, 80>(a, n_gen, scores, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace marche
