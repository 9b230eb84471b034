// GEMMs whose two operands are both stored token-major: X [K, M] and Y [K, N]
// with the contraction index k (a token of an example) on the rows.
//
// Clipped sum (eq. 3 without the noise; the reweighted second backward of
// Sec. "Ghost Clipping Mechanism"): S = sum_i c_i A_i^T G_i. Stacking the B
// examples' tokens gives one GEMM with K = B*T in which row k of X is scaled
// by c[k / T]. The backward pass is linear in the upstream gradient, so this
// equals the gradient of the loss reweighted by the clip factors.
//
// Direct norm (the materialising alternative, "normal clipping" of Sec.
// "Training Configurations"): ||A_i^T G_i||_F^2 per example, from the same
// GEMM restricted to the example's T rows; each 256x256 output tile is
// squared and summed in registers at the example's last row. A work item of
// the direct-load kernel covers a run of consecutive examples of one tile.
// Optionally each example's tile is also written to a gradient store, from
// which store_sum_kernel forms the clipped sums as weighted sums of the
// stored tiles instead of a second GEMM. The direct form beats the Gram form
// when T + 1 exceeds about R * 2 d_in d_out / (d_in + d_out), R the measured
// ratio of the two kernels' throughputs (about 0.4 to 0.5).
//
// Kernels. dl_gemm_kernel (bf16: the clipped sum and the direct norm) stages
// rows in LDS and transposes on the way out of LDS; split_fixup_kernel
// finishes the tiles of its split tail. split_gemm_kernel (fp32) cuts its operands into
// three bf16 planes while staging them and multiplies on the bf16 matrix cores.
#include "common.hpp"
#include "kernels.hpp"

namespace dpg {

constexpr int GM_THREADS = 512;

enum { MODE_SUM = 0, MODE_NORM = 1 };

// Two bf16 held in one dword, each multiplied by s in fp32 and rounded back
// to bf16 (round to nearest even).
__device__ __forceinline__ uint32_t scale_bf16x2(uint32_t w, float s) {
  f32x2 v = {__uint_as_float(w << 16) * s, __uint_as_float(w & 0xFFFF0000u) * s};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Tile (mt, nt) of work item rel within a layer: the direction with fewer
// tiles varies fastest, so consecutive items (which run side by side on one
// XCD) share a tile of the operand that has more of them in L2.
__device__ __forceinline__ void tile_of(const GemmLayer& L, uint32_t rel, int& mt, int& nt) {
  if (L.tn <= L.tm) {
    mt = (int)(rel / (uint32_t)L.tn);
    nt = (int)(rel - (uint32_t)mt * L.tn);
  } else {
    nt = (int)(rel / (uint32_t)L.tm);
    mt = (int)(rel - (uint32_t)nt * L.tm);
  }
}

// The Gaussian mechanism, where a clipped sum fuses it (a.noise): value = (prior +
// sum + sigma_c * z) * inv_b, where z is the standard normal the noise generator
// assigns to the element's row-major index in the output tensor, i.e. the draw
// dp_add_noise would add to that element.
__device__ __forceinline__ float noise_at(const GemmArgs& a, uint32_t tid, uint64_t j) {
  float z[4];
  gauss4(j >> 2, a.seed, tid, a.step, z);
  const int q = (int)(j & 3);
  return q == 0 ? z[0] : q == 1 ? z[1] : q == 2 ? z[2] : z[3];
}

// The draws of 4 consecutive elements j0 .. j0+3 of a tensor: one Philox block
// where j0 is a multiple of 4, parts of two otherwise.
__device__ __forceinline__ void noise4_at(const GemmArgs& a, uint32_t tid, uint64_t j0,
                                          float (&z)[4]) {
  gauss4(j0 >> 2, a.seed, tid, a.step, z);
  const int sh = (int)(j0 & 3);
  if (sh != 0) {
    float y[4];
    gauss4((j0 >> 2) + 1, a.seed, tid, a.step, y);
    const float x[7] = {z[0], z[1], z[2], z[3], y[0], y[1], y[2]};
#pragma unroll
    for (int k = 0; k < 4; ++k) z[k] = sh == 1 ? x[k + 1] : sh == 2 ? x[k + 2] : x[k + 3];
  }
}

// Writes (or adds) one 256x256 tile of an output stored transposed, out[n][m]
// (row length M; sums from a gradient store only): each wave's 4x2 32x32
// blocks at rows m0 + wm*128 + i*32, columns n0 + wn*64 + j*32. In a 32x32
// block, lane l holds column l%32 and, for accumulator e, row (e/4)*8 +
// (l/32)*4 + e%4, so its 4 accumulators e = 4g..4g+3 are 4 consecutive elements of one
// output row starting at a multiple of 4, and one Philox block serves them when the row
// length is a multiple of 4. Stores bypass L2 residency (the output is
// written once) so that they do not evict operand rows.
__device__ __forceinline__ void store_tile_transposed(const GemmArgs& a, const GemmLayer& L,
                                                      int64_t m0, int64_t n0, int wm, int wn,
                                                      int lane, f32x16 (&acc)[4][2]) {
  float* out = L.out;
  const int64_t ldo = L.ldo;
  const bool accum = L.accumulate != 0;
  const bool noise = a.noise != 0;
  const uint32_t tid = L.tensor_id;
  const int mw = (int)m0 + wm * 128 + (lane >> 5) * 4;  // row of e = 0 in block i = 0
  const int nw = (int)n0 + wn * 64 + (lane & 31);         // column in block j = 0
  const bool full = m0 + GM_BM <= L.M && n0 + GM_BN <= L.N;
  const bool vec4 = full && (ldo & 3) == 0 && (((uintptr_t)out) & 15) == 0 &&
                    (!noise || (L.M & 3) == 0);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int n = nw + j * 32;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int m = mw + i * 32 + g * 8;
        float* p = out + (int64_t)n * ldo + m;
        if (vec4) {
          f32x4 v = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2],
                     acc[i][j][4 * g + 3]};
          if (accum) v += *(const f32x4*)p;
          if (noise) {
            float z[4];
            gauss4(((uint64_t)n * (uint64_t)L.M + (uint64_t)m) >> 2, a.seed, tid, a.step, z);
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = (v[r] + a.sigma_c * z[r]) * a.inv_b;
          }
          __builtin_nontemporal_store(v, (f32x4*)p);
        } else if (n < L.N) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (m + r < L.M) {
              float v = (accum ? p[r] : 0.f) + acc[i][j][4 * g + r];
              if (noise)
                v = (v + a.sigma_c * noise_at(a, tid, (uint64_t)n * (uint64_t)L.M + m + r)) *
                    a.inv_b;
              p[r] = v;
            }
        }
      }
    }
}

// Row-major store of one tile through LDS, for the non-transposed layout
// (the host orders every launch so that the kernel's rows are the output's
// rows). Each wave copies one 32x32 block at a time into its own 32 x 36
// float slice of LDS (MFMA layout in: lane l writes column l%32 of its 16
// rows), then reads it back as float4s of 4 consecutive columns: lane l takes
// row l/8 + 8*it, columns 4*(l%8) .. +3, so 8 lanes store 128 contiguous bytes
// of a row and every float4 is one Philox block of the output tensor (when
// the row length is a multiple of 4) for the fused Gaussian mechanism.
constexpr int EP_LD = 36;  // floats per LDS row of a block (16-byte aligned rows, fewer conflicts)

__device__ __forceinline__ void store_tile_rows(const GemmArgs& a, const GemmLayer& L, int64_t m0,
                                                int64_t n0, int wm, int wn, int lane,
                                                f32x16 (&acc)[4][2], float* slice) {
  float* out = L.out;
  const int64_t ldo = L.ldo;
  const bool accum = L.accumulate != 0;
  const bool noise = a.noise != 0;
  const uint32_t tid = L.tensor_id;
  // Rows of whole aligned float4s: a float4 lies in the matrix or outside it.
  const bool vec = (ldo & 3) == 0 && (((uintptr_t)out) & 15) == 0 && (L.N & 3) == 0;
  const int rw = (lane >> 5) * 4;  // row of e = 0 within a block
  const int cw = lane & 31;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int64_t mb = m0 + wm * 128 + i * 32, nb = n0 + wn * 64 + j * 32;
      if (mb >= L.M || nb >= L.N) continue;  // a block wholly past the matrix
#pragma unroll
      for (int e = 0; e < 16; ++e) slice[(rw + (e >> 2) * 8 + (e & 3)) * EP_LD + cw] = acc[i][j][e];
      // The block's 4 float4s per lane: prior values (when accumulating) are
      // requested first and the noise is drawn while they are in flight.
      const int c4 = 4 * (lane & 7);
      const int64_t n = nb + c4;
      f32x4 v[4], prior[4];
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int r = (lane >> 3) + 8 * it;
        v[it] = *(const f32x4*)(slice + r * EP_LD + c4);
      }
      if (vec) {
        const bool nin = n < L.N;
        if (accum) {
#pragma unroll
          for (int it = 0; it < 4; ++it) {
            const int64_t m = mb + (lane >> 3) + 8 * it;
            if (nin && m < L.M) prior[it] = *(const f32x4*)(out + m * ldo + n);
          }
        }
        if (noise) {
#pragma unroll
          for (int it = 0; it < 4; ++it) {
            const int64_t m = mb + (lane >> 3) + 8 * it;
            float z[4];
            gauss4(((uint64_t)m * (uint64_t)L.N + (uint64_t)n) >> 2, a.seed, tid, a.step, z);
#pragma unroll
            for (int q = 0; q < 4; ++q) v[it][q] += a.sigma_c * z[q];
          }
        }
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int64_t m = mb + (lane >> 3) + 8 * it;
          f32x4 x = v[it];
          if (accum) x += prior[it];
          if (noise) x *= a.inv_b;
          if (nin && m < L.M) __builtin_nontemporal_store(x, (f32x4*)(out + m * ldo + n));
        }
      } else {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int64_t m = mb + (lane >> 3) + 8 * it;
          if (m >= L.M) continue;
          float* p = out + m * ldo + n;
          float z[4];
          if (noise) noise4_at(a, tid, (uint64_t)m * (uint64_t)L.N + n, z);
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (n + q < L.N) {
              float x = (accum ? p[q] : 0.f) + v[it][q];
              if (noise) x = (x + a.sigma_c * z[q]) * a.inv_b;
              p[q] = x;
            }
        }
      }
    }
}

// A raw 256 x 256 partial tile, row-major, staged through LDS like
// store_tile_rows (8 lanes write 128 contiguous bytes of a row). Plain
// stores, unlike the output's: the fix-up launch right after reads the
// partials back, partly from the caches (its launch 1-2 % shorter at the
// tied head than with the streaming hint).
__device__ __forceinline__ void store_partial(float* dst, int wm, int wn, int lane,
                                              f32x16 (&acc)[4][2], float* slice) {
  const int rw = (lane >> 5) * 4, cw = lane & 31, c4 = 4 * (lane & 7);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
#pragma unroll
      for (int e = 0; e < 16; ++e) slice[(rw + (e >> 2) * 8 + (e & 3)) * EP_LD + cw] = acc[i][j][e];
      const int mb = wm * 128 + i * 32, nb = wn * 64 + j * 32;
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int r = (lane >> 3) + 8 * it;
        const f32x4 v = *(const f32x4*)(slice + r * EP_LD + c4);
        *(f32x4*)(dst + (mb + r) * GM_BN + nb + c4) = v;
      }
    }
}

// The split tail tiles: one thread per 4 consecutive elements of a row of
// one tile; the ksplit partials are added in order, then the prior, the
// noise and the division as in store_tile_rows.
__global__ __launch_bounds__(256) void split_fixup_kernel(GemmArgs args) {
  const GemmArgs& a = *(const GemmArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  (void)args;
  constexpr int QPT = GM_BM * GM_BN / 4;            // float4s per tile
  const uint32_t t = blockIdx.x / (QPT / 256);      // split tile
  const int q = (int)(blockIdx.x - t * (QPT / 256)) * 256 + (int)threadIdx.x;
  const uint32_t tile = a.n_full + t;
  const int ln = (int)(threadIdx.x & (WAVE - 1));
  const int l = wave_find(tile, ln < a.n_layers ? a.L[ln].tile_begin : 0u, a.n_layers);
  const GemmLayer& L = a.L[l];
  int mt, nt;
  tile_of(L, tile - L.tile_begin, mt, nt);
  const int r = q / (GM_BN / 4), c4 = (q - r * (GM_BN / 4)) * 4;
  const int64_t m = (int64_t)mt * GM_BM + r, n = (int64_t)nt * GM_BN + c4;
  if (m >= L.M || n >= L.N) return;
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  const float* src = a.part + (size_t)t * a.ksplit * (GM_BM * GM_BN) + r * GM_BN + c4;
  for (int k = 0; k < a.ksplit; ++k) v += *(const f32x4*)(src + (size_t)k * (GM_BM * GM_BN));
  float* p = L.out + m * L.ldo + n;
  const bool accum = L.accumulate != 0, noise = a.noise != 0;
  const bool vec = n + 4 <= L.N && (L.N & 3) == 0 && (L.ldo & 3) == 0 &&
                   (((uintptr_t)L.out) & 15) == 0;
  if (vec) {
    if (noise) {
      float z[4];
      gauss4(((uint64_t)m * (uint64_t)L.N + (uint64_t)n) >> 2, a.seed, L.tensor_id, a.step, z);
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] += a.sigma_c * z[k];
    }
    if (accum) v += *(const f32x4*)p;
    if (noise) v *= a.inv_b;
    *(f32x4*)p = v;
  } else {
    float z[4];
    if (noise) noise4_at(a, L.tensor_id, (uint64_t)m * (uint64_t)L.N + n, z);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (n + k < L.N) {
        float x = (accum ? p[k] : 0.f) + v[k];
        if (noise) x = (x + a.sigma_c * z[k]) * a.inv_b;
        p[k] = x;
      }
  }
}

// The fp32 clipped sum and direct norm: split_gemm_kernel. Every fp32 operand
// is cut exactly into three bf16 planes (split_f32 in common.hpp), and a
// product becomes six bf16 ones. Six 32x32x16 bf16 MFMAs take 192 cycles where
// the eight fp32 32x32x2 ones for the same 16 k take 512. The clipped sums of
// DistilGPT2 at B = 24, T = 128, V = 50257 unpadded (498 GFLOP): 5165 us on the
// fp32 MFMAs, 2310 us here.
//
// Errors against fp64, beside the fp32 MFMAs' (normal, uniform, GELU, softmax
// and shifted operands). Clipped sums, all six products on the running
// accumulator: 0.05 to 0.97 of theirs from K = 3 to 65536 (K = 1024: 1.8e-7 for
// 5.8e-7, of one sign 7.0e-8 for 4.2e-7); sums of fewer rows are left to the fp32 MFMAs.
// Direct norms: the matrix core cuts what lies below a fixed distance from the
// largest term of a sum, always towards zero, and a norm adds that up over the
// matrix where the additions' other errors average out: on the running accumulator 1.9
// times theirs (T = 1024, GELU outputs and softmax gradients). There a block's
// large products (x0 y0) of a stage and its five small ones are summed from
// zero, apart, and the VALU adds both to the accumulator: 0.8 to 1.1 of theirs
// (4.0e-8 for 4.3e-8), and 346 us where the running accumulator takes 304 and the fp32
// MFMAs 485 (four layers 768 -> 3072, B = 24, T = 128). Where the products of 16 tokens
// spread over many binary orders and K is short, both are larger (lognormal
// operands of sigma 2, K = 32: sums 1.2e-7 for 1.1e-7, norms 2.4e-7 for
// 1.4e-7; smaller again from K = 100 and 200 on).
//
// Tile 256x256, 16 k per stage, 8 waves of 128x64 as in the bf16 kernel.
// Waves 0-3 stage X, waves 4-7 Y: a wave takes 8 k rows and 128 columns, a
// lane two neighbouring columns (8 bytes per row, so rows need 4-byte
// alignment only), converts them after the load and writes a 16-byte chunk of 8
// consecutive k per column and plane. (A stage of 32 k in three planes would
// not fit LDS twice.) The conversion is about 6 VALU instructions per
// element, once per tile and stage; the X waves convert before their MFMAs and
// the Y waves after theirs, so that a SIMD's two waves (one of each) keep its
// matrix core busy meanwhile. LDS is double-buffered, one barrier per stage;
// the loads of stage s + 2 are in flight while stage s is multiplied.
constexpr int SP_PLANE = 2 * GM_BM;         // 16-byte chunks of one plane: two k halves
constexpr int SP_OP = 3 * SP_PLANE;         // of one operand
constexpr int SP_STAGE = 2 * SP_OP;         // of one stage
constexpr int SP_FEW = 2;                   // rows of a sum up to which the planes' error is larger
static_assert((GM_THREADS / WAVE) * 32 * EP_LD * 4 <= 2 * SP_STAGE * 16, "epilogue slices fit");

// Chunk of column m within a half plane: even columns first, odd ones behind
// them with their 8-chunk groups swapped in pairs, so that both the writes
// (a lane's even, then its odd column) and the reads of 32 consecutive columns
// touch all banks evenly.
__device__ __forceinline__ int sp_slot(int m) { return ((m >> 1) ^ ((m & 1) << 3)) + (m & 1) * (GM_BM / 2); }

template <int MODE>
__global__ __launch_bounds__(GM_THREADS) void split_gemm_kernel(GemmArgs args) {
  // Index the layer table in place in the kernel-argument segment.
  const GemmArgs& a = *(const GemmArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  (void)args;
  __shared__ __attribute__((aligned(1024))) u32x4 lds[2 * SP_STAGE];
  __shared__ float red[GM_THREADS / WAVE];

  // Whole tiles, then the K ranges of the split tail's (see dl_gemm_kernel).
  uint32_t item;
  int kc = -1;
  if (MODE == MODE_NORM || blockIdx.x < a.n_full) {
    item = xcd_remap(blockIdx.x, MODE == MODE_NORM ? gridDim.x : a.n_full);
  } else {
    const uint32_t j = blockIdx.x - a.n_full;
    item = a.n_full + j / (uint32_t)a.ksplit;
    kc = (int)(j - (j / (uint32_t)a.ksplit) * (uint32_t)a.ksplit);
  }
  const int ln = (int)(threadIdx.x & (WAVE - 1));
  const int l = wave_find(item, ln < a.n_layers ? a.L[ln].tile_begin : 0u, a.n_layers);
  const GemmLayer& L = a.L[l];
  uint32_t rel = item - L.tile_begin;
  int b = 0;
  if (MODE == MODE_NORM) {
    const uint32_t ntile = (uint32_t)L.tm * (uint32_t)L.tn;
    b = (int)(rel / ntile);
    rel -= (uint32_t)b * ntile;
  }
  int mt, nt;
  tile_of(L, rel, mt, nt);
  const int64_t m0 = (int64_t)mt * GM_BM;
  const int64_t n0 = (int64_t)nt * GM_BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w & 1, wn = w >> 1;

  // Staging: rows 8 kh .. 8 kh + 7 of a stage, columns 128 mh + 2 lane, + 1.
  // The descriptor spans the rows summed over (the batch, or one example);
  // rows past them are pointed at its end and read as zeros. Columns past M/N
  // read padding or the next row and only reach outputs that are left out.
  const bool load_x = w < 4;
  const int kh = (w & 3) >> 1, mh = w & 1;
  const int64_t ld = load_x ? L.ldx : L.ldy;
  const uint32_t ld_bytes = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(ld * 4));
  const int rows = MODE == MODE_NORM ? a.T : a.B * a.T;
  const char* base = (const char*)(load_x ? L.X : L.Y) + (MODE == MODE_NORM ? (int64_t)b * a.T * ld * 4 : 0);
  const rsrc_t rsrc = make_rsrc(base, (uint64_t)rows * ld_bytes);
  const uint32_t voff = (uint32_t)(((load_x ? m0 : n0) + mh * 128 + 2 * lane) * 4);
  const int slot0 = mh * 64 + lane;
  u32x4* const wr = lds + (load_x ? 0 : SP_OP) + kh * GM_BM;
  int s0 = 0, nS = (rows + SP_BK - 1) / SP_BK;  // stages s0 .. s0 + nS - 1
  if (MODE == MODE_SUM && kc >= 0) {
    const int per = (nS + a.ksplit - 1) / a.ksplit;
    s0 = kc * per;
    nS = s0 + per < nS ? per : (s0 < nS ? nS - s0 : 0);
  }

  // Clip factors: row j of this wave's 8 rows of the next stage to load lies
  // in example e_ld + (r_ld + j) / T; lane j fetches its factor.
  // x / T = hi32(x * rcpT) for x < T + 8 (T <= 65536).
  const int nT = __builtin_amdgcn_readfirstlane(a.T), nB = __builtin_amdgcn_readfirstlane(a.B);
  const uint32_t rcpT = 0xFFFFFFFFu / (uint32_t)nT + 1u;
  auto over_T = [&](int x) { return nT == 1 ? x : (int)__umulhi((uint32_t)x, rcpT); };
  int row_ld = s0 * SP_BK + kh * 8;   // this wave's first row of the next stage to load
  int e_ld = row_ld / nT, r_ld = row_ld - e_ld * nT;
  float cv = 1.f;   // factor of row lane % 8 of the loaded stage

  u32x2 raw[8];
  auto load = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      raw[j] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(
                   rsrc, voff, (uint32_t)min(row_ld + j, rows) * ld_bytes, 0));
    row_ld += SP_BK;
    if constexpr (MODE == MODE_SUM) {
      cv = a.c[min(e_ld + over_T(r_ld + (lane & 7)), nB - 1)];
      r_ld += SP_BK;
      const int de = __builtin_amdgcn_readfirstlane(r_ld < nT ? 0 : r_ld / nT);
      e_ld += de;
      r_ld -= de * nT;
    }
  };
  // The loaded stage, scaled and cut, into LDS buffer `buf`.
  auto convert = [&](int buf) __attribute__((always_inline)) {
    u32x4* const dst = wr + buf * SP_STAGE;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      u32x4 p0, p1, p2;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float x[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int j = 2 * k + h;
          x[h] = __uint_as_float(raw[j][q]);
          if constexpr (MODE == MODE_SUM) {
            // An example with c = 0 (a non-finite norm) is left out of the sum:
            // its rows are zeroed in both operands (0 * inf would be NaN).
            const float c = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(cv), j));
            x[h] *= load_x ? c : 1.f;
            x[h] = __uint_as_float(__float_as_uint(x[h]) & (c == 0.f ? 0u : 0xFFFFFFFFu));
          }
        }
        const Split2 sp = split_f32(x[0], x[1]);
        p0[k] = sp.p[0];
        p1[k] = sp.p[1];
        p2[k] = sp.p[2];
      }
      const int at = q == 0 ? slot0 : GM_BM / 2 + (slot0 ^ 8);
      dst[at] = p0;
      dst[at + SP_PLANE] = p1;
      dst[at + 2 * SP_PLANE] = p2;
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  f32x16 acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x16{};
  const int r32 = lane & 31, half = lane >> 5;
  const u32x4* const rd_x = lds + half * GM_BM + wm * 64 + sp_slot(r32);
  const u32x4* const rd_y = lds + SP_OP + half * GM_BM + wn * 32 + sp_slot(r32);
  auto compute = [&](int buf) __attribute__((always_inline)) {
    // The next block row's fragments are read while this one's are multiplied, and
    // (direct norm) a block's large products are added while the next block's are
    // multiplied. Fences bound how far the reads move up (all at once, they spill).
    const u32x4* const bx = rd_x + buf * SP_STAGE;
    const u32x4* const by = rd_y + buf * SP_STAGE;
    u32x4 y[2][3], x[2][3];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      x[0][p] = bx[p * SP_PLANE];
      y[0][p] = by[p * SP_PLANE];
      y[1][p] = by[p * SP_PLANE + 16];
    }
    f32x16 big;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const u32x4(&xi)[3] = x[i & 1];
      if (i < 3) {
#pragma unroll
        for (int p = 0; p < 3; ++p) x[(i + 1) & 1][p] = bx[p * SP_PLANE + (i + 1) * 16];
      }
      if constexpr (MODE == MODE_SUM) {
#pragma unroll
        for (int t = 0; t < SPLIT_TERMS; ++t)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = mfma32_bf16(xi[split_a(t)], y[j][split_b(t)], acc[i][j]);
        __builtin_amdgcn_sched_barrier(0);
      } else {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const f32x16 small = split_small(xi, y[j], f32x16{});
          if (j == 1) split_add(acc[i][0], big);
          else if (i > 0) split_add(acc[i - 1][1], big);
          big = mfma32_bf16(xi[0], y[j][0], f32x16{});
          split_add(acc[i][j], small);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    if constexpr (MODE == MODE_NORM) split_add(acc[3][1], big);
  };

  load();
  convert(0);
  load();
  __syncthreads();
  for (int s = 0; s < nS; ++s) {
    const int buf = s & 1;
    const bool more = s + 1 < nS;
    if (load_x && more) {
      convert(buf ^ 1);
      load();
    }
    __builtin_amdgcn_sched_barrier(0);
    compute(buf);
    __builtin_amdgcn_sched_barrier(0);
    if (!load_x && more) {
      convert(buf ^ 1);
      load();
    }
    __syncthreads();
  }

  // The wave's part of the tile on the fp32 matrix cores, from memory. An
  // infinity's planes hold NaN, and where a product overflows, plane products
  // of both signs may: a result that is not finite is computed again with this,
  // so that it is the infinity or NaN that fp32 products give. So is a sum of values
  // so small that their planes may have lost bits (all results below 2^-60).
  auto again = [&]() __attribute__((always_inline)) {
    int ln = lane;
    asm volatile("" : "+v"(ln));  // no address of this loop is kept across the main one
    const int k_end = min((s0 + nS) * SP_BK, rows);
    const int64_t row0 = MODE == MODE_NORM ? (int64_t)b * a.T : 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = f32x16{};
#pragma unroll 1
    for (int k0 = s0 * SP_BK; k0 < k_end; k0 += 2) {
      const int k = k0 + (ln >> 5);
      const bool kin = k < k_end;
      const float c = MODE == MODE_SUM && kin ? a.c[k / nT] : 1.f;
      const bool use = kin && c != 0.f;
      float xf[4], yf[2];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t m = m0 + wm * 128 + i * 32 + (ln & 31);
        xf[i] = use && m < L.M ? ((const float*)L.X)[(row0 + k) * L.ldx + m] * c : 0.f;
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int64_t n = n0 + wn * 64 + j * 32 + (ln & 31);
        yf[j] = use && n < L.N ? ((const float*)L.Y)[(row0 + k) * L.ldy + n] : 0.f;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma32_f32(xf[i], yf[j], acc[i][j]);
    }
  };

  if constexpr (MODE == MODE_SUM) {
    // (Blocks that straddle the matrix's last row count whole: what lies past it is
    // finite, or costs the second pass.)
    float size = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (m0 + wm * 128 + i * 32 >= L.M) break;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        float t = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) t += fabsf(acc[i][j][e]);
        if (n0 + wn * 64 + j * 32 + r32 < L.N) size += t;
      }
    }
    if (rows <= SP_FEW || __any(!(size <= FLT_MAX)) ||
        (!__any(size >= 0x1p-60f) && __any(size > 0.f)))
      again();
    float* const slice = (float*)lds + w * 32 * EP_LD;
    // The host orders every launch so that the kernel's rows are the output's.
    if (kc < 0)
      store_tile_rows(a, L, m0, n0, wm, wn, lane, acc, slice);
    else
      store_partial(a.part + ((size_t)(item - a.n_full) * a.ksplit + kc) * (GM_BM * GM_BN), wm, wn,
                    lane, acc, slice);
  } else {
    float part = 0.f;
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass) {
      // Rows and columns left in the tile past this lane's first element. Opaque, so
      // that the elements' masks are not kept from one pass to the next.
      int lim_m = (int)(L.M - m0) - (wm * 128 + (lane >> 5) * 4);
      int lim_n = (int)(L.N - n0) - (wn * 64 + (lane & 31));
      asm volatile("" : "+v"(lim_m), "+v"(lim_n));
      part = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const bool nin = j * 32 < lim_n;
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const float v = acc[i][j][e];
            part += (nin && i * 32 + (e >> 2) * 8 + (e & 3) < lim_m) ? v * v : 0.f;
          }
        }
      if (pass == 1 || !__any(!(part <= FLT_MAX))) break;
      again();
    }
    part = wave_sum(part);
    if (lane == 0) red[w] = part;
    __syncthreads();
    if (tid == 0) {
      float t = 0.f;
#pragma unroll
      for (int q = 0; q < GM_THREADS / WAVE; ++q) t += red[q];
      a.ws[(int64_t)b * a.slots + L.slot_begin + rel] = t;
    }
  }
}

// ---------------------------------------------------------------------------
// Direct-load kernel for the bf16 clipped sum and direct norm. In its PLAIN, BIG,
// RAGGED and SCALED forms (16-byte aligned rows; see GemmForm) nothing is staged
// through VGPRs; the STAGED and ROWS forms load through registers further down.
//
// Global rows go straight into LDS through buffer loads that write LDS
// (each lane's 16 bytes land at M0 + 16*lane), so LDS keeps the token-major
// layout: stage row r = token, 256 features = 32 chunks of 16 bytes, chunk c
// stored at physical chunk c ^ dl_sw(r). The MFMA fragments (8 consecutive k
// of one column per lane) come out of LDS through the transposing read
// ds_read_b64_tr_b16, which gathers 4 rows x 4 columns per 16-lane group:
// two such reads give one 32x32x16 operand. With the swizzle the 16 chunks a
// half-wave touches fall in 16 distinct bank groups.
//
// Ring of 4 stages of 32 k (32 KB each: X then Y), worked in ping-pong by
// two groups of four waves, one wave of each group per SIMD: while one group
// issues a stage's 16 MFMAs (at raised wave priority), the other reads the
// next stage's fragments out of LDS, issues its share of a later stage's
// loads and, at an example boundary, rescales its accumulators; a barrier
// swaps the roles. So each SIMD always has one wave feeding its matrix core
// and one wave doing everything else, and the VALU work of the rescale runs
// beside the other group's MFMAs. Group 0 (waves 0-3, the X loaders)
// computes stage s in phase 2s and reads stage s+1 in phase 2s+1; group 1
// (waves 4-7, the Y loaders) reads stage s in phase 2s and computes it in
// phase 2s+1. Stage s's slot is free once phase 2s ends: group 0 refills it
// with stage s+4 in phase 2s+1, and group 1 refills the slot of stage s-1
// with stage s+3 in phase 2s. Every wave waits for its own loads of stage
// s+1 at the end of phase 2s, so the barrier that ends the phase certifies
// that stage s+1 has landed. Every phase issues the same 4 loads per wave
// (stages past the end read zeros through the range check into a slot that
// is never read again), so the wait counts are constants.
//
// The loads are issued from inline assembly: the compiler would otherwise
// treat every later LDS read as possibly aliasing an LDS-writing load and
// drain all of them (vmcnt(0)) before it, serialising the ring. Its wait
// bookkeeping stays sound: untracked loads only make its own waits stricter.
// Clip factors are staged in LDS so that the loop issues no other vector
// memory instruction; each is read one example ahead, so that a rescale never
// waits behind the fragment reads. Scaling is on the fp32 accumulators:
// rescaled by c_prev / c_next at example boundaries and by the last factor at the
// end, examples with c = 0 skipped (so that inf or NaN in their rows adds
// nothing). The SCALED form multiplies a wave's Y fragments by their rows' factors
// instead, in the memory phase (4 fragments of 12: 80 VALU instructions beside
// the other group's 16 MFMAs): sums of 3072 tokens in examples of 21 (twelve layers 768 ->
// 3072) 217 us, 401 with the rows scaled on their way through registers, loaded
// one stage ahead only. In the direct norm the example boundary instead squares and sums
// each wave's part of the tile (and writes the tile to the gradient store,
// if there is one), then clears the accumulators for the next example.
constexpr int DL_BK = DL_SUM_BK;            // k rows per stage
constexpr int DL_NS = 4;                    // stages in the ring
constexpr int DL_ROWB = GM_BM * 2;          // bytes per LDS row (256 bf16)
constexpr int DL_OPB = DL_BK * DL_ROWB;     // one operand's stage: 16 KB
constexpr int DL_STB = 2 * DL_OPB;          // one stage: X then Y
constexpr int DL_MAXB = DL_SUM_MAXB;        // clip factors held in LDS
constexpr int DL_LOADS = 4;                 // loads per wave per stage
static_assert(GM_BM == GM_BN, "square tiles");
static_assert(DL_STB == (GM_THREADS / WAVE) * DL_LOADS * 1024, "one KB per load");
static_assert(NG_MAX * (GM_THREADS / WAVE) <= DL_MAXB, "direct norm: a part per example and wave fits the factor table");
static_assert((GM_THREADS / WAVE) * 32 * EP_LD * 4 <= DL_NS * DL_STB, "epilogue slices fit the ring");

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(3))) char lds_char_t;
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4_t;

// Physical chunk of chunk c in stage row r is c ^ dl_sw(r). The 4 rows read
// together are r = 4a..4a+3; dl_sw maps them to 0, 6, 12, 10, whose bits 1-2
// and bits 2-3 are both all distinct, so the reads are conflict-free whether
// the LDS serves 16 or 32 lanes of a 64-bit read per cycle.
__device__ __forceinline__ int dl_sw(int r) {
  const int q = r & 3;
  return (q << 2) ^ (q << 1);
}

__device__ __forceinline__ u32x2 lds_read_tr(const lds_char_t* p) {
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_t*)p));
}

// 32x32x16 operand: lane l gets column l%32 at k rows 8*(l/32) .. +7 of the
// 16-row half stage at `off` (two reads of 4 rows each).
__device__ __forceinline__ u32x4 dl_frag(const lds_char_t* base, uint32_t off) {
  const u32x2 lo = lds_read_tr(base + off), hi = lds_read_tr(base + off + 4 * DL_ROWB);
  return u32x4{lo[0], lo[1], hi[0], hi[1]};
}

// s_waitcnt vmcnt(N) leaving the other counters alone (gfx9 encoding).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// MODE_SUM: the clipped sum over all K = B*T rows. MODE_NORM (the direct
// norm): K restricted to example b's T rows, no factors, and the tile's
// in-range elements squared and summed in registers.
// Gradient store layout (GRAD_STORE): within a tile's 65536 floats, wave w's
// accumulator block (i, j), floats 4q .. 4q+3 of lane l, sit at
// ((w * 8 + i * 2 + j) * 4 + q) * 256 + 4 l: every store and load moves one
// contiguous KB per wave.
__device__ __forceinline__ size_t store_lane_offset(int w, int lane) {
  return (size_t)w * 8 * 4 * 256 + (size_t)lane * 4;
}
__device__ __forceinline__ size_t store_chunk(int i, int j, int q) {
  return (size_t)((i * 2 + j) * 4 + q) * 256;
}

// FORM: how the launch's stages are cut and loaded (see GemmForm).
template <int MODE, int FORM>
__global__ __launch_bounds__(GM_THREADS) void dl_gemm_kernel(GemmArgs args) {
  constexpr bool BIG = FORM == FORM_BIG;
  constexpr bool STAGED = FORM == FORM_STAGED || FORM == FORM_ROWS;  // through registers
  constexpr bool SCALED = FORM == FORM_SCALED;
  constexpr bool ROWS = FORM == FORM_ROWS || SCALED;                 // stages over all rows
  // Stages whose rows follow one another through the batch, loaded straight into LDS.
  constexpr bool WHOLE = FORM == FORM_PLAIN || FORM == FORM_BIG || SCALED;
  const GemmArgs& a = *(const GemmArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  (void)args;
  __shared__ __attribute__((aligned(1024))) char ring_raw[DL_NS * DL_STB];
  __shared__ float cs[DL_MAXB];
  // SCALED: each wave's row factors of the stages with even and odd index.
  __shared__ __attribute__((aligned(16))) float row_c[SCALED ? GM_THREADS / WAVE : 1][2][DL_BK];
  lds_char_t* ring = (lds_char_t*)(lds_void_t*)ring_raw;

  // Whole tiles come first (spread over the XCDs); the K ranges of the split
  // tail tiles are dispatched last, in round-robin over the XCDs.
  uint32_t item;
  int kc = -1;  // K range of a split tile, or -1
  if (MODE == MODE_NORM || blockIdx.x < a.n_full) {
    item = xcd_remap(blockIdx.x, MODE == MODE_NORM ? gridDim.x : a.n_full);
  } else {
    const uint32_t j = blockIdx.x - a.n_full;
    item = a.n_full + j / (uint32_t)a.ksplit;
    kc = (int)(j - (j / (uint32_t)a.ksplit) * (uint32_t)a.ksplit);
  }
  const int ln = (int)(threadIdx.x & (WAVE - 1));
  const int l = wave_find(item, ln < a.n_layers ? a.L[ln].tile_begin : 0u, a.n_layers);
  const GemmLayer& L = a.L[l];
  uint32_t rel = item - L.tile_begin;
  const int64_t K = (int64_t)a.B * a.T;
  // Stages: DL_BK rows each, cut per example (the last one of an example may
  // be short) or, with ROWS, over all K rows. This item covers stages gs0 ..
  // gs0 + nS - 1 of the launch.
  const int spe = (a.T + DL_BK - 1) / DL_BK;  // stages per example
  int b = 0;
  int gs0 = 0, nS = ROWS ? (int)((K + DL_BK - 1) / DL_BK) : a.B * spe;
  if (MODE == MODE_SUM && kc >= 0) {
    const int per = (nS + a.ksplit - 1) / a.ksplit;  // stages per range
    gs0 = kc * per;
    nS = gs0 + per < nS ? per : (gs0 < nS ? nS - gs0 : 0);
  }
  int n_ex = 1;  // direct norm: examples b .. b + n_ex - 1 of this item
  if constexpr (MODE == MODE_NORM) {
    const uint32_t ntile = (uint32_t)L.tm * (uint32_t)L.tn;
    const int grp = (int)(rel / ntile);
    rel -= (uint32_t)grp * ntile;
    b = grp * a.eg;
    n_ex = a.B - b < a.eg ? a.B - b : a.eg;
    gs0 = b * spe;
    nS = n_ex * spe;
  }
  // First row of the item, and the end of the example it lies in.
  const int e0 = ROWS ? 0 : gs0 / spe;
  const int64_t k_begin = ROWS ? (int64_t)gs0 * DL_BK
                               : (int64_t)e0 * a.T + (int64_t)(gs0 - e0 * spe) * DL_BK;
  int mt, nt;
  tile_of(L, rel, mt, nt);
  const int64_t m0 = (int64_t)mt * GM_BM;
  const int64_t n0 = (int64_t)nt * GM_BN;

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w & 1, wn = w >> 1;

  // Load role: waves 0-3 fill X rows 8w..8w+7 of every stage, waves 4-7 the
  // same rows of Y. Load t writes rows 2t, 2t+1 of that block: lane l takes
  // row l/32 and physical chunk l%32, i.e. logical chunk (l%32) ^ dl_sw(row).
  const bool load_x = w < 4;
  const int wq = w & 3;
  const uint32_t ld_bytes = (uint32_t)((load_x ? L.ldx : L.ldy) * 2);
  const int64_t col0 = load_x ? m0 : n0;
  uint32_t lvo[2];  // lane offsets of loads with t even / odd
#pragma unroll
  for (int par = 0; par < 2; ++par) {
    const int c = (lane & 31) ^ dl_sw(2 * par + (lane >> 5));
    lvo[par] = (uint32_t)((lane >> 5) * ld_bytes + (col0 + 8 * c) * 2);
  }
  const uint32_t lds_role = (uint32_t)(load_x ? 0 : DL_OPB) + (uint32_t)wq * 8 * DL_ROWB;
  const uint64_t gbase = (uint64_t)(load_x ? (const void*)L.X : (const void*)L.Y);
  const uint64_t nrec64 = (uint64_t)K * ld_bytes;
  const uint32_t nrec = nrec64 > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)nrec64;
  const u32x4 desc = {(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)gbase),
                      (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(gbase >> 32)),
                      (uint32_t)__builtin_amdgcn_readfirstlane((int)nrec), (uint32_t)RSRC_WORD3};
  const uint32_t ring_base = (uint32_t)(uintptr_t)ring;
  // Load t (of DL_LOADS) of this wave's share of stage s.
  // An operand of 4 GiB or more does not fit the 32-bit offsets: its
  // descriptor's base moves to each stage's first row instead (the records
  // left from there, none past the last stage). A separate instance, so that
  // launches without such an operand keep the plain loop.
  const bool big = BIG && nrec64 > 0xFFFFFFFFull;
  // Examples of any length: the stages to load are visited in order, so the
  // first row of the next one and the end of its example are carried along. The descriptor starts at that
  // row and ends with the example: rows past it read as zeros, and no offset
  // grows with the operand.
  struct Cursor {
    uint64_t base;   // address of this wave's first row of the stage
    int left;        // rows left from the stage's first row to the example's end
  };
  auto uniform64 = [](uint64_t x) {  // keeps wave-uniform arithmetic on the scalar unit
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
  };
  const int nT = __builtin_amdgcn_readfirstlane(a.T);
  const uint32_t ld_u = (uint32_t)__builtin_amdgcn_readfirstlane((int)ld_bytes);
  Cursor ld_at{uniform64(gbase + (uint64_t)(k_begin + wq * 8) * ld_bytes),
               __builtin_amdgcn_readfirstlane(ROWS ? (int)min(K - k_begin, (int64_t)INT32_MAX)
                                                   : (int)((int64_t)(e0 + 1) * a.T - k_begin))};
  auto next_stage = [&](Cursor& q) {
    const int step = q.left < DL_BK ? q.left : DL_BK;
    q.base += (uint64_t)ld_u * (uint32_t)step;
    q.left -= step;
    if (!ROWS && q.left == 0) q.left = nT;
  };
  auto issue = [&](int s, int t) {
    if constexpr (!WHOLE) {
      const uint32_t dst = ring_base + (uint32_t)((s % DL_NS) * DL_STB) + lds_role;
      const int rows = ld_at.left - wq * 8;  // from this wave's first row on
      const uint32_t nr = s < nS && rows > 0 ? (uint32_t)rows * ld_u : 0u;
      const u32x4 d = {(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)ld_at.base),
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(ld_at.base >> 32)),
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)nr), (uint32_t)RSRC_WORD3};
      const uint32_t m0v = (uint32_t)__builtin_amdgcn_readfirstlane((int)(dst + t * 1024));
      const uint32_t so = (uint32_t)__builtin_amdgcn_readfirstlane((int)(2 * t * ld_u));
      asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen sc1 lds"
                   :: "s"(m0v), "v"(lvo[t & 1]), "s"(d), "s"(so));
      if (t == DL_LOADS - 1) next_stage(ld_at);
      return;
    }
    const uint32_t dst = ring_base + (uint32_t)((s % DL_NS) * DL_STB) + lds_role;
    const int64_t row0 = k_begin + (int64_t)s * DL_BK + wq * 8;
    uint32_t sbase;
    u32x4 d = desc;
    if (big) {
      const uint64_t base = gbase + (uint64_t)row0 * ld_bytes;
      const uint64_t rem = s < nS ? (uint64_t)(K - row0) * ld_bytes : 0ull;
      const uint32_t nr = rem > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)rem;
      d = u32x4{(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)base),
                (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(base >> 32)),
                (uint32_t)__builtin_amdgcn_readfirstlane((int)nr), (uint32_t)RSRC_WORD3};
      sbase = 0;
    } else {
      sbase = s < nS ? (uint32_t)(row0 * ld_bytes) : nrec;
    }
    {
      const uint32_t m0v = (uint32_t)__builtin_amdgcn_readfirstlane((int)(dst + t * 1024));
      const uint32_t so = (uint32_t)__builtin_amdgcn_readfirstlane((int)(sbase + 2 * t * ld_bytes));
      // M0 (the LDS destination) is a reserved register that the compiler
      // sets right before each of its own users; this kernel has none. The
      // loads are device-scope (sc1), which measured 0-3 % faster; unlike the
      // Gram's streams they keep the temporal hint, as neighbouring tiles
      // share operand panels through L2 (nt measured slower).
      asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen sc1 lds"
                   :: "s"(m0v), "v"(lvo[t & 1]), "s"(d), "s"(so));
    }
  };

  // Transposing-read lane offsets of this wave's 4 X blocks and 2 Y blocks:
  // within each 16-lane group, lane j addresses row j/4 and columns
  // 4*(j%4) .. +3 of the group's 16 columns.
  const int g = lane >> 4, jl = lane & 15;
  const int rrow = 8 * (g >> 1) + (jl >> 2);
  const int F = dl_sw(jl >> 2);
  uint32_t ox[4], oy[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = wm * 128 + i * 32 + 16 * (g & 1) + 4 * (jl & 3);
    ox[i] = (uint32_t)(rrow * DL_ROWB + (((m >> 3) ^ F) << 4) + ((m & 7) << 1));
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int n = wn * 64 + j * 32 + 16 * (g & 1) + 4 * (jl & 3);
    oy[j] = (uint32_t)(DL_OPB + rrow * DL_ROWB + (((n >> 3) ^ F) << 4) + ((n & 7) << 1));
  }

  f32x16 acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  if constexpr (MODE == MODE_SUM)
    for (int i = tid; i < min(a.B, DL_MAXB); i += GM_THREADS) cs[i] = a.c[i];
  // A batch of more examples than the table holds reads the factors of the
  // others from memory.
  auto factor = [&](int e) {
    if ((WHOLE && !SCALED) || e < DL_MAXB) return cs[e];
    float x = a.c[e];
    // Opaque: merged with the other load it would be one load through a
    // generic pointer, whose wait drains the ring.
    asm volatile("" : "+v"(x));
    return x;
  };
  // Held in a register: a kernel-argument read inside the loop would be a
  // scalar load whose wait (lgkmcnt) also waits for every LDS read in flight.
  const int nB = __builtin_amdgcn_readfirstlane(a.B);
  // Stage indices below are local to this item, whose stages may start inside
  // example e0 (a split range): the first stage is treated as a boundary,
  // where nothing is yet accumulated.
  float c_acc = 0.f;            // factor of what is accumulated; 0: nothing yet
  float c_nx = 0.f;             // factor of the example that starts at stage s_nx
  bool skip = false;
  int s_nx = 0, e_nx = e0;      // next example boundary (a local stage) and its example
  // Direct norm: the squared Frobenius norm of this wave's part of the tile
  // for local example le goes to red[le * 8 + w] (the factor table is unused
  // in this mode); the workgroup adds the 8 waves' parts at the end. The
  // columns past M or N were loaded from beyond the rows' valid width and
  // only reach out-of-range elements, which the sum leaves out.
  float* red = cs;
  const bool full = m0 + GM_BM <= L.M && n0 + GM_BN <= L.N;
  int le = 0;
  if constexpr (MODE == MODE_NORM) s_nx = spe;
  auto fin = [&]() __attribute__((always_inline)) {
    float part = 0.f;
    if (full) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) part = fmaf(acc[i][j][e], acc[i][j][e], part);
    } else {
      // Rows and columns left in the tile past this lane's first element.
      // Opaque here, so that the compiler does not keep the masks of every
      // accumulator live across the main loop.
      int lim_m = (int)(L.M - m0) - (wm * 128 + (lane >> 5) * 4);
      int lim_n = (int)(L.N - n0) - (wn * 64 + (lane & 31));
      asm volatile("" : "+v"(lim_m), "+v"(lim_n));
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const bool nin = j * 32 < lim_n;
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const float v = acc[i][j][e];
            part += (nin && i * 32 + (e >> 2) * 8 + (e & 3) < lim_m) ? v * v : 0.f;
          }
        }
    }
    part = wave_sum(part);
    if (lane == 0) red[le * (GM_THREADS / WAVE) + w] = part;
    if (a.store) {
      // the example's tile, for a later clipped sum from the store
      float* dst = a.store + ((((size_t)L.slot_begin + rel) * (size_t)a.B + (size_t)(b + le))
                              << 16) + store_lane_offset(w, lane);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2],
                             acc[i][j][4 * q + 3]};
            __builtin_nontemporal_store(v, (f32x4*)(dst + store_chunk(i, j, q)));
          }
    }
    ++le;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = f32x16{};
  };
  // Called once per stage, in increasing order, in the memory phase before
  // that stage's MFMAs. Clipped sum: at an example boundary, rescales the
  // accumulators by c_prev / c_next and fetches the factor of the example
  // after. Direct norm: at an example boundary, reduces the finished
  // example's part of the tile and clears the accumulators.
  auto enter = [&](int s) __attribute__((always_inline)) {
    if (MODE == MODE_NORM && s == s_nx) {
      fin();
      s_nx += spe;
    }
    if (MODE == MODE_SUM && !ROWS && s == s_nx) {
      const float ce = c_nx;
      ++e_nx;
      s_nx = e_nx * spe - gs0;
      if (e_nx < nB) c_nx = factor(e_nx);
      skip = !(ce != 0.f);
      if (!skip) {
        if (c_acc != 0.f) {
          const float f = c_acc / ce;
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] *= f;
        }
        c_acc = ce;
      }
    }
  };
  // rd: both halves (k 0..15 and 16..31) of stage s, 4 X and 2 Y fragments
  // each. rd_issue: the same reads in four groups of three, each group after
  // one of this wave's loads of stage sl. Spreading the loads over the phase
  // keeps the L1's queue of pending requests from filling in one burst (2-4 %
  // faster than issuing all loads first or all reads first).
  auto frag = [&](const lds_char_t* base, int idx) {
    const int h = idx / 6, k = idx % 6;
    return dl_frag(base, (k < 4 ? ox[k] : oy[k - 4]) + h * 16 * DL_ROWB);
  };
  auto rd = [&](int s, u32x4 (&f)[12]) {
    const lds_char_t* base = ring + (s % DL_NS) * DL_STB;
#pragma unroll
    for (int idx = 0; idx < 12; ++idx) f[idx] = frag(base, idx);
  };
  auto rd_issue = [&](int s, int sl, u32x4 (&f)[12]) {
    const lds_char_t* base = ring + (s % DL_NS) * DL_STB;
#pragma unroll
    for (int q = 0; q < DL_LOADS; ++q) {
      issue(sl, q);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < 3; ++r) f[3 * q + r] = frag(base, 3 * q + r);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto compute = [&](const u32x4 (&f)[12]) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
    if (!skip) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = mfma32_bf16(f[6 * h + i], f[6 * h + 4 + j], acc[i][j]);
    }
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // SCALED. A lane looks up the factor of row lane % 32 of a stage, one stage before
  // its wave reads that stage's fragments, and leaves it in the wave's own slot of LDS.
  // The example of row r_sc + x is e_sc + x / T, and x / T = hi32(x * rcpT)
  // for the x < T + DL_BK here (T <= 2 DL_BK).
  const uint32_t rcp_sc = SCALED ? 0xFFFFFFFFu / (uint32_t)nT + 1u : 0u;
  auto over_T = [&](int x) { return nT == 1 ? x : (int)__umulhi((uint32_t)x, rcp_sc); };
  int e_sc = SCALED ? (int)(k_begin / nT) : 0;
  int r_sc = SCALED ? (int)(k_begin - (int64_t)e_sc * nT) : 0;
  bool left_out[2] = {false, false};  // some row of the stage has factor 0
  auto look_up = [&](int s) __attribute__((always_inline)) {
    const float c = factor(min(e_sc + over_T(r_sc + (lane & 31)), nB - 1));
    row_c[SCALED ? w : 0][s & 1][lane & 31] = c;
    left_out[s & 1] = __any(c == 0.f);
    const int x = r_sc + DL_BK, de = over_T(x);
    e_sc += de;
    r_sc = x - de * nT;
  };
  // Multiplies stage s's Y fragments by their rows' factors. Where an example is left
  // out, its rows are zeroed in both operands (0 * inf would be NaN).
  auto scale = [&](int s, u32x4 (&f)[12]) __attribute__((always_inline)) {
    const float* rc = row_c[SCALED ? w : 0][s & 1] + 8 * (lane >> 5);
    f32x4 c[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int q = 0; q < 2; ++q) c[h][q] = *(const f32x4*)(rc + 16 * h + 4 * q);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const f32x4& ck = c[h][k >> 1];
          const uint32_t v = f[6 * h + 4 + j][k];
          const f32x2 x = {__uint_as_float(v << 16) * ck[2 * (k & 1)],
                           __uint_as_float(v & 0xFFFF0000u) * ck[2 * (k & 1) + 1]};
          f[6 * h + 4 + j][k] = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
        }
    if (left_out[s & 1]) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const f32x4& ck = c[h][k >> 1];
          const uint32_t keep = (ck[2 * (k & 1)] == 0.f ? 0u : 0xFFFFu) |
                                (ck[2 * (k & 1) + 1] == 0.f ? 0u : 0xFFFF0000u);
#pragma unroll
          for (int q = 0; q < 6; ++q) f[6 * h + q][k] &= keep;
        }
    }
  };
  // Phase boundary; nothing is scheduled across it.
  auto bar = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
  };

  u32x4 fr[12];
  if constexpr (STAGED) {
    // Register-staged loads (rows of any alignment, waves 0-3 X, waves 4-7
    // Y as above): in the memory phase of stage s both groups write stage s + 2
    // to LDS (the slot of stage s - 2) and load stage s + 3 into the same
    // registers, one stage's time before their write. (Two sets, loaded two
    // stages ahead, do not fit the register file.) Lane l takes rows 2t + l/32, logical chunk l%32, so a
    // row's 512 bytes are read in order.
    const int64_t ncol = load_x ? L.M : L.N;
    const int ncl = (int)min(ncol - (col0 + 8 * (lane & 31)), (int64_t)8);  // of this lane's 8
    const uint32_t lo0 = (uint32_t)((lane >> 5) * ld_bytes + (lane & 31) * 16);
    typedef u32x4 Set[DL_LOADS];
    // Address of the tile's first column in this wave's first row of a stage.
    // Chunks past the matrix's columns read the row's padding or the next
    // row, and only feed outputs that are not stored; what must not happen is
    // a read past the matrix's end. `tight`: some chunk of these 8 rows would.
    // (reach: from this wave's first row to the end of the tile in its eighth.)
    const uint64_t mend = uniform64(gbase + (uint64_t)K * ld_bytes);
    const uint64_t col_b = uniform64((uint64_t)col0 * 2);
    const uint64_t reach = 7ull * ld_u + col_b + GM_BM * 2;
    auto at = [&](const Cursor& q) { return (const char*)(q.base + col_b); };
    auto tight = [&](const Cursor& q) { return q.base + reach > mend; };
    // `lo`: the lane's offset, copied where it is used so that no address
    // derived from it is kept in registers across the loop.
    auto fresh = [](uint32_t x) {
      asm volatile("" : "+v"(x));
      return x;
    };
    auto in_span = [&](const Cursor& q, int t, uint32_t lo) {  // the lane's chunk of row 2t + lane / 32
      return q.base + col_b + (uint64_t)(2 * t) * ld_u + lo + 16 <= mend;
    };
    auto load_set = [&](int s, Set& q) __attribute__((always_inline)) {
      if (s >= nS) return;
      const char* p = at(ld_at);
      const int rows = ld_at.left - wq * 8;  // rows left from this wave's first
      const uint32_t lo = fresh(lo0);
      if (!tight(ld_at)) {
        // Rows past the example repeat its last row here (or, where the wave
        // has none of its rows, are not read) and are zeroed when written.
        if (rows >= 8) {
#pragma unroll
          for (int t = 0; t < DL_LOADS; ++t) q[t] = load16_any(p + (size_t)(2 * t) * ld_u + lo);
        } else if (rows > 0) {
          const uint32_t odd = lane < 32 ? lo : lo - ld_u;  // the lane's offset in an even row
#pragma unroll
          for (int t = 0; t < DL_LOADS; ++t)
            q[t] = load16_any(p + (size_t)min(2 * t, rows - 1) * ld_u +
                              (2 * t + 1 < rows ? lo : odd));
        }
      } else {
#pragma unroll
        for (int t = 0; t < DL_LOADS; ++t) {
          q[t] = u32x4{0u, 0u, 0u, 0u};
          if (2 * t + (lane >> 5) < rows && in_span(ld_at, t, lo))
            q[t] = load16_any(p + (size_t)(2 * t) * ld_u + lo);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      next_stage(ld_at);
      __builtin_amdgcn_sched_barrier(0);
    };
    Cursor wr_at = ld_at;
    // ROWS: example and row within it of this wave's first row of the next
    // stage to write; row r_wr + j lies (r_wr + j) / T examples on, and
    // x / T = hi32(x * rcpT) for the x < T + DL_BK here (T <= 2 DL_BK).
    int e_wr = ROWS ? (int)((k_begin + wq * 8) / a.T) : 0;
    int r_wr = ROWS ? (int)((k_begin + wq * 8) - (int64_t)e_wr * a.T) : 0;
    const uint32_t rcpT = 0xFFFFFFFFu / (uint32_t)nT + 1u;
    auto write_set = [&](int s, Set& q) __attribute__((always_inline)) {
      if (s >= nS) return;
      char* dst = ring_raw + (s % DL_NS) * DL_STB + lds_role;
      const int rows = wr_at.left - wq * 8;
      const bool edge = tight(wr_at);
#pragma unroll
      for (int t = 0; t < DL_LOADS; ++t) {
        const uint32_t lo = fresh(lo0);
        const int lf = (int)fresh((uint32_t)lane);
        const int r = 2 * t + (lf >> 5);
        float c = 1.f;
        if constexpr (ROWS) {
          const int x = r_wr + r;
          c = factor(min(e_wr + (nT == 1 ? x : (int)__umulhi((uint32_t)x, rcpT)), nB - 1));
          // X rows scaled by their example's factor; the rows of an example
          // with c = 0 are zeroed in both operands (0 * inf would be NaN).
          if (load_x) {
#pragma unroll
            for (int k = 0; k < 4; ++k) q[t][k] = scale_bf16x2(q[t][k], c);
          }
          if (c == 0.f) q[t] = u32x4{0u, 0u, 0u, 0u};
        }
        if (rows < 8 && r >= rows) q[t] = u32x4{0u, 0u, 0u, 0u};
        char* const d = dst + r * DL_ROWB + (((lf & 31) ^ dl_sw(r)) << 4);
        *(u32x4*)d = q[t];
        // The chunk that would read past the matrix's end, element by element.
        if (edge && r < rows && c != 0.f && ncl > 0 && !in_span(wr_at, t, lo)) {
          global_u16* src = (global_u16*)(uintptr_t)(at(wr_at) + (size_t)(2 * t) * ld_u + lo);
#pragma unroll 1
          for (int k = 0; k < ncl; ++k) {
            uint32_t v = src[k];
            if (ROWS && load_x) v = scale_bf16x2(v, c);
            ((uint16_t*)d)[k] = (uint16_t)v;
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (ROWS) {
        const int x = r_wr + DL_BK;
        const int de = nT == 1 ? x : (int)__umulhi((uint32_t)x, rcpT);
        e_wr += de;
        r_wr = x - de * nT;
      }
      next_stage(wr_at);
      __builtin_amdgcn_sched_barrier(0);
    };
    Set q;
    load_set(0, q);
    if constexpr (ROWS) bar();  // write_set reads the factor table, which every wave fills
    write_set(0, q);
    load_set(1, q);
    write_set(1, q);
    load_set(2, q);
    bar();
    if constexpr (MODE == MODE_SUM && !ROWS) c_nx = factor(min(e0, nB - 1));
    if (w < 4) {
      rd(0, fr);
      enter(0);
      for (int s = 0; s < nS; ++s) {
        compute(fr);
        bar();
        write_set(s + 2, q);
        load_set(s + 3, q);
        rd(s + 1, fr);
        if (s + 1 < nS) enter(s + 1);
        bar();
      }
    } else {
      for (int s = 0; s < nS; ++s) {
        write_set(s + 2, q);
        load_set(s + 3, q);
        rd(s, fr);
        enter(s);
        bar();
        compute(fr);
        bar();
      }
    }
  } else if (w < 4) {
#pragma unroll
    for (int p = 0; p < DL_NS; ++p)
#pragma unroll
      for (int t = 0; t < DL_LOADS; ++t) issue(p, t);
    wait_vmcnt<DL_LOADS * (DL_NS - 1)>();
    bar();  // stage 0 has landed, the factor table is filled
    if constexpr (MODE == MODE_SUM && !ROWS) c_nx = factor(min(e0, nB - 1));
    if constexpr (SCALED) look_up(0);
    rd(0, fr);
    if constexpr (SCALED) {
      scale(0, fr);
      look_up(1);
    }
    enter(0);
    for (int s = 0; s < nS; ++s) {
      compute(fr);
      wait_vmcnt<DL_LOADS * (DL_NS - 2)>();
      bar();
      rd_issue(s + 1, s + DL_NS, fr);  // past the last stage: reads an unused slot
      if constexpr (SCALED) {
        scale(s + 1, fr);
        look_up(s + 2);
      }
      if (s + 1 < nS) enter(s + 1);
      bar();
    }
  } else {
#pragma unroll
    for (int p = 0; p < DL_NS - 1; ++p)
#pragma unroll
      for (int t = 0; t < DL_LOADS; ++t) issue(p, t);
    wait_vmcnt<DL_LOADS * (DL_NS - 2)>();
    bar();
    if constexpr (MODE == MODE_SUM && !ROWS) c_nx = factor(min(e0, nB - 1));
    if constexpr (SCALED) look_up(0);
    for (int s = 0; s < nS; ++s) {
      rd_issue(s, s + DL_NS - 1, fr);
      if constexpr (SCALED) {
        scale(s, fr);
        look_up(s + 1);
      }
      enter(s);
      wait_vmcnt<DL_LOADS * (DL_NS - 2)>();
      bar();
      compute(fr);
      bar();
    }
  }
  // No load may still be writing LDS when the workgroup ends.
  wait_vmcnt<0>();
  if constexpr (MODE == MODE_SUM) {
    if constexpr (!ROWS) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] *= c_acc;
    }
    if (kc >= 0) {
      // A split range: its raw partial tile, for the fixup kernel.
      __syncthreads();
      float* slice = (float*)ring_raw + w * 32 * EP_LD;
      store_partial(a.part + ((size_t)(item - a.n_full) * a.ksplit + kc) * (GM_BM * GM_BN),
                    wm, wn, lane, acc, slice);
    } else {
      // The ring is free once every wave is past its last read of it.
      __syncthreads();
      float* slice = (float*)ring_raw + w * 32 * EP_LD;
      store_tile_rows(a, L, m0, n0, wm, wn, lane, acc, slice);
    }
  } else {
    fin();  // the last example
    __syncthreads();
    if (tid < n_ex) {
      float t = 0.f;
#pragma unroll
      for (int q = 0; q < GM_THREADS / WAVE; ++q) t += red[tid * (GM_THREADS / WAVE) + q];
      a.ws[(int64_t)(b + tid) * a.slots + L.slot_begin + rel] = t;
    }
  }
}

// Clipped sum from a gradient store (the materialising form of eq. 3: the
// per-example gradients, already formed by the direct norm, weighted and
// added): one workgroup per output tile, its 8 waves in the register layout
// of dl_gemm_kernel, acc = sum_e c_e tile_e in example order (examples with
// c_e = 0 are left out, as in the GEMM), then the GEMM's own epilogue (prior,
// fused noise, 1/B; row-major, or transposed per layer). HBM-bound: B tiles
// read per output tile.
__global__ __launch_bounds__(GM_THREADS) void store_sum_kernel(GemmArgs args) {
  const GemmArgs& a = *(const GemmArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  (void)args;
  __shared__ __attribute__((aligned(1024))) char stage[(GM_THREADS / WAVE) * 32 * EP_LD * 4];
  const uint32_t item = xcd_remap(blockIdx.x, gridDim.x);
  const int ln = (int)(threadIdx.x & (WAVE - 1));
  const int l = wave_find(item, ln < a.n_layers ? a.L[ln].tile_begin : 0u, a.n_layers);
  const GemmLayer& L = a.L[l];
  const uint32_t rel = item - L.tile_begin;
  int mt, nt;
  tile_of(L, rel, mt, nt);
  const int64_t m0 = (int64_t)mt * GM_BM, n0 = (int64_t)nt * GM_BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w & 1, wn = w >> 1;
  const float* src = a.store + ((((size_t)L.store_slot + rel) * (size_t)a.B) << 16) +
                     store_lane_offset(w, lane);
  f32x16 acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x16{};
  const int nB = __builtin_amdgcn_readfirstlane(a.B);
  for (int e = 0; e < nB; ++e) {
    const float ce = a.c[e];
    if (!(ce != 0.f)) continue;
    const float* p = src + ((size_t)e << 16);
    // two halves of 16 loads each (i = 0, 1 and i = 2, 3), all in flight
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      f32x4 v[2][2][4];
#pragma unroll
      for (int ii = 0; ii < 2; ++ii)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            v[ii][j][q] = __builtin_nontemporal_load((const f32x4*)(p + store_chunk(2 * hh + ii, j, q)));
#pragma unroll
      for (int ii = 0; ii < 2; ++ii)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              acc[2 * hh + ii][j][4 * q + r] = fmaf(ce, v[ii][j][q][r], acc[2 * hh + ii][j][4 * q + r]);
    }
  }
  if (L.store_transpose) {
    store_tile_transposed(a, L, m0, n0, wm, wn, lane, acc);
  } else {
    float* slice = (float*)stage + w * 32 * EP_LD;
    store_tile_rows(a, L, m0, n0, wm, wn, lane, acc, slice);
  }
}

hipError_t launch_store_sum(const GemmArgs& a, hipStream_t s) {
  if (a.n_items == 0) return hipSuccess;
  if (!a.store || !a.c) return hipErrorInvalidValue;
  hipLaunchKernelGGL(store_sum_kernel, dim3(a.n_items), dim3(GM_THREADS), 0, s, a);
  return hipGetLastError();
}

template <int MODE>
static void launch_dl(const GemmArgs& a, int form, uint32_t grid, hipStream_t s) {
  const dim3 g(grid), blk(GM_THREADS);
  if (form == FORM_PLAIN) {
    hipLaunchKernelGGL((dl_gemm_kernel<MODE, FORM_PLAIN>), g, blk, 0, s, a);
  } else if (form == FORM_BIG) {
    hipLaunchKernelGGL((dl_gemm_kernel<MODE, FORM_BIG>), g, blk, 0, s, a);
  } else if (form == FORM_RAGGED) {
    hipLaunchKernelGGL((dl_gemm_kernel<MODE, FORM_RAGGED>), g, blk, 0, s, a);
  } else if (form == FORM_STAGED) {
    hipLaunchKernelGGL((dl_gemm_kernel<MODE, FORM_STAGED>), g, blk, 0, s, a);
  } else if constexpr (MODE == MODE_SUM) {
    if (form == FORM_ROWS)
      hipLaunchKernelGGL((dl_gemm_kernel<MODE, FORM_ROWS>), g, blk, 0, s, a);
    else
      hipLaunchKernelGGL((dl_gemm_kernel<MODE, FORM_SCALED>), g, blk, 0, s, a);
  }
}

template <int MODE>
static hipError_t launch_kt(const GemmArgs& a0, int dt, bool vec, int cus, size_t part_bytes,
                            hipStream_t s) {
  if (a0.n_items == 0) return hipSuccess;
  GemmArgs a = a0;
  a.n_full = a.n_items;
  a.n_split = 0;
  a.ksplit = 1;
  // Example groups exist only on the bf16 kernel, the gradient store only on
  // its direct loads of whole stages.
  if (MODE == MODE_NORM && (a.eg < 1 || a.eg > NG_MAX || (a.eg > 1 && dt != DT_BF16) ||
                            (a.store && !(dt == DT_BF16 && vec && a.T % DL_BK == 0))))
    return hipErrorInvalidValue;
  if (MODE == MODE_SUM && a.store) return hipErrorInvalidValue;
  uint32_t grid = a.n_items;
  if (MODE == MODE_SUM && a.part != nullptr && ((uintptr_t)a.part & 15) == 0) {
    const int form = sum_form(dt, vec, a.T, a.B);
    const TailSplit t = tail_split(a.n_items, sum_stages(form, a.T, a.B), form, a.noise != 0, cus);
    if (t.n_split > 0 && (size_t)t.n_split * t.ks * SPLIT_TILE_BYTES <= part_bytes) {
      a.n_full = t.n_full;
      a.n_split = t.n_split;
      a.ksplit = t.ks;
      grid = t.n_full + t.n_split * (uint32_t)t.ks;
    }
  }
  if (dt == DT_BF16) {
    const int form = a.big ? (int)FORM_BIG
                           : (MODE == MODE_NORM ? norm_form(vec, a.T) : sum_form(dt, vec, a.T, a.B));
    launch_dl<MODE>(a, form, grid, s);
  } else {
    hipLaunchKernelGGL((split_gemm_kernel<MODE>), dim3(grid), dim3(GM_THREADS), 0, s, a);
  }
  if (a.n_split > 0) {
    hipLaunchKernelGGL(split_fixup_kernel, dim3(a.n_split * (GM_BM * GM_BN / 4 / 256)),
                       dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_clipped_sum(const GemmArgs& a, int dt, bool vec, int cus, size_t part_bytes,
                              hipStream_t s) {
  return launch_kt<MODE_SUM>(a, dt, vec, cus, part_bytes, s);
}

hipError_t launch_direct_norm(const GemmArgs& a, int dt, bool vec, hipStream_t s) {
  return launch_kt<MODE_NORM>(a, dt, vec, 0, 0, s);
}

}  // namespace dpg
