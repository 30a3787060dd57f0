// Cache append on the matrix cores (bf16 in, fp32 accumulate).
//   Y = X [W_ke | W_dkv]   (Section 3.2: c = x A^{kv} and the elite key rows W^k_{e,h}; Section 3.1:
//   what a RoPElite model caches), computed transposed, Y^T[n, t] = sum_k W^T[n, k] X^T[k, t]:
//     A (32 x 16 per step) = W^T: the weight tile sits in LDS as stored ([k][n], n contiguous) and
//                            is read transposed (ds_read_b64_tr_b16),
//     B (16 x 32)          = X^T: a lane's eight consecutive k of one token are contiguous in x,
//     D[n, t]              : a lane ends up with ONE token and groups of four consecutive output
//                            columns, so the (even, odd) pairs that RoPE rotates stay in one lane.
//
// append_skinny: a decoding batch (2 <= T <= 64 tokens).  The weights are the traffic; they are
// streamed once, split over column blocks and over the contraction dimension so that every
// compute unit pulls a share.  fp32 partials go to the workspace; the finish kernel of the
// small-batch path sums the contraction splits, rotates and stores.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"
#include "append_skinny.hpp"

namespace ekv {

template <int TT>   // 32-token tiles (1 or 2)
__global__ __launch_bounds__(256) void append_skinny_kernel(const AppendSkinnyParams P) {
  __shared__ __attribute__((aligned(16))) char wsm[kSkLds];
  append_skinny_body<TT>(P, blockIdx.x, blockIdx.y, wsm);
}

AppendSkinnyParams make_append_skinny_params(const AppendArgs& a, float* partial, int kc) {
  const elitekv_dims& d = a.dims;
  AppendSkinnyParams P;
  P.x = (const bf16_t*)a.x; P.T = (int)a.T; P.W_ke = (const bf16_t*)a.W_ke; P.W_dkv = (const bf16_t*)a.W_dkv;
  P.W_dkv2 = (const bf16_t*)a.W_dkv2; P.partial = partial; P.d_ck = a.d_ck; P.d = d.d_model;
  P.NE = 2 * d.r * d.n_heads; P.d_c = d.d_c; P.kc = kc;
  return P;
}

bool append_skinny_supported(const elitekv_dims& d, int64_t T, int d_ck) {
  if (d.dtype != ELITEKV_BF16 || T < kMatrixRows || T > 64) return false;
  const int NE = 2 * d.r * d.n_heads;
  return NE % kSkCols == 0 && d.d_c % kSkCols == 0 && d_ck % kSkCols == 0 && d.d_model % 8 == 0;
}

// contraction splits: about one work-group per compute unit, whole stages per split
int append_skinny_ksplit(const elitekv_dims& d) {
  const int blocks = (2 * d.r * d.n_heads + d.d_c) / kSkCols;
  int ks = (256 + blocks - 1) / blocks;
  const int max_ks = (d.d_model + kSkStage - 1) / kSkStage;
  if (ks > max_ks) ks = max_ks;
  return ks < 1 ? 1 : ks;
}

int append_skinny_kc(const elitekv_dims& d, int ks) {
  const int kc = (d.d_model + ks - 1) / ks;
  return (kc + kSkStage - 1) / kSkStage * kSkStage;
}

size_t append_skinny_workspace(const elitekv_dims& d, int64_t T) {
  return (size_t)append_skinny_ksplit(d) * (size_t)T * (size_t)(2 * d.r * d.n_heads + d.d_c) * sizeof(float);
}

hipError_t launch_append_skinny(const AppendArgs& a, hipStream_t stream) {
  const elitekv_dims& d = a.dims;
  const int NE = 2 * d.r * d.n_heads, N = NE + d.d_c;
  int ks = append_skinny_ksplit(d);
  const int kc = append_skinny_kc(d, ks);
  ks = (d.d_model + kc - 1) / kc;            // splits that still have rows; never more than planned
  float* partial = (float*)a.ws;
  const dim3 grid(N / kSkCols, ks);
  const AppendSkinnyParams P = make_append_skinny_params(a, partial, kc);
  if (a.T <= 32) append_skinny_kernel<1><<<grid, 256, 0, stream>>>(P);
  else append_skinny_kernel<2><<<grid, 256, 0, stream>>>(P);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_append_finish(a, partial, ks, stream);
}

// ---------------------------------------------------------------------------------------------
// append_gemm: prefill-sized appends (T > 64).  A dense contraction bounded by the matrix cores.
// Work-group tile: 128 output columns x (64 * WN) tokens, 2 x 2 waves, each wave 64 columns x
// (32 * WN) tokens = 2 x WN accumulator tiles of 32 x 32.  Both operands go through LDS in
// double-buffered stages of 64 contraction rows (global -> registers -> LDS, the loads of stage
// s+1 in flight while stage s is multiplied).  The epilogue (gemm_store, shared by all the GEMM kernels) takes the tile
// through LDS, rotates the elite pairs there and stores whole pieces of bf16 rows.
// ---------------------------------------------------------------------------------------------
constexpr int kGmCols = 128;                   // output columns per work-group
constexpr int kGmStage = 64;                   // contraction rows per stage
constexpr int kGmARow = kGmCols * 2 + 32;      // bytes of a staged weight row [k][128 n] (+ bank spread)
constexpr int kGmBRow = kGmStage * 2 + 16;     // bytes of a staged token row [t][64 k] (+ bank spread)

template <int NI>
struct GemmStore {
  static constexpr int kRow = NI * 32 + 4;    // floats of a token's columns in LDS
  static constexpr int kWaveBytes = 32 * kRow * 4;
};

template <int WN>
struct GemmLayout {
  static constexpr int BN = 64 * WN;                          // tokens per work-group
  static constexpr int A_BYTES = kGmStage * kGmARow;
  static constexpr int B_BYTES = BN * kGmBRow;
  static constexpr int STAGE = A_BYTES + B_BYTES;
  static constexpr int LDS_BYTES = 2 * STAGE;
  static_assert(4 * GemmStore<2>::kWaveBytes <= LDS_BYTES, "the epilogue reuses the staging buffers");
  static constexpr int NB = BN * 8 / 256;                     // 16-byte token pieces per thread per stage
};

// Epilogue of the GEMM kernels.  A wave holds 32 NI columns (from nw) x 32 NJ tokens (from tw): registers 4 g .. 4 g + 3 of
// accumulator tile (i, j) are columns nw + 32 i + 8 g + 4 (lane / 32) + {0, 1, 2, 3} of token tw + 32 j + lane % 32.  The tile
// leaves through the wave's own piece of LDS, 32 tokens at a time, so that a store instruction writes whole pieces of
// rows (64 NI bytes; straight from the accumulators it would touch 32 rows with 16 bytes each), and so that the
// rotation of the elite pairs is one short loop: unrolled over the accumulators it was 230 KB of code, which every work-group
// fetched anew.  1536 x 7680 x 2048 tokens, 256 x 256 tiles: 80 -> 61 us a launch; 4096 x 2048 x 32768: 620 -> 534.
template <int NI, int NJ, typename Acc>
__device__ __forceinline__ void gemm_store(const Acc& acc, char* lds, int wave, int nw, int64_t tw, int lane, int64_t T,
                                           const int32_t* __restrict__ pos, const int64_t* __restrict__ slot,
                                           const int32_t* __restrict__ elite_idx, bf16_t* __restrict__ ke_plane,
                                           bf16_t* __restrict__ c_plane, int64_t plane_rows, int n_h, int d_h, int r, int d_c,
                                           const RopeTable& rope) {
  using G = GemmStore<NI>;
  constexpr int kLanes = NI * 4, kRows = 64 / kLanes;         // lanes per row of the tile, rows per instruction
  float* buf = reinterpret_cast<float*>(lds + wave * G::kWaveBytes);
  const int NE = 2 * r * n_h;
  const int n32 = lane & 31, hi = lane >> 5;
  // this lane's eight columns on the way out
  const int cl = (lane % kLanes) * 8, n = nw + cl, rl = lane / kLanes;
  const bool elite = n < NE;
  double theta[4] = {0.0, 0.0, 0.0, 0.0};
  if (elite) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {             // slots of the four pairs, which may belong to different heads
      const int m = n + 2 * e;
      int ch = elite_idx[(m / (2 * r)) * r + ((m % (2 * r)) >> 1)];
      ch = min(max(ch, 0), d_h / 2 - 1);
      theta[e] = rope.theta[ch];
    }
  }
  bf16_t* plane = elite ? ke_plane + n : c_plane + (n - NE);
  const int64_t ld_out = elite ? NE : d_c;
  // destination rows (-1: not stored) and positions of the tile's tokens, one token per lane and j, requested at once
  int64_t rows[NJ];
  int32_t posn[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int64_t t = min(tw + j * 32 + n32, T - 1);
    rows[j] = slot ? slot[t] : t;                             // no slot list: rows are written in place
    posn[j] = pos ? pos[t] : 0;
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j)
    if (tw + j * 32 + n32 >= T || rows[j] >= plane_rows || rows[j] < 0) rows[j] = -1;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const am_f32x16& a = acc(i, j);
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<float4*>(buf + n32 * G::kRow + i * 32 + 8 * g + 4 * hi) =
            make_float4(a[4 * g], a[4 * g + 1], a[4 * g + 2], a[4 * g + 3]);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");        // the wave's own pieces
#pragma unroll 4
    for (int it = 0; it < 32 / kRows; ++it) {
      const int tl = it * kRows + rl;
      const float4 lo = *reinterpret_cast<const float4*>(buf + tl * G::kRow + cl);
      const float4 up = *reinterpret_cast<const float4*>(buf + tl * G::kRow + cl + 4);
      float v[8] = {lo.x, lo.y, lo.z, lo.w, up.x, up.y, up.z, up.w};
      const int64_t row = ((int64_t)__shfl((int)(rows[j] >> 32), tl, kWave) << 32) | (uint32_t)__shfl((int)rows[j], tl, kWave);
      const int32_t p = __shfl(posn[j], tl, kWave);
      if (row < 0) continue;
      if (elite) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float sn, cs;
          rope_sincos_poly(p, theta[e], &sn, &cs);
          const float x0 = v[2 * e] * cs - v[2 * e + 1] * sn, x1 = v[2 * e] * sn + v[2 * e + 1] * cs;
          v[2 * e] = x0; v[2 * e + 1] = x1;
        }
      }
      ekv_u32x4 pk;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        pk[e] = (uint32_t)f32_to_bf16_bits(v[2 * e]) | ((uint32_t)f32_to_bf16_bits(v[2 * e + 1]) << 16);
      __builtin_nontemporal_store(pk, reinterpret_cast<ekv_u32x4*>(plane + row * ld_out));
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");        // read before the next tokens overwrite it
  }
}

template <int WN>
__global__ __launch_bounds__(256) void append_gemm_kernel(
    const bf16_t* __restrict__ x, const int32_t* __restrict__ pos, const int64_t* __restrict__ slot, int64_t T,
    const bf16_t* __restrict__ W_ke, const bf16_t* __restrict__ W_dkv, const bf16_t* __restrict__ W_dkv2, int d_ck,
    const int32_t* __restrict__ elite_idx, bf16_t* __restrict__ ke_plane, bf16_t* __restrict__ c_plane, int64_t plane_rows, int d, int n_h, int d_h,
    int r, int d_c, RopeTable rope) {
  using L = GemmLayout<WN>;
  extern __shared__ __attribute__((aligned(16))) char gsm[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave & 1, wn = wave >> 1;                    // wave's 64-column half, token half
  const int n32 = lane & 31, hi = lane >> 5, i16 = lane & 15, q16 = lane >> 4;
  const int NE = 2 * r * n_h;
  const int n0 = blockIdx.x * kGmCols;
  const int64_t t0 = (int64_t)blockIdx.y * L::BN;
  const int nstages = (d + kGmStage - 1) / kGmStage;

  // this thread always loads the same 8-column piece (tid % 16) of a weight row; each 64-column
  // half of the block lies in one of the weight matrices
  const bf16_t* wbase;
  int64_t wstride;
  weight_column(n0 + ((tid & 8) ? 64 : 0), NE, d_ck, d_c, W_ke, W_dkv, W_dkv2, &wbase, &wstride);
  wbase += (tid & 7) * 8;

  uint4 areg[4], breg[L::NB];
  auto load_stage = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {               // weights: 64 rows x 16 pieces
      const int e = i * 256 + tid, k = k0 + (e >> 4);
      areg[i] = make_uint4(0, 0, 0, 0);
      if (k < d) areg[i] = *reinterpret_cast<const uint4*>(wbase + (int64_t)k * wstride);
    }
#pragma unroll
    for (int i = 0; i < L::NB; ++i) {           // tokens: BN rows x 8 pieces
      const int e = i * 256 + tid, ch = e & 7;
      const int64_t t = t0 + (e >> 3);
      const int k = k0 + ch * 8;
      breg[i] = make_uint4(0, 0, 0, 0);
      if (t < T && k < d) breg[i] = *reinterpret_cast<const uint4*>(x + t * d + k);
    }
  };
  auto store_stage = [&](int buf) {
    char* As = gsm + buf * L::STAGE;
    char* Bs = As + L::A_BYTES;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = i * 256 + tid;
      *reinterpret_cast<uint4*>(As + (e >> 4) * kGmARow + (e & 15) * 16) = areg[i];
    }
#pragma unroll
    for (int i = 0; i < L::NB; ++i) {
      const int e = i * 256 + tid;
      *reinterpret_cast<uint4*>(Bs + (e >> 3) * kGmBRow + (e & 7) * 16) = breg[i];
    }
  };

  am_f32x16 acc[2][WN];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) acc[i][j] = (am_f32x16)(0.f);

  // operand offsets inside a stage
  const int a_off = (8 * (q16 >> 1) + (i16 >> 2)) * kGmARow + wm * 128 + 32 * (q16 & 1) + 8 * (i16 & 3);
  const int b_off = (wn * 32 * WN + n32) * kGmBRow + hi * 16;

  auto compute = [&](int buf) {
    const char* As = gsm + buf * L::STAGE;
    const char* Bs = As + L::A_BYTES;
#pragma unroll
    for (int ks = 0; ks < kGmStage / 16; ++ks) {
      am_bf16x8 a[2], b[WN];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const char* base = As + a_off + ks * 16 * kGmARow + i * 64;
        const am_s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((am_lds_s16x4_t*)(base));
        const am_s16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((am_lds_s16x4_t*)(base + 4 * kGmARow));
        a[i] = __builtin_bit_cast(am_bf16x8, __builtin_shufflevector(lo, hi4, 0, 1, 2, 3, 4, 5, 6, 7));
      }
#pragma unroll
      for (int j = 0; j < WN; ++j)
        b[j] = *reinterpret_cast<const am_bf16x8*>(Bs + b_off + j * 32 * kGmBRow + ks * 32);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  };

  load_stage(0);
  store_stage(0);
  __syncthreads();
  for (int s = 0; s < nstages; ++s) {
    const bool more = s + 1 < nstages;
    if (more) load_stage((s + 1) * kGmStage);
    compute(s & 1);
    if (more) store_stage((s + 1) & 1);
    __syncthreads();
  }

  // (the last stage's barrier has passed: the staging buffers are free)
  gemm_store<2, WN>([&](int i, int j) -> const am_f32x16& { return acc[i][j]; }, gsm, wave, n0 + wm * 64, t0 + wn * 32 * WN, lane,
                    T, pos, slot, elite_idx, ke_plane, c_plane, plane_rows, n_h, d_h, r, d_c, rope);
}

// ---------------------------------------------------------------------------------------------
// append_gemm_dma: the same GEMM with both operands brought in by direct global->LDS loads into a
// ring of NS stages of 32 contraction rows (no register staging, one barrier per stage, the loads
// of the next NS-2 stages in flight while a stage is multiplied).  CM x WNW waves: CM along the
// 64 CM columns, WNW along the tokens; the widest tiles run eight waves, two per SIMD.  A direct load writes 1 KiB
// (64 lanes x 16 bytes) contiguously, so the LDS layouts are made of 1 KiB blocks:
//   weights  [32 k][64 CM n]: blocks of 8 rows x 128 bytes, 16-byte pieces XOR-swizzled by row
//            (conflict-free transposed reads), block (kb, nb) at (kb*CM + nb) KiB;
//   tokens   [BN t][32 k]:  blocks of 16 rows x 64 bytes, pieces XOR-swizzled by row.
// Needs d_model % 32 == 0 (whole stages); other shapes take append_gemm_kernel.
// ---------------------------------------------------------------------------------------------

__device__ __forceinline__ int gd_swz8(int row) { return ((row & 3) << 1) | ((row >> 2) & 1); }
// token blocks (16 rows x 64 bytes): a 16-byte read of 16 lanes = 16 rows at one logical piece; the four
// rows r, r+4, r+8, r+12 that share a 64-byte bank window take four different pieces
__device__ __forceinline__ int gd_swz4(int row) { return (row >> 2) & 3; }

// (M0 is read one wait state after its write: the s_nop, which the compiler does not put into inline assembly)
__device__ __forceinline__ void gd_dma16(const void* gptr, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_base), "v"(gptr) : "memory", "m0");
}

// WN = 32-token tiles per wave, WNW = waves along the tokens, CM = waves along the columns (64 columns each)
template <int WN, int NS, int WNW, int CM>
struct GemmDmaLayout {
  static constexpr int BN = 32 * WN * WNW;                    // tokens per work-group
  static constexpr int COLS = 64 * CM;                        // output columns per work-group
  static constexpr int NWAVES = CM * WNW;
  static constexpr int A_BYTES = kGdStage * COLS * 2;         // weight stage
  static constexpr int WB = A_BYTES / 1024;                   // ... in 1 KiB blocks (kb = 0..3, nb = 0..CM-1)
  static constexpr int B_BYTES = BN * 64;                     // token stage
  static constexpr int STAGE = A_BYTES + B_BYTES;
  static constexpr int LDS_BYTES = NS * STAGE;
  static constexpr int LOADS = STAGE / 1024;                  // direct loads per stage per work-group
  static constexpr int LPW = LOADS / NWAVES;                  // ... per wave
  static_assert(LOADS % NWAVES == 0, "the loads of a stage are divided evenly among the waves");
  static_assert(LDS_BYTES <= 160 * 1024, "exceeds the LDS of a compute unit");
  static_assert(NWAVES * GemmStore<2>::kWaveBytes <= LDS_BYTES, "the epilogue reuses the ring");
  static_assert(NS >= 3 && NS <= 12 && (NS - 2) * LPW <= 63, "ring depth outside what the load counter can express");
};

struct GemmTileMap {              // which (column block, token block) a work-group takes; see gemm_tile_map
  int xt, tb_x, cb_x, group, col_blocks;
};
__device__ __forceinline__ bool gemm_tile_of(const GemmTileMap& m, int wg, int* cb, int64_t* tb) {
  const int xcd = wg & 7, seq = wg >> 3;
  const int g = seq / (m.group * m.cb_x), rem = seq - g * m.group * m.cb_x;
  const int in_group = min(m.group, m.tb_x - g * m.group);
  *tb = (int64_t)(g * m.group + rem % in_group) * m.xt + xcd % m.xt;
  const int c = rem / in_group;
  *cb = (xcd / m.xt) * m.cb_x + c;
  return c < m.cb_x && *cb < m.col_blocks;
}

// SPB = stages consumed per barrier (1 or 2).  With 2 the work-group synchronises once per 64 contraction rows:
// half as many barriers and load waits, the operands of the second stage of a pair read while the first is
// multiplied, NS - 2 stages in flight behind the pair.
// KG = groups of waves that split the contraction rows of every stage between them (1 or 2).  With 2 (eight waves on
// a 128 x 128 tile) the waves of a group own 64 x 64 outputs each instead of 64 x 32 and take one of the two 16-row
// k-steps of every stage: a wave then reads 4 KB instead of 6 KB of operands from LDS per four MFMAs (the LDS, not the
// matrix cores, is the busiest unit of this tile: 48 KB read + 16 KB written per stage against 128 B per cycle), and the
// two groups add their halves through LDS once, before the epilogue.
template <int WN, int NS, int WNW, int CM, int SPB, int KG>
__global__ __launch_bounds__(64 * CM * WNW) void append_gemm_dma_kernel(
    const bf16_t* __restrict__ x, const int32_t* __restrict__ pos, const int64_t* __restrict__ slot, int64_t T,
    const bf16_t* __restrict__ W_ke, const bf16_t* __restrict__ W_dkv, const bf16_t* __restrict__ W_dkv2, int d_ck,
    const int32_t* __restrict__ elite_idx, bf16_t* __restrict__ ke_plane, bf16_t* __restrict__ c_plane,
    int64_t plane_rows, int d, int n_h, int d_h, int r, int d_c, RopeTable rope, int64_t x_ld, int x_off2, int d2,
    GemmTileMap map, int* clear, int n_clear) {
  using L = GemmDmaLayout<WN, NS, WNW, CM>;
  extern __shared__ __attribute__((aligned(16))) char gsm[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (blockIdx.x == 0)
    for (int i = tid; i < n_clear; i += blockDim.x) clear[i] = 0;
  static_assert(KG == 1 || (KG == 2 && WN == 1 && WNW == 4 && CM == 2), "contraction groups: eight waves on 128 x 128");
  constexpr int WNC = KG * WN;                     // 32-token tiles a wave accumulates
  constexpr int KSN = 2 / KG;                      // k-steps of a stage a wave multiplies
  const int kg = KG == 2 ? wave >> 2 : 0;          // contraction group of this wave
  const int wv = KG == 2 ? wave & 3 : wave;        // wave inside its group
  const int wm = wv % CM, wn = wv / CM;
  const int n32 = lane & 31, hi = lane >> 5, i16 = lane & 15, q16 = lane >> 4;
  const int NE = 2 * r * n_h;
  int cb;
  int64_t tblock;
  if (!gemm_tile_of(map, blockIdx.x, &cb, &tblock)) return;
  const int64_t t0 = tblock * L::BN;
  if (t0 >= T) return;
  // an odd last half block of columns is computed together with the half before it, which is then written twice
  const int n0 = min(cb * L::COLS, NE + d_c - L::COLS);
  // a column block inside W_dkv2 may contract a different column slice of the input rows (d2 > 0; the host
  // makes sure that no block straddles the two matrices then)
  const bool second = d2 > 0 && n0 - NE >= d_ck;
  const bf16_t* xs = second ? x + x_off2 : x;
  const int nstages = (second ? d2 : d) / kGdStage;

  // ---- loader.  Wave w issues loads w*LPW .. w*LPW+LPW-1 of a stage; load index < WB is weight block
  // (kb = idx / CM, nb = idx % CM), the others are token blocks of 16 rows.
  const char* gsrc[L::LPW];      // this lane's global address for the next stage to be requested
  int64_t gstep[L::LPW];         // bytes to advance per stage
#pragma unroll
  for (int u = 0; u < L::LPW; ++u) {
    const int idx = wave * L::LPW + u;
    if (idx < L::WB) {
      const int kb = idx / CM, nb = idx % CM, row = lane >> 3, pc = (lane & 7) ^ gd_swz8(row);
      const bf16_t* wb;
      int64_t ws;
      weight_column(n0 + nb * 64, NE, d_ck, d_c, W_ke, W_dkv, W_dkv2, &wb, &ws);
      gsrc[u] = reinterpret_cast<const char*>(wb + (int64_t)(kb * 8 + row) * ws + pc * 8);
      gstep[u] = (int64_t)kGdStage * ws * 2;
    } else {
      const int tb = idx - L::WB, row = lane >> 2, pc = (lane & 3) ^ gd_swz4(row);
      const int64_t t = min(t0 + tb * 16 + row, T - 1);        // rows past the end repeat the last token
      gsrc[u] = reinterpret_cast<const char*>(xs + t * x_ld + pc * 8);
      gstep[u] = (int64_t)kGdStage * 2;
    }
  }
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)gsm);
  int issue_slot = 0;            // ring slot of the next stage to be requested; stages are requested in order
  auto issue = [&]() {
    const uint32_t base = __builtin_amdgcn_readfirstlane(lds0 + issue_slot * L::STAGE + wave * L::LPW * 1024);
#pragma unroll
    for (int u = 0; u < L::LPW; ++u) {
      gd_dma16(gsrc[u], base + u * 1024);
      gsrc[u] += gstep[u];
    }
    issue_slot = (issue_slot + 1 == NS) ? 0 : issue_slot + 1;
  };

  am_f32x16 acc[2][WNC];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < WNC; ++j) acc[i][j] = (am_f32x16)(0.f);

  // ---- operand read offsets inside a stage
  // weights, transposed read: k rows 8*(q16/2) + 4e + i16/4 of a k-step (block kb = 2*ks + q16/2 ...)
  int a_off[2][2];               // [i: 32-column tile of the wave's 64-column half][e: rows 0-3 | 4-7]
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int r8 = 4 * e + (i16 >> 2);
      const int piece = (i << 2) | ((q16 & 1) << 1) | ((i16 & 3) >> 1);       // 16-byte piece inside the 128-byte row
      a_off[i][e] = ((q16 >> 1) * CM + wm) * 1024 + r8 * 128 + ((piece ^ gd_swz8(r8)) << 4) + ((i16 & 1) << 3);
    }
  // tokens: row n32 of tile j (block 2*(wn*WN + j) + n32/16), piece 2*ks + hi
  int b_off[2];                  // [ks]
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int row = n32 & 15;
    b_off[ks] = L::A_BYTES + (wn * WNC * 2 + (n32 >> 4)) * 1024 + row * 64 + (((2 * ks + hi) ^ gd_swz4(row)) << 4);
  }

  const int b_off_g = kg ? b_off[1] : b_off[0];   // contraction groups: the group's k-step
  // wait until this wave's direct loads have landed except those of the `ahead` most recent stages
  auto wait_loads = [&](int ahead) {
    switch (ahead) {
      case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
#define EKV_WAIT(K) case K: if constexpr (K <= NS - 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(K * L::LPW) : "memory"); break;
      EKV_WAIT(1) EKV_WAIT(2) EKV_WAIT(3) EKV_WAIT(4) EKV_WAIT(5) EKV_WAIT(6) EKV_WAIT(7) EKV_WAIT(8) EKV_WAIT(9) EKV_WAIT(10)
#undef EKV_WAIT
      default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    }
  };
  // operands of one stage in registers: both 16-row k-steps
  struct StageOps {
    am_bf16x8 a[KSN][2];         // [k-step][32-column tile]
    am_bf16x8 b[KSN][WNC];       // [k-step][32-token tile]
  };
  int read_slot = 0;             // ring slot of the next stage to be read into registers; stages are read in order
  auto read_ops = [&](StageOps& o) {
    const char* st = gsm + read_slot * L::STAGE;
    read_slot = (read_slot + 1 == NS) ? 0 : read_slot + 1;
#pragma unroll
    for (int kq = 0; kq < KSN; ++kq) {
      const int ks = KG == 2 ? kg : kq;            // the group's k-step of the stage
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        // a k-step is two 8-row weight blocks per 64-column block: 2 * CM KiB
        const am_s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((am_lds_s16x4_t*)(st + ks * 2048 * CM + a_off[i][0]));
        const am_s16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((am_lds_s16x4_t*)(st + ks * 2048 * CM + a_off[i][1]));
        o.a[kq][i] = __builtin_bit_cast(am_bf16x8, __builtin_shufflevector(lo, hi4, 0, 1, 2, 3, 4, 5, 6, 7));
      }
#pragma unroll
      for (int j = 0; j < WNC; ++j) o.b[kq][j] = *reinterpret_cast<const am_bf16x8*>(st + (KG == 2 ? b_off_g : b_off[kq]) + j * 2048);
    }
  };
  auto multiply = [&](const StageOps& o) {
#pragma unroll
    for (int ks = 0; ks < KSN; ++ks)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < WNC; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.a[ks][i], o.b[ks][j], acc[i][j], 0, 0, 0);
  };

  if constexpr (SPB == 1) {
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
      if (s < nstages) issue();
    // Ring pipeline: stages s+1 .. s+NS-2 stay in flight while stage s is consumed.  (A version skewed
    // by one stage -- the operands of stage s+1 read into a second register set while stage s is
    // multiplied -- hides the LDS latency and the barrier but keeps one stage less in flight; it
    // measured 5 % slower with eight waves and 20 % slower with four.)
    for (int s = 0; s < nstages; ++s) {
      wait_loads(min(nstages - 1 - s, NS - 2));                   // this wave's loads of stage s have landed
      __syncthreads();             // every wave's part of stage s is in LDS; everyone is done with stage s-1
      if (s + NS - 1 < nstages) issue();                          // into the buffer stage s-1 occupied
      StageOps ops;
      read_ops(ops);
      multiply(ops);
    }
  } else {
    static_assert(SPB == 2 && NS >= 4, "pairs of stages need a ring of at least four");
#pragma unroll
    for (int s = 0; s < NS - 2; ++s)
      if (s < nstages) issue();
    // Stages s and s+1 are consumed behind one barrier; before it NS-4 later stages may still be in flight,
    // after it the two buffers of stages s-2 and s-1 are refilled (NS-2 stages in flight behind the pair).
    for (int s = 0; s < nstages; s += 2) {
      wait_loads(max(min(nstages, s + NS - 2) - (s + 2), 0));     // this wave's loads of stages s, s+1 have landed
      __syncthreads();
      if (s + NS - 2 < nstages) issue();
      if (s + NS - 1 < nstages) issue();
      StageOps o0, o1;
      read_ops(o0);
      if (s + 1 < nstages) read_ops(o1);
      multiply(o0);
      if (s + 1 < nstages) multiply(o1);
    }
  }

  if constexpr (KG == 2) {
    // The two groups hold sums over different contraction rows of the same 64 x 64 outputs.  Group g finishes the
    // g-th 32-token tile: every wave leaves the tile it does not finish in LDS (the ring is free now), adds what its
    // partner of the other group left for it, and runs the epilogue on 64 columns x 32 tokens.
    static_assert(8 * 2 * 16 * 64 * 4 <= L::LDS_BYTES, "the exchange reuses the ring");
    __syncthreads();
    float* xb = reinterpret_cast<float*>(gsm);
    auto put = [&](int writer, const am_f32x16 (&t)[2]) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) xb[((writer * 2 + i) * 16 + v) * 64 + lane] = t[i][v];
    };
    am_f32x16 fin[2][1];
    if (kg == 0) {
      const am_f32x16 other[2] = {acc[0][1], acc[1][1]};
      put(wv * 2 + 0, other);
      fin[0][0] = acc[0][0]; fin[1][0] = acc[1][0];
    } else {
      const am_f32x16 other[2] = {acc[0][0], acc[1][0]};
      put(wv * 2 + 1, other);
      fin[0][0] = acc[0][1]; fin[1][0] = acc[1][1];
    }
    __syncthreads();
    const int partner = wv * 2 + (1 - kg);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) fin[i][0][v] += xb[((partner * 2 + i) * 16 + v) * 64 + lane];
    __syncthreads();
    gemm_store<2, 1>([&](int i, int j) -> const am_f32x16& { return fin[i][j]; }, gsm, wave, n0 + wm * 64,
                     t0 + (wn * 2 + kg) * 32, lane, T, pos, slot, elite_idx, ke_plane, c_plane, plane_rows, n_h, d_h, r, d_c,
                     rope);
  } else {
    __syncthreads();                          // every wave is done with the ring
    gemm_store<2, WN>([&](int i, int j) -> const am_f32x16& { return acc[i][j]; }, gsm, wave, n0 + wm * 64,
                      t0 + wn * 32 * WN, lane, T, pos, slot, elite_idx, ke_plane, c_plane, plane_rows, n_h, d_h, r, d_c, rope);
  }
}

// ---------------------------------------------------------------------------------------------
// append_gemm_wide: 256 columns x 256 tokens per work-group by FOUR waves, one per SIMD, each 128 x 128 outputs.
// At this tile the LDS is what eight waves of 64 x 128 keep busy: per 16 contraction rows they read 48 KB and the direct
// loads write 16 KB, 512 cycles of 128 bytes, beside 512 cycles of matrix instructions.  Four waves read 32 KB.  With one
// wave per SIMD nothing else hides a wave's waits, so the loop is skewed by one k-step of 16 rows and ordered by hand: while
// the 16 products of a k-step run, the operands of the next one are read into a second register set, two reads per product;
// the barrier that publishes the next stage sits between two products; the direct loads of the stage that takes the freed
// buffer go out one per product.
// 4096 x 2048 x 32768 tokens: 493 us = 1114 TFLOP/s (eight waves 521).
// ---------------------------------------------------------------------------------------------
template <int NS>
struct GemmWideLayout {
  static constexpr int A_BYTES = kGdStage * 256 * 2, STAGE = 2 * A_BYTES, LDS_BYTES = NS * STAGE, LPW = STAGE / 1024 / 4;
  static_assert(LDS_BYTES <= 160 * 1024 && (NS - 1) * LPW <= 63, "ring depth");
};

template <int NS>
__global__ __launch_bounds__(256, 1) void append_gemm_wide_kernel(
    const bf16_t* __restrict__ x, const int32_t* __restrict__ pos, const int64_t* __restrict__ slot, int64_t T,
    const bf16_t* __restrict__ W_ke, const bf16_t* __restrict__ W_dkv, const bf16_t* __restrict__ W_dkv2, int d_ck,
    const int32_t* __restrict__ elite_idx, bf16_t* __restrict__ ke_plane, bf16_t* __restrict__ c_plane,
    int64_t plane_rows, int d, int n_h, int d_h, int r, int d_c, RopeTable rope, int64_t x_ld, int x_off2, int d2,
    GemmTileMap map, int* clear, int n_clear) {
  using L = GemmWideLayout<NS>;
  extern __shared__ __attribute__((aligned(16))) char gsm[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (blockIdx.x == 0)
    for (int i = tid; i < n_clear; i += blockDim.x) clear[i] = 0;
  const int wm = wave & 1, wn = wave >> 1;
  const int n32 = lane & 31, hi = lane >> 5, i16 = lane & 15, q16 = lane >> 4;
  const int NE = 2 * r * n_h, N = NE + d_c;
  int cb;
  int64_t tb;
  if (!gemm_tile_of(map, blockIdx.x, &cb, &tb)) return;
  const int64_t t0 = tb * 256;
  if (t0 >= T) return;
  const int n0 = min(cb * 256, N - 256);      // an odd last half block is computed with the half before it, twice
  const bool second = d2 > 0 && n0 - NE >= d_ck;
  const bf16_t* xs = second ? x + x_off2 : x;
  const int nstages = (second ? d2 : d) / kGdStage;

  // ---- loader: waves 0, 1 bring the weights (16 blocks of 8 rows x 64 columns), waves 2, 3 the tokens (16 blocks of 16)
  const char* gsrc[L::LPW];
  int64_t gstep[L::LPW];
#pragma unroll
  for (int u = 0; u < L::LPW; ++u) {
    const int idx = wave * L::LPW + u;
    if (idx < 16) {
      const int kb = idx >> 2, nb = idx & 3, row = lane >> 3, pc = (lane & 7) ^ gd_swz8(row);
      const bf16_t* wb;
      int64_t ws;
      weight_column(n0 + nb * 64, NE, d_ck, d_c, W_ke, W_dkv, W_dkv2, &wb, &ws);
      gsrc[u] = reinterpret_cast<const char*>(wb + (int64_t)(kb * 8 + row) * ws + pc * 8);
      gstep[u] = (int64_t)kGdStage * ws * 2;
    } else {
      const int tbk = idx - 16, row = lane >> 2, pc = (lane & 3) ^ gd_swz4(row);
      const int64_t t = min(t0 + tbk * 16 + row, T - 1);         // rows past the end repeat the last token
      gsrc[u] = reinterpret_cast<const char*>(xs + t * x_ld + pc * 8);
      gstep[u] = (int64_t)kGdStage * 2;
    }
  }
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)gsm);
  int issue_slot = 0;
  auto issue_one = [&](int u) {
    const uint32_t base = __builtin_amdgcn_readfirstlane(lds0 + issue_slot * L::STAGE + wave * L::LPW * 1024);
    gd_dma16(gsrc[u], base + u * 1024);
    gsrc[u] += gstep[u];
    if (u == L::LPW - 1) issue_slot = (issue_slot + 1 == NS) ? 0 : issue_slot + 1;
  };

  am_f32x16 acc[4][4];                        // [32-column tile][32-token tile]
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = (am_f32x16)(0.f);

  int a_off[2][2];                            // [32-column tile of a 64-column block][rows 0-3 | 4-7 of a weight block]
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int r8 = 4 * e + (i16 >> 2);
      const int piece = (i << 2) | ((q16 & 1) << 1) | ((i16 & 3) >> 1);
      a_off[i][e] = ((q16 >> 1) * 4 + wm * 2) * 1024 + r8 * 128 + ((piece ^ gd_swz8(r8)) << 4) + ((i16 & 1) << 3);
    }
  int b_off[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int row = n32 & 15;
    b_off[ks] = L::A_BYTES + (wn * 8 + (n32 >> 4)) * 1024 + row * 64 + (((2 * ks + hi) ^ gd_swz4(row)) << 4);
  }

  struct Ops {
    am_s16x4 a[4][2];
    am_bf16x8 b[4];
  };
  // operand read u (of 12) of k-step ks of the stage at st: the first products need tile 0 of both
  auto read_one = [&](Ops& o, const char* st, int ks, int u) {
    const int k = u / 3, w = u % 3;
    if (w < 2) o.a[k][w] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                   (am_lds_s16x4_t*)(st + ks * 8192 + (k >> 1) * 1024 + a_off[k & 1][w]));
    else o.b[k] = *reinterpret_cast<const am_bf16x8*>(st + b_off[ks] + k * 2048);
  };
  auto product = [&](const Ops& o, int m) {
    const int i = m >> 2, j = m & 3;
    const am_bf16x8 a = __builtin_bit_cast(am_bf16x8, __builtin_shufflevector(o.a[i][0], o.a[i][1], 0, 1, 2, 3, 4, 5, 6, 7));
    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, o.b[j], acc[i][j], 0, 0, 0);
  };
  auto wait_loads = [&](int ahead) {
    switch (ahead) {
      case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
#define EKV_WAIT(K) case K: if constexpr (K <= NS - 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(K * L::LPW) : "memory"); break;
      EKV_WAIT(1) EKV_WAIT(2) EKV_WAIT(3) EKV_WAIT(4)
#undef EKV_WAIT
      default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    }
  };

  for (int s = 0; s < NS && s < nstages; ++s) {
#pragma unroll
    for (int u = 0; u < L::LPW; ++u) issue_one(u);
  }
  Ops o0, o1;
  wait_loads(min(nstages, NS) - 1);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int u = 0; u < 12; ++u) read_one(o0, gsm, 0, u);
  int slot_s = 0;
  // stage s: its first k-step is in o0.  STEADY: a stage s + NS exists.
  auto stage = [&](int s, auto steady) {
    constexpr bool STEADY = decltype(steady)::value;
    const char* st = gsm + slot_s * L::STAGE;
    slot_s = (slot_s + 1 == NS) ? 0 : slot_s + 1;
    const char* st_next = gsm + slot_s * L::STAGE;
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      if (m < 6) { read_one(o1, st, 1, 2 * m); read_one(o1, st, 1, 2 * m + 1); }
      product(o0, m);
      __builtin_amdgcn_sched_barrier(0);
    }
    const bool more = STEADY || s + 1 < nstages, refill = STEADY || s + NS < nstages;
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      if (m == 2 && more) {
        // this wave has the whole of stage s in registers, and its loads of stage s + 1 have landed
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (STEADY) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * L::LPW) : "memory");
        else wait_loads(min(nstages - 2 - s, NS - 2));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      }
      if (m >= 2 && m < 8 && more) { read_one(o0, st_next, 0, 2 * m - 4); read_one(o0, st_next, 0, 2 * m - 3); }
      if (m >= 8 && refill) issue_one(m - 8);
      product(o1, m);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  int s = 0;
  for (; s + NS < nstages; ++s) stage(s, std::true_type{});
  for (; s < nstages; ++s) stage(s, std::false_type{});

  __syncthreads();                            // every wave is done with the ring
  gemm_store<4, 4>([&](int i, int j) -> const am_f32x16& { return acc[i][j]; }, gsm, wave, n0 + wm * 128, t0 + wn * 128, lane,
                   T, pos, slot, elite_idx, ke_plane, c_plane, plane_rows, n_h, d_h, r, d_c, rope);
}

bool append_gemm_supported(const elitekv_dims& d, int64_t T, int d_ck) {
  if (d.dtype != ELITEKV_BF16 || T <= 64) return false;
  const int NE = 2 * d.r * d.n_heads;
  // 128-column blocks in all, each 64-column half inside one weight matrix
  return (NE + d.d_c) % kGmCols == 0 && NE % 64 == 0 && d.d_c % 64 == 0 && d_ck % 64 == 0 && d.d_model % 8 == 0;
}

template <int WN>
static hipError_t launch_gemm_wn(const AppendArgs& a, hipStream_t stream) {
  using L = GemmLayout<WN>;
  const elitekv_dims& d = a.dims;
  const int N = 2 * d.r * d.n_heads + d.d_c;
  static LdsLimit lds_limit;
  const hipError_t le = raise_lds_limit(lds_limit, reinterpret_cast<const void*>(&append_gemm_kernel<WN>), L::LDS_BYTES);
  if (le != hipSuccess) return le;
  const dim3 grid(N / kGmCols, (unsigned)((a.T + L::BN - 1) / L::BN));
  append_gemm_kernel<WN><<<grid, 256, L::LDS_BYTES, stream>>>(
      (const bf16_t*)a.x, a.pos, a.slot, a.T, (const bf16_t*)a.W_ke, (const bf16_t*)a.W_dkv,
      (const bf16_t*)a.W_dkv2, a.d_ck, a.elite_idx, (bf16_t*)a.ke_plane, (bf16_t*)a.c_plane, a.plane_rows, d.d_model, d.n_heads, d.head_dim, d.r, d.d_c,
      rope_table(d.rope_base, d.head_dim));
  return hipGetLastError();
}

// The XCDs as a grid of xt token groups x 8 / xt column groups, every XCD's tiles in groups of `group` token blocks, all
// columns of a group one after the other: the 32 compute units of an XCD then hold about group x (32 / group) tiles at any
// moment and share their rows and weights through its L2 (with one token block after the other they asked for 32 different
// weight blocks at once, which the Infinity Cache delivers to eight XCDs at 7.5 TB/s).  Fewest rounds first, then no XCD
// without work while others have a quarter more than need be (ten column blocks over eight column groups of two: 512 x 2560
// columns x 8192 tokens, 256 x 256 tiles: 67 -> 44 us a launch), then the fewest distinct blocks.
static GemmTileMap gemm_tile_map(int64_t T, int N, int tokens, int cols) {
  const int64_t tblocks = (T + tokens - 1) / tokens;
  const int cblocks = (N + cols - 1) / cols;
  GemmTileMap best{};
  int64_t best_cost = INT64_MAX, least = INT64_MAX;            // least: tiles of the busiest XCD
  for (int xt = 8; xt >= 1; xt /= 2) least = std::min(least, (tblocks + xt - 1) / xt * ((cblocks + 8 / xt - 1) / (8 / xt)));
  for (int xt = 8; xt >= 1; xt /= 2) {
    GemmTileMap m;
    m.xt = xt;
    m.tb_x = (int)((tblocks + xt - 1) / xt);
    m.cb_x = (cblocks + 8 / xt - 1) / (8 / xt);
    m.group = m.tb_x < 6 ? m.tb_x : 6;
    m.col_blocks = cblocks;
    const int64_t tiles = (int64_t)m.tb_x * m.cb_x, rounds = (tiles + 31) / 32;
    const int at_once = (32 + m.group - 1) / m.group;
    const int64_t cost = rounds * 10000 + (4 * tiles > 5 * least ? 1000 : 0) + m.group + std::min(m.cb_x, at_once);
    if (cost < best_cost) { best = m; best_cost = cost; }
  }
  return best;
}

template <int WN, int NS, int WNW, int CM, int SPB = 1, int KG = 1>
static hipError_t launch_gemm_dma(const AppendArgs& a, hipStream_t stream) {
  using L = GemmDmaLayout<WN, NS, WNW, CM>;
  const elitekv_dims& d = a.dims;
  const int N = 2 * d.r * d.n_heads + d.d_c;
  static LdsLimit lds_limit;
  const hipError_t le = raise_lds_limit(lds_limit, reinterpret_cast<const void*>(&append_gemm_dma_kernel<WN, NS, WNW, CM, SPB, KG>),
                                        L::LDS_BYTES);
  if (le != hipSuccess) return le;
  const GemmTileMap m = gemm_tile_map(a.T, N, L::BN, L::COLS);
  append_gemm_dma_kernel<WN, NS, WNW, CM, SPB, KG><<<8u * m.tb_x * m.cb_x, 64 * CM * WNW, L::LDS_BYTES, stream>>>(
      (const bf16_t*)a.x, a.pos, a.slot, a.T, (const bf16_t*)a.W_ke, (const bf16_t*)a.W_dkv,
      (const bf16_t*)a.W_dkv2, a.d_ck, a.elite_idx, (bf16_t*)a.ke_plane, (bf16_t*)a.c_plane, a.plane_rows,
      d.d_model, d.n_heads, d.head_dim, d.r, d.d_c, rope_table(d.rope_base, d.head_dim),
      a.x_ld ? a.x_ld : (int64_t)d.d_model, a.x_off2, a.d2, m, a.clear, a.n_clear);
  return hipGetLastError();
}

static hipError_t launch_gemm_wide(const AppendArgs& a, hipStream_t stream) {
  constexpr int NS = 5;
  using L = GemmWideLayout<NS>;
  const elitekv_dims& d = a.dims;
  static LdsLimit lds_limit;
  const hipError_t le = raise_lds_limit(lds_limit, reinterpret_cast<const void*>(&append_gemm_wide_kernel<NS>), L::LDS_BYTES);
  if (le != hipSuccess) return le;
  const GemmTileMap m = gemm_tile_map(a.T, 2 * d.r * d.n_heads + d.d_c, 256, 256);
  append_gemm_wide_kernel<NS><<<8u * m.tb_x * m.cb_x, 256, L::LDS_BYTES, stream>>>(
      (const bf16_t*)a.x, a.pos, a.slot, a.T, (const bf16_t*)a.W_ke, (const bf16_t*)a.W_dkv,
      (const bf16_t*)a.W_dkv2, a.d_ck, a.elite_idx, (bf16_t*)a.ke_plane, (bf16_t*)a.c_plane, a.plane_rows,
      d.d_model, d.n_heads, d.head_dim, d.r, d.d_c, rope_table(d.rope_base, d.head_dim),
      a.x_ld ? a.x_ld : (int64_t)d.d_model, a.x_off2, a.d2, m, a.clear, a.n_clear);
  return hipGetLastError();
}

int append_gemm_tile(const AppendArgs& a) {
  const elitekv_dims& d = a.dims;
  const int64_t col_blocks = (2 * d.r * d.n_heads + d.d_c) / kGmCols;
  if (d.d_model % kGdStage)
    return col_blocks * ((a.T + 255) / 256) >= 1024 ? ELITEKV_TILE_STAGED_256_128 : ELITEKV_TILE_STAGED_64_128;
  const int split = 2 * d.r * d.n_heads + a.d_ck;              // first column of W_dkv2
  const int N = 2 * d.r * d.n_heads + d.d_c;
  const double K = a.d2 > d.d_model ? a.d2 : d.d_model;
  // The tile whose rounds of work-groups cost least.  A round's cost in us, fixed part (first stages from cold memory,
  // epilogue) + contraction rows, fitted to measurements of every tile at 64 to 5120 rows, 384 to 9600 columns, 200 to 30000
  // tokens: on the mean 1 % behind the best tile, 10 % with the constants fitted to 768 rows and more only (256 x 4096
  // x 30000 tokens took the third line, 245 us, instead of the first or second, about 165).
  //   tokens x columns     work-groups at once     a round         measured, 1536 x 7680 rows x columns, 1000 / 2048 / 8192 tokens
  //   256 x 256, 4 waves   256                     20.1 + 0.0220 K 53 / 61 / 208 us
  //   256 x 256, 8 waves   256                     15.7 + 0.0245 K 53 / 59 / 210
  //   128 x 128, 8 waves   256                     7.7 + 0.0101 K  43 / 77 / 267
  //   128 x 128, 4 waves   512                     6.7 + 0.0165 K  33 / 60 / 227
  //    64 x 128            512                     6.9 + 0.0113 K  44 / 82 / 306
  //                        256 (alone on its unit) 4.2 + 0.0085 K  43 against 47 us of 128 x 128, 4096 x 1024, 2048 tokens
  // (4096 x 2048: 97 / 113 / 55 / 56 / 59 at 2048 tokens, 468 / 507 / 665 / 583 / 748 at 30000.  A 256 x 128 tile by eight waves,
  // 36 / 63 / 230 above, was nowhere more than 3 % faster than the best of these.  The four waves are chosen only where a
  // unit runs two of their work-groups: alone they are the slower form of 128 x 128.)
  auto cost = [&](int tokens, int cols, int slots, double fixed, double per_row) {
    const GemmTileMap m = gemm_tile_map(a.T, N, tokens, cols);
    const int64_t per_xcd = (int64_t)m.tb_x * m.cb_x;
    if (tokens == 128 && slots == 512 && per_xcd <= 32) return 1e30;
    return (double)((per_xcd + slots / 8 - 1) / (slots / 8)) * (fixed + per_row * K);
  };
  const bool wide_ok = N >= 256 && (a.d2 == 0 || (N % 256 == 0 && split % 256 == 0));
  const double c[5] = {wide_ok ? cost(256, 256, 256, 20.1, .022) : 1e30, wide_ok ? cost(256, 256, 256, 15.7, .0245) : 1e30,
                       cost(128, 128, 256, 7.7, .0101), cost(128, 128, 512, 6.7, .0165),
                       col_blocks * ((a.T + 63) / 64) <= 256 ? cost(64, 128, 256, 4.2, .0085) : cost(64, 128, 512, 6.9, .0113)};
  constexpr int tile[5] = {ELITEKV_TILE_256_256_WIDE, ELITEKV_TILE_256_256, ELITEKV_TILE_128_128, ELITEKV_TILE_128_128_PAIRS,
                           ELITEKV_TILE_64_128};
  int best = 4;                                                // of equal costs the smaller tile
  for (int i = 3; i >= 0; --i)
    if (c[i] < c[best]) best = i;
  return tile[best];
}

hipError_t launch_append_gemm(const AppendArgs& a, hipStream_t stream) {
  const elitekv_dims& d = a.dims;
  if (a.d2 > 0 || a.x_ld > 0) {
    // column slices of wider rows: only the direct-load kernels take them, with whole stages in both slices
    // and no 128-column block across the two matrices
    const int split = 2 * d.r * d.n_heads + a.d_ck;
    if (d.d_model % kGdStage || a.d2 % kGdStage || a.x_off2 % 8 || a.x_ld % 8 || (a.d2 > 0 && split % kGmCols))
      return hipErrorInvalidValue;
  }
  const int tile = append_gemm_tile(a);
  if (a.n_clear > 0 && (tile == ELITEKV_TILE_STAGED_64_128 || tile == ELITEKV_TILE_STAGED_256_128))
    return hipErrorInvalidValue;                               // these do not clear
  switch (tile) {
    case ELITEKV_TILE_256_256_WIDE: return launch_gemm_wide(a, stream);
    case ELITEKV_TILE_256_256: return launch_gemm_dma<4, 4, 2, 4>(a, stream);
    case ELITEKV_TILE_128_128: return launch_gemm_dma<1, 6, 4, 2, 2, 2>(a, stream);
    case ELITEKV_TILE_128_128_PAIRS: return launch_gemm_dma<2, 4, 2, 2>(a, stream);
    case ELITEKV_TILE_64_128: return launch_gemm_dma<1, 6, 2, 2>(a, stream);
    case ELITEKV_TILE_STAGED_256_128: return launch_gemm_wn<4>(a, stream);
    default: return launch_gemm_wn<1>(a, stream);
  }
}

}  // namespace ekv
