// Decode and append kernels in fp32 arithmetic with the whole chip in use: the fp32 dtype, and bf16 shapes whose widths
// the bf16 kernels are not compiled for, as long as the widths are multiples of 16 (decode_tiled_supported,
// append_tiled_supported).  The attention's products run on the fp32 matrix cores; the others, bound by their bytes, on the
// vector units.  Sums are fp32 throughout, products exact fp32 fused multiply-adds.
//
// The path of the remaining shapes (decode_generic.hip, append_generic.hip) gives a work-group one head or 256 columns
// and walks the whole contraction serially: 64 work-groups on 256 compute units, one load in flight per lane.
// Measured at 7B 25 %, fp32, two sequences of 1000 tokens (us): append 554, query 44, attention 190, merge 291.
#include "common.hpp"
#include "launch.hpp"

namespace ekv {

typedef __attribute__((ext_vector_type(4))) float tf_f32x4;

__device__ __forceinline__ tf_f32x4 ld4(const float* p) { return *reinterpret_cast<const tf_f32x4*>(p); }
__device__ __forceinline__ tf_f32x4 ld4(const bf16_t* p) {
  const uint2 v = *reinterpret_cast<const uint2*>(p);
  tf_f32x4 r;
  r[0] = __uint_as_float(v.x << 16); r[1] = __uint_as_float(v.x & 0xffff0000u);
  r[2] = __uint_as_float(v.y << 16); r[3] = __uint_as_float(v.y & 0xffff0000u);
  return r;
}

// ---- append: Y = X [W_ke | W_dkv | W_dkv2], rotated and stored ----
// A work-group owns 16 columns and the whole contraction for TT tokens: 256 groups of four lanes, a group takes every
// 256th block of four weight rows (64 bytes of each), so that all of the weights are in flight at once and no partial
// sums leave the work-group.  Bound by the weights' bytes.  
// Two tokens, 4096 x 2048 weights from HBM: 18.7 us (1.8 TB/s; append_generic_kernel 554).
constexpr int kTaThreads = 1024, kTaCols = 16;

template <typename T, int TT>
__device__ __forceinline__ void append_tiled_body(
    int slice, int n_slices, int64_t t0, const T* __restrict__ x, const int32_t* __restrict__ pos,
    const int64_t* __restrict__ slot, int64_t T_tokens, const T* __restrict__ W_ke, const T* __restrict__ W_dkv,
    const T* __restrict__ W_dkv2, int d_ck, const int32_t* __restrict__ elite_idx, T* __restrict__ ke_plane,
    T* __restrict__ c_plane, int64_t plane_rows, int d, int n_h, int d_h, int r, int d_c, const RopeTable& rope) {
  __shared__ float red[kTaThreads / 64][TT][kTaCols];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int NE = 2 * r * n_h;
  // neighbouring slices share 128-byte lines of the weights: both on one XCD (linear index modulo 8) where they pair up
  if ((n_slices & 15) == 0) slice = 2 * (8 * (slice >> 4) + (slice & 7)) + ((slice >> 3) & 1);
  const int n0 = slice * kTaCols;
  const T* w;
  int64_t wstride;
  weight_column(n0, NE, d_ck, d_c, W_ke, W_dkv, W_dkv2, &w, &wstride);
  w += (lane & 3) * 4;

  tf_f32x4 acc[TT];
#pragma unroll
  for (int t = 0; t < TT; ++t) acc[t] = (tf_f32x4)(0.f);
#pragma unroll 4
  for (int k = (tid >> 2) * 4; k < d; k += kTaThreads) {
    tf_f32x4 wr[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) wr[u] = ld4(w + (int64_t)(k + u) * wstride);
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      const int64_t tok = min(t0 + t, T_tokens - 1);     // tokens past the end repeat the last one and are not stored
      const tf_f32x4 xv = ld4(x + tok * d + k);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[t][e] = fmaf(xv[u], wr[u][e], acc[t][e]);
    }
  }
#pragma unroll
  for (int t = 0; t < TT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float v = acc[t][e];
#pragma unroll
      for (int o = 32; o >= 4; o >>= 1) v += __shfl_xor(v, o, kWave);
      if (lane < 4) red[wave][t][lane * 4 + e] = v;
    }
  __syncthreads();
  if (tid >= TT * kTaCols) return;
  const int t = tid / kTaCols, col = tid % kTaCols, n = n0 + col;
  float mine = 0.f;
#pragma unroll
  for (int g = 0; g < kTaThreads / 64; ++g) mine += red[g][t][col];
  const float other = __shfl_xor(mine, 1, kWave);        // the other element of the elite pair
  const int64_t tok = t0 + t;
  if (tok >= T_tokens) return;
  const int64_t row = slot[tok];
  if (row < 0 || row >= plane_rows) return;
  if (n < NE) {
    int chunk = elite_idx[(n / (2 * r)) * r + ((n % (2 * r)) >> 1)];
    chunk = min(max(chunk, 0), d_h / 2 - 1);
    float s, c;
    rope_sincos(pos[tok], rope.theta[chunk], &s, &c);
    st(ke_plane, row * NE + n, (n & 1) ? (other * s + mine * c) : (mine * c - other * s));
  } else {
    st(c_plane, row * d_c + (n - NE), mine);
  }
}

template <typename T, int TT>
__global__ __launch_bounds__(kTaThreads) void append_tiled_kernel(
    const T* __restrict__ x, const int32_t* __restrict__ pos, const int64_t* __restrict__ slot, int64_t T_tokens,
    const T* __restrict__ W_ke, const T* __restrict__ W_dkv, const T* __restrict__ W_dkv2, int d_ck,
    const int32_t* __restrict__ elite_idx, T* __restrict__ ke_plane, T* __restrict__ c_plane, int64_t plane_rows,
    int d, int n_h, int d_h, int r, int d_c, RopeTable rope) {
  append_tiled_body<T, TT>(blockIdx.x, gridDim.x, (int64_t)blockIdx.y * TT, x, pos, slot, T_tokens, W_ke, W_dkv, W_dkv2, d_ck,
                           elite_idx, ke_plane, c_plane, plane_rows, d, n_h, d_h, r, d_c, rope);
}

// Up to kTaMaxTokens tokens, and where it costs less than append_generic_kernel.  Every tile of eight tokens reads the
// weights again and a work-group has a start of its own, so the cost goes with the work-groups; the serial kernel's goes
// with the contraction rows, and doubles where the token tiles read more weights than the L2s hold.  Fitted, us, to 32 to
// 4096 rows x 32 to 4144 columns x 1 to 256 tokens in both types: never more than a tenth or two us behind the faster one.
// This kernel / append_generic_kernel, fp32:
//   rows x columns    1 token     8 tokens    64 tokens    256 tokens
//     64 x 2512       8.3 / 8.8   10 / 10      41 / 10     150 / 10
//    512 x 1520       8 / 30      10 / 33      26 / 34      96 / 34
//   1024 x 2512       8 / 56      12 / 60      56 / 111    198 / 109
//   4096 x 2048       14 / 400    18 / 430     64 / 425    244 / 420
constexpr int64_t kTaMaxTokens = 256;
static bool append_tiled_pays(const elitekv_dims& d, int64_t T) {
  const double rows = d.d_model;
  const int64_t N = 2 * (int64_t)d.r * d.n_heads + d.d_c, groups = N / kTaCols * ((T + 7) / 8);
  const int64_t at_once = T <= 4 ? 512 : 256;
  const int64_t bytes = N * d.d_model * (d.dtype == ELITEKV_FP32 ? 4 : 2), tiles8 = T < 64 ? T : 64;
  return (groups + at_once - 1) / at_once * (7. + .003 * rows) <= 3. + (bytes * tiles8 > 64LL * (4 << 20) ? .105 : .06) * rows;
}
static bool append_tiled_covers(const elitekv_dims& d, int d_ck) {
  return d.d_model % 4 == 0 && (2 * d.r * d.n_heads) % kTaCols == 0 && d_ck % kTaCols == 0 && (d.d_c - d_ck) % kTaCols == 0;
}
bool append_tiled_supported(const elitekv_dims& d, int64_t T, int d_ck) {
  return T <= kTaMaxTokens && append_tiled_covers(d, d_ck) && append_tiled_pays(d, T);
}

template <typename T>
static void launch_append_tiled_t(const AppendArgs& a, hipStream_t stream) {
  const elitekv_dims& d = a.dims;
  const int slices = (2 * d.r * d.n_heads + d.d_c) / kTaCols;
#define EKV_APPEND(TT)                                                                                               \
  append_tiled_kernel<T, TT><<<dim3(slices, (unsigned)((a.T + TT - 1) / TT)), kTaThreads, 0, stream>>>(              \
      (const T*)a.x, a.pos, a.slot, a.T, (const T*)a.W_ke, (const T*)a.W_dkv, (const T*)a.W_dkv2, a.d_ck, a.elite_idx, \
      (T*)a.ke_plane, (T*)a.c_plane, a.plane_rows, d.d_model, d.n_heads, d.head_dim, d.r, d.d_c,                     \
      rope_table(d.rope_base, d.head_dim))
  if (a.T == 1) EKV_APPEND(1);
  else if (a.T == 2) EKV_APPEND(2);
  else if (a.T <= 4) EKV_APPEND(4);
  else EKV_APPEND(8);
#undef EKV_APPEND
}

hipError_t launch_append_tiled(const AppendArgs& a, hipStream_t stream) {
  if (a.dims.dtype == ELITEKV_FP32) launch_append_tiled_t<float>(a, stream);
  else launch_append_tiled_t<bf16_t>(a, stream);
  return hipGetLastError();
}

// ---- query preparation ----
// Work-group = (NT / 4 latent columns, head, up to BT query rows): eight lanes read one W_uk row of the head together
// (16 bytes each), so W_uk is read once per BT rows; bound by its bytes.  
// Two rows, 7B 25 %: 10.8 us for 22 MB (qprep_generic_kernel 44.5).
template <typename T, int BT, int NT>
__device__ __forceinline__ void qprep_tiled_body(int kb, int h, int b0, const T* __restrict__ q,
                                                 const int32_t* __restrict__ q_pos, const T* __restrict__ W_uk,
                                                 const int32_t* __restrict__ elite_idx, float* __restrict__ qe,
                                                 float* __restrict__ qt, int B, int n_h, int d_h, int r, int d_q,
                                                 const RopeTable& rope, float scale_log2e) {
  __shared__ __align__(16) float q_ne[BT][256];     // d_h <= 256 checked on the host
  __shared__ unsigned long long elite[2];
  const int tid = threadIdx.x;
  const int nd = d_h - 2 * r, half = d_h / 2;
  if (tid < 2) elite[tid] = 0ull;
  for (int e = tid; e < BT * 256; e += NT) q_ne[e >> 8][e & 255] = 0.f;
  __syncthreads();
  for (int j = tid; j < r; j += NT) {
    const int i = elite_idx[h * r + j];
    if (i >= 0 && i < half) atomicOr(&elite[i >> 6], 1ull << (i & 63));
  }
  __syncthreads();
  const unsigned long long e0 = elite[0], e1 = elite[1];
  for (int e = tid; e < BT * half; e += NT) {
    const int bt = e / half, i = e % half;
    if (((i < 64 ? e0 : e1) >> (i & 63)) & 1ull) continue;
    // non-elite chunks keep their order: the chunk's place is the number of non-elite ones before it
    const unsigned long long below = (1ull << (i & 63)) - 1ull;
    const int before = i < 64 ? __popcll(~e0 & below) : __popcll(~e0) + __popcll(~e1 & below);
    if (2 * before + 1 >= nd) continue;             // only if the caller passed repeated indices
    const T* qrow = q + ((int64_t)min(b0 + bt, B - 1) * n_h + h) * d_h;
    q_ne[bt][2 * before] = ld(qrow, 2 * i) * scale_log2e;
    q_ne[bt][2 * before + 1] = ld(qrow, 2 * i + 1) * scale_log2e;
  }
  if (kb == 0) {
    for (int e = tid; e < BT * r; e += NT) {
      const int b = b0 + e / r, j = e % r;
      if (b >= B) continue;
      int i = elite_idx[h * r + j];
      i = min(max(i, 0), half - 1);
      float s, c;
      rope_sincos(q_pos[b], rope.theta[i], &s, &c);
      const T* qrow = q + ((int64_t)b * n_h + h) * d_h;
      const float u = ld(qrow, 2 * i), v = ld(qrow, 2 * i + 1);
      float* o = qe + ((int64_t)b * n_h + h) * 2 * r;
      o[2 * j] = (u * c - v * s) * scale_log2e;
      o[2 * j + 1] = (u * s + v * c) * scale_log2e;
    }
  }
  __syncthreads();
  const int sub = tid & 7;
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int k = kb * (NT / 4) + p * (NT / 8) + (tid >> 3);
    float acc[BT];
#pragma unroll
    for (int b = 0; b < BT; ++b) acc[b] = 0.f;
    const T* w = W_uk + ((int64_t)min(k, d_q - 1) * n_h + h) * nd;
#pragma unroll 4
    for (int v = sub; v < nd / 4; v += 8) {
      const tf_f32x4 wv = ld4(w + 4 * v);
#pragma unroll
      for (int b = 0; b < BT; ++b) {
        const tf_f32x4 qv = ld4(&q_ne[b][4 * v]);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[b] = fmaf(qv[e], wv[e], acc[b]);
      }
    }
#pragma unroll
    for (int b = 0; b < BT; ++b) {
      float a = acc[b];
      a += __shfl_xor(a, 1, kWave);
      a += __shfl_xor(a, 2, kWave);
      a += __shfl_xor(a, 4, kWave);
      if (sub == 0 && k < d_q && b0 + b < B) qt[((int64_t)(b0 + b) * n_h + h) * d_q + k] = a;
    }
  }
}

template <typename T, int BT>
__global__ __launch_bounds__(256) void qprep_tiled_kernel(const T* __restrict__ q, const int32_t* __restrict__ q_pos,
                                                          const T* __restrict__ W_uk,
                                                          const int32_t* __restrict__ elite_idx, float* __restrict__ qe,
                                                          float* __restrict__ qt, int B, int n_h, int d_h, int r, int d_q,
                                                          RopeTable rope, float scale_log2e) {
  qprep_tiled_body<T, BT, 256>(blockIdx.x, blockIdx.y, blockIdx.z * BT, q, q_pos, W_uk, elite_idx, qe, qt, B, n_h, d_h, r,
                               d_q, rope, scale_log2e);
}

// The first launch of a decode step of up to eight sequences: append and query preparation do not depend on each other and
// are one grid, the append's work-groups first (both kinds 1024 threads).
// Two sequences, 7B 25 %, fp32: 19.8 us (one after the other 18.7 + 10.8 and a launch gap; the step 66.2 -> 55.9).
struct TiledFrontArgs {
  int64_t plane_rows;
  int B, d, n_h, d_h, r, d_c, d_ck, d_q, n_slices, q_blocks;
  float scale_log2e;
};
template <typename T, int BT>
__global__ __launch_bounds__(kTaThreads) void front_tiled_kernel(
    const T* __restrict__ x, const T* __restrict__ q, const int32_t* __restrict__ pos, const int64_t* __restrict__ slot,
    const T* __restrict__ W_ke, const T* __restrict__ W_dkv, const T* __restrict__ W_dkv2, const T* __restrict__ W_uk,
    const int32_t* __restrict__ elite_idx, T* __restrict__ ke_plane, T* __restrict__ c_plane, float* __restrict__ qe,
    float* __restrict__ qt, TiledFrontArgs A, RopeTable rope) {
  const int wg = blockIdx.x;
  if (wg < A.n_slices) {
    append_tiled_body<T, BT>(wg, A.n_slices, 0, x, pos, slot, A.B, W_ke, W_dkv, W_dkv2, A.d_ck, elite_idx, ke_plane, c_plane,
                             A.plane_rows, A.d, A.n_h, A.d_h, A.r, A.d_c, rope);
  } else {
    const int i = wg - A.n_slices;
    qprep_tiled_body<T, BT, kTaThreads>(i % A.q_blocks, i / A.q_blocks, 0, q, pos, W_uk, elite_idx, qe, qt, A.B, A.n_h,
                                        A.d_h, A.r, A.d_q, rope, A.scale_log2e);
  }
}

// ---- split attention ----
// Work-group (8 waves) = (split, 16 heads, query row).  Per tile of 16 cached tokens every wave takes its slice of CPW
// blocks of 16 latent columns:
//   scores  S[token, head]  += C[token, col] q~[head, col]    v_mfma_f32_16x16x4_f32, A = tile, B = query (registers)
//   values  U^T[col, head]  += C[token, col] P[token, head]   the same instruction, A = the tile read transposed from LDS
// A score tile leaves a lane with one head and four tokens, which is the B operand of the value products as it stands, and
// the accumulators of a lane belong to that same head, so the rescaling is lane-local.  A lane's 16 bytes of a tile (four
// columns of one token) are the A operands of four score instructions: the contraction is taken in the order in which the
// memory has it.  The waves' partial scores are exchanged through LDS (one barrier per tile, two buffers); the elite term,
// whose keys differ from head to head, is added by vector instructions, two tokens per wave.  Bound by the fp32 matrix
// cores (d_c / 2 instructions of 32 cycles per tile and 16 heads) and, at a few tiles per work-group, by the start.
// Two sequences of 1000 tokens, 7B 25 %: 18 us (attn_generic_kernel 190).
constexpr int kTtTok = 16, kTtWaves = 8, kTtKeRegs = 4, kTtComputeUnits = 256;

template <typename T, int CPW>
__global__ __launch_bounds__(kTtWaves * 64) void attn_tiled_kernel(
    const T* __restrict__ ke_plane, const T* __restrict__ c_plane, const float* __restrict__ qe,
    const float* __restrict__ qt, const int32_t* __restrict__ seq_len, float* __restrict__ part_m,
    float* __restrict__ part_l, float* __restrict__ part_u, int n_h, int two_r, int d_c, int d_q, int d_u,
    int64_t max_seq_len, int64_t batch_stride_rows, int64_t plane_rows, int n_splits, int q_per_seq) {
  constexpr int CS = CPW * 16 + 4;                        // row of a wave's slice in LDS: conflict-free both ways
  extern __shared__ __align__(16) float smem[];
  float* cs = smem + (threadIdx.x >> 6) * kTtTok * CS;    // [wave][16 tokens][CS]
  tf_f32x4* sp = reinterpret_cast<tf_f32x4*>(smem + kTtWaves * kTtTok * CS);   // [2][8 waves + elite][64 lanes]
  float* qe_s = smem + kTtWaves * kTtTok * CS + 2 * (kTtWaves + 1) * 64 * 4;   // [16 heads][two_r]

  const int split = blockIdx.x, h0 = blockIdx.y * 16, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i16 = lane & 15, quad = lane >> 4;
  const int head = h0 + i16;
  const int head_ld = min(head, n_h - 1);                 // lanes past the last head repeat it and store nothing

  const int64_t row0 = (int64_t)(b / q_per_seq) * batch_stride_rows;
  int64_t len = seq_len[b];
  len = min(len, max_seq_len);
  len = min(len, plane_rows - row0);
  len = max(len, (int64_t)0);
  const int64_t n_tiles = (len + kTtTok - 1) / kTtTok;

  const int blk0 = wave * CPW, v_blk0 = (d_c - d_u) / 16, q_blks = d_q / 16, n_blks = d_c / 16;
  auto load_tile = [&](int64_t tile, tf_f32x4 (&cv)[CPW]) {
    const int64_t tok = min(tile * kTtTok + i16, len - 1);
    const T* src = c_plane + (row0 + tok) * d_c + blk0 * 16 + quad * 4;
#pragma unroll
    for (int i = 0; i < CPW; ++i) cv[i] = blk0 + i < n_blks ? ld4(src + i * 16) : (tf_f32x4)(0.f);
  };

  tf_f32x4 acc[CPW], cv[CPW], qv[CPW];
#pragma unroll
  for (int i = 0; i < CPW; ++i) acc[i] = (tf_f32x4)(0.f);
  float m = -INFINITY, l = 0.f;
  int64_t tile = split;
  if (tile < n_tiles) {
    load_tile(tile, cv);
    const float* qrow = qt + ((int64_t)b * n_h + head_ld) * d_q + blk0 * 16 + quad * 4;
#pragma unroll
    for (int i = 0; i < CPW; ++i) qv[i] = blk0 + i < q_blks ? ld4(qrow + i * 16) : (tf_f32x4)(0.f);
    for (int e = tid; e < 16 * two_r; e += kTtWaves * 64)
      qe_s[e] = qe[((int64_t)b * n_h + min(h0 + e / two_r, n_h - 1)) * two_r + e % two_r];
  }
  __syncthreads();

  // elite term: this lane's (token, head) pair is token 2 wave + quad / 2, head i16; quad & 1 takes every other 4 values
  const int ke_units = two_r / 4, ke_par = quad & 1, ke_tok = 2 * wave + (quad >> 1);
  int buf = 0;
  for (; tile < n_tiles; tile += n_splits, buf ^= 1) {
    const T* krow = ke_plane + ((row0 + min(tile * kTtTok + ke_tok, len - 1)) * n_h + head_ld) * two_r;
    tf_f32x4 kv[kTtKeRegs];
#pragma unroll
    for (int u = 0; u < kTtKeRegs; ++u)
      kv[u] = 2 * u + ke_par < ke_units ? ld4(krow + (2 * u + ke_par) * 4) : (tf_f32x4)(0.f);

    tf_f32x4 s4[2] = {(tf_f32x4)(0.f), (tf_f32x4)(0.f)};
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
      *reinterpret_cast<tf_f32x4*>(cs + i16 * CS + i * 16 + quad * 4) = cv[i];
      if (blk0 + i < q_blks) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          s4[e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(cv[i][e], qv[i][e], s4[e & 1], 0, 0, 0);
      }
    }
    if (tile + n_splits < n_tiles) load_tile(tile + n_splits, cv);     // in flight until the next tile's scores

    float es = 0.f;
#pragma unroll
    for (int u = 0; u < kTtKeRegs; ++u)
      if (2 * u + ke_par < ke_units) {
        const float* qp = qe_s + i16 * two_r + (2 * u + ke_par) * 4;
#pragma unroll
        for (int e = 0; e < 4; ++e) es = fmaf(kv[u][e], qp[e], es);
      }
    for (int u = kTtKeRegs; 2 * u + ke_par < ke_units; ++u) {          // elite rows of more than 32 values
      const tf_f32x4 kx = ld4(krow + (2 * u + ke_par) * 4);
      const float* qp = qe_s + i16 * two_r + (2 * u + ke_par) * 4;
#pragma unroll
      for (int e = 0; e < 4; ++e) es = fmaf(kx[e], qp[e], es);
    }
    es += __shfl_xor(es, 16, kWave);
    tf_f32x4* spb = sp + buf * (kTtWaves + 1) * 64;
    spb[wave * 64 + lane] = s4[0] + s4[1];
    if (ke_par == 0)
      reinterpret_cast<float*>(spb + kTtWaves * 64 + (ke_tok >> 2) * 16 + i16)[ke_tok & 3] = es;
    __syncthreads();

    tf_f32x4 s = spb[kTtWaves * 64 + lane];
#pragma unroll
    for (int w = 0; w < kTtWaves; ++w) s += spb[w * 64 + lane];
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (tile * kTtTok + quad * 4 + v >= len) s[v] = -INFINITY;
    float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
    mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
    mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
    const float m_new = fmaxf(m, mx);
    const float m_sub = m_new == -INFINITY ? 0.f : m_new;  // nothing visible yet (keys of -inf): weights and sum stay 0
    const float alpha = exp2f(m - m_sub);                  // m = -inf on the first tile gives 0
    tf_f32x4 p;
#pragma unroll
    for (int v = 0; v < 4; ++v) p[v] = exp2f(s[v] - m_sub);
    float ps = (p[0] + p[1]) + (p[2] + p[3]);
    ps += __shfl_xor(ps, 16, kWave);
    ps += __shfl_xor(ps, 32, kWave);
    l = l * alpha + ps;
    m = m_new;
    if (__any(alpha != 1.f)) {
#pragma unroll
      for (int i = 0; i < CPW; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][e] *= alpha;
    }
#pragma unroll
    for (int i = 0; i < CPW; ++i)
      if (blk0 + i >= v_blk0 && blk0 + i < n_blks) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(cs[(quad * 4 + v) * CS + i * 16 + i16], p[v], acc[i], 0, 0, 0);
      }
  }

  if (head >= n_h) return;
  const int64_t pi = ((int64_t)b * n_splits + split) * n_h + head;
  if (wave == 0 && quad == 0) {
    part_m[pi] = m;
    part_l[pi] = l;
  }
  if (l == 0.f) return;                                    // nothing visible: the merge does not read the accumulators
#pragma unroll
  for (int i = 0; i < CPW; ++i)
    if (blk0 + i >= v_blk0 && blk0 + i < n_blks)
      *reinterpret_cast<tf_f32x4*>(part_u + pi * d_u + (blk0 + i - v_blk0) * 16 + quad * 4) = acc[i];
}

// ---- merge of the splits ----
// Work-group = (256 latent columns, head, query row): four groups of 64 lanes take every fourth split, 16 bytes per lane.
// Bound by the split accumulators' bytes where there are many rows, by the trips to memory where there are few: with up to two
// work-groups a compute unit (kTmFewGroups) AHEAD accumulators of every lane are requested before the weights of the splits
// are formed, and one for every one that is used from then on.  A decode step, us, without / with: 1 x 1000 tokens (192
// work-groups, 63 splits) 50.2 / 47.5, 1 x 8000 (128 splits) 81.2 / 75.3, 2 x 1000 (384) 56.1 / 55.3 (little more than two runs differ by), 2 x 3000 at 12.5 % 43.6 /
// 40.5.  With more work-groups the registers cost more than the trips: 4 x 300 (768) 53.4 / 55.0, 64 x 1000 389 / 410.
// 63 splits of two rows, 7B 25 %: 8.1 us for 25 MB (9.3 without AHEAD; merge_upproj_generic_kernel, with the up-projection below, 291).
constexpr int kTmAhead = 16, kTmFewGroups = 2 * kTtComputeUnits;

template <int AHEAD>
__global__ __launch_bounds__(256) void merge_tiled_kernel(const float* __restrict__ part_m,
                                                          const float* __restrict__ part_l, const float* part_u,
                                                          float* ubar, int ubar_rows, int n_h, int d_u, int n_splits) {
  extern __shared__ __align__(16) float smem[];
  tf_f32x4* sums = reinterpret_cast<tf_f32x4*>(smem);      // [4][64]
  float* red = smem + 1024;                                // [8]
  float* w = red + 8;                                      // [n_splits]
  const int h = blockIdx.y, b = blockIdx.z, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t base = (int64_t)b * n_splits * n_h + h;
  const int k = blockIdx.x * 256 + lane * 4;
  // the first 256 maxima and sums, then the first accumulators (what lies in the place of an empty split's is not used)
  float m = -INFINITY, l0 = 0.f;
  if (tid < n_splits) {
    m = part_m[base + (int64_t)tid * n_h];
    l0 = part_l[base + (int64_t)tid * n_h];
  }
  const float m0 = m;
  tf_f32x4 u[AHEAD > 0 ? AHEAD : 1];
  const float* pu = part_u + base * d_u + min(k, d_u - 4);
#pragma unroll
  for (int i = 0; i < AHEAD; ++i)
    if (wave + 4 * i < n_splits) u[i] = ld4(pu + (int64_t)(wave + 4 * i) * n_h * d_u);
  for (int s = tid + 256; s < n_splits; s += 256) m = fmaxf(m, part_m[base + (int64_t)s * n_h]);
  m = wave_max(m);
  if (lane == 0) red[wave] = m;
  __syncthreads();
  m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  float lsum = 0.f;
  for (int s = tid; s < n_splits; s += 256) {
    const float ls = s == tid ? l0 : part_l[base + (int64_t)s * n_h];
    const float ws = ls > 0.f ? exp2f((s == tid ? m0 : part_m[base + (int64_t)s * n_h]) - m) : 0.f;
    w[s] = ws;
    lsum += ws * ls;
  }
  lsum = wave_sum(lsum);
  if (lane == 0) red[4 + wave] = lsum;
  __syncthreads();
  const float L = (red[4] + red[5]) + (red[6] + red[7]);
  tf_f32x4 a = (tf_f32x4)(0.f);
  if constexpr (AHEAD > 0) {
    for (int s0 = wave; s0 < n_splits; s0 += 4 * AHEAD) {
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) {
        const int s = s0 + 4 * i, next = s + 4 * AHEAD;
        if (s < n_splits) {
          const float ws = w[s];
          if (ws != 0.f) {                                 // wave-uniform; an empty split has left no accumulators
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e] = fmaf(ws, u[i][e], a[e]);
          }
        }
        if (next < n_splits) u[i] = ld4(pu + (int64_t)next * n_h * d_u);
      }
    }
  } else if (k < d_u) {
#pragma unroll 8
    for (int s = wave; s < n_splits; s += 4) {
      const float ws = w[s];
      if (ws != 0.f) {
        const tf_f32x4 us = ld4(pu + (int64_t)s * n_h * d_u);
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = fmaf(ws, us[e], a[e]);
      }
    }
  }
  sums[wave * 64 + lane] = a;
  __syncthreads();
  if (wave != 0 || k >= d_u) return;
  const float inv = L > 0.f ? 1.f / L : 0.f;
  a = (sums[lane] + sums[64 + lane]) + (sums[128 + lane] + sums[192 + lane]);
#pragma unroll
  for (int e = 0; e < 4; ++e) a[e] *= inv;
  // (ubar may be the first split's accumulators: this work-group alone reads and writes these columns of the head, and
  // every wave's sums have passed the barrier)
  *reinterpret_cast<tf_f32x4*>(ubar + ((int64_t)b * ubar_rows * n_h + h) * d_u + k) = a;
}

// ---- up-projection o = ubar W_uv ----
// Work-group = (32 output columns of a head, up to BT query rows), the whole contraction: 128 groups of eight lanes, each
// 128 bytes of every 128th row of W_uv, all of them in flight at once.  Bound by the bytes of W_uv.  
// 25 MB in 9.2 us.
constexpr int kTuCols = 32;

template <typename T, int BT>
__global__ __launch_bounds__(1024) void upproj_tiled_kernel(const float* __restrict__ ubar, int ubar_rows,
                                                            const T* __restrict__ W_uv, T* __restrict__ out, int B,
                                                            int n_h, int d_h, int d_u) {
  extern __shared__ __align__(16) float smem[];
  float* us = smem;                                        // [BT][d_u]
  float* red = smem + BT * d_u;                            // [16 waves][BT][kTuCols]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int h = blockIdx.y, j0 = blockIdx.x * kTuCols, b0 = blockIdx.z * BT;
  for (int e = tid; e < BT * d_u / 4; e += 1024) {
    const int bt = e / (d_u / 4), k4 = e % (d_u / 4);
    reinterpret_cast<tf_f32x4*>(us)[e] = ld4(ubar + ((int64_t)min(b0 + bt, B - 1) * ubar_rows * n_h + h) * d_u + 4 * k4);
  }
  __syncthreads();
  tf_f32x4 acc[BT];
#pragma unroll
  for (int b = 0; b < BT; ++b) acc[b] = (tf_f32x4)(0.f);
  const T* w = W_uv + (int64_t)h * d_h + j0 + (lane & 7) * 4;
#pragma unroll 12
  for (int k = tid >> 3; k < d_u; k += 128) {
    const tf_f32x4 wv = ld4(w + (int64_t)k * n_h * d_h);
#pragma unroll
    for (int b = 0; b < BT; ++b) {
      const float u = us[b * d_u + k];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[b][e] = fmaf(u, wv[e], acc[b][e]);
    }
  }
#pragma unroll
  for (int b = 0; b < BT; ++b)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float v = acc[b][e];
#pragma unroll
      for (int o = 32; o >= 8; o >>= 1) v += __shfl_xor(v, o, kWave);
      if (lane < 8) red[(wave * BT + b) * kTuCols + lane * 4 + e] = v;
    }
  __syncthreads();
  if (tid >= BT * kTuCols) return;
  const int bt = tid / kTuCols, col = tid % kTuCols;
  if (b0 + bt >= B) return;
  float a = 0.f;
#pragma unroll
  for (int g = 0; g < 16; ++g) a += red[(g * BT + bt) * kTuCols + col];
  st(out, ((int64_t)(b0 + bt) * n_h + h) * d_h + j0 + col, a);
}

// Widths in whole blocks of 16 columns (a block is a score block, a value block or both), rows of W_uk and elite rows in
// whole 16-byte (fp32) / 8-byte (bf16) pieces, output columns in whole slices; at d_c = 2048 a tile fills the LDS.
// One or two heads of a latent of four blocks leave 14 of the 16 lanes' heads and four of the eight waves without work:
// with long shares of a sequence per work-group, or more rows than compute units, the any-shape kernels are faster.  One
// head, 64 columns, us, this / any-shape: 60 rows of 700 tokens 32.8 / 30.6, 128 of 700 (bf16) 53.5 / 40.3, 300 of 100
// 30.6 / 27.5; 32 of 700 25.8 / 29.8; two heads, 300 of 100 34.6 / 30.2, 128 of 700 52.6 / 61.9; 144 columns: always faster.
bool decode_tiled_supported(const elitekv_dims& d, int d_ck, int64_t rows, int64_t max_seq) {
  const bool narrow = d.d_c <= 64 && d.n_heads <= 2;
  if (narrow && (rows > kTtComputeUnits || (d.n_heads == 1 && rows * ((max_seq + 15) / 16) >= 10 * kTtComputeUnits))) return false;
  return d.d_c % 16 == 0 && d_ck % 16 == 0 && d.d_c <= 2048 && (d.head_dim - 2 * d.r) % 4 == 0 && (2 * d.r) % 4 == 0 &&
         2 * d.r <= 128 && d.head_dim % kTuCols == 0 && d.head_dim <= 256;
}

template <typename T, int CPW>
static hipError_t launch_attn_tiled(const DecodeArgs& a, const DecodePlan& p, const float* qe, const float* qt, float* pm,
                                    float* pl, float* pu, hipStream_t stream) {
  static LdsLimit limit;
  const elitekv_dims& d = a.dims;
  const size_t lds = sizeof(float) * (size_t)(kTtWaves * kTtTok * (CPW * 16 + 4) + 2 * (kTtWaves + 1) * 256 + 32 * d.r);
  const hipError_t e = raise_lds_limit(limit, (const void*)attn_tiled_kernel<T, CPW>, lds);
  if (e != hipSuccess) return e;
  attn_tiled_kernel<T, CPW><<<dim3(p.n_splits, (d.n_heads + 15) / 16, (unsigned)a.B), kTtWaves * 64, lds, stream>>>(
      (const T*)a.ke_plane, (const T*)a.c_plane, qe, qt, a.seq_len, pm, pl, pu, d.n_heads, 2 * d.r, d.d_c, p.d_q, p.d_u,
      a.max_seq_len, a.batch_stride_rows, a.plane_rows, p.n_splits, a.q_per_seq);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_decode_tiled_t(const DecodeArgs& a, const DecodePlan& p, hipStream_t stream) {
  const elitekv_dims& d = a.dims;
  const int n_h = d.n_heads, d_h = d.head_dim, B = (int)a.B;
  float* qe = (float*)(a.ws + p.off_qe);
  float* qt = (float*)(a.ws + p.off_qt);
  float* pm = (float*)(a.ws + p.off_m);
  float* pl = (float*)(a.ws + p.off_l);
  float* pu = (float*)(a.ws + p.off_u);
  float* ubar = (float*)(a.ws + p.off_opart);
  hipError_t e = hipSuccess;
  if (a.stages & 1) {
#define EKV_QPREP(BT)                                                                                               \
  qprep_tiled_kernel<T, BT><<<dim3((p.d_q + 63) / 64, n_h, (B + BT - 1) / BT), 256, 0, stream>>>(      \
      (const T*)a.q, a.q_pos, (const T*)a.W_uk, a.elite_idx, qe, qt, B, n_h, d_h, d.r, p.d_q,                       \
      rope_table(d.rope_base, d_h), kLog2e / sqrtf((float)d_h))
    if (B == 1) EKV_QPREP(1);
    else if (B == 2) EKV_QPREP(2);
    else EKV_QPREP(4);
#undef EKV_QPREP
  }
  if (a.stages & 2) {
    const int cpw = (d.d_c / 16 + kTtWaves - 1) / kTtWaves;
#define EKV_ATTN(C) e = launch_attn_tiled<T, C>(a, p, qe, qt, pm, pl, pu, stream)
    if (cpw <= 2) EKV_ATTN(2);
    else if (cpw <= 4) EKV_ATTN(4);
    else if (cpw <= 6) EKV_ATTN(6);
    else if (cpw <= 8) EKV_ATTN(8);
    else if (cpw <= 12) EKV_ATTN(12);
    else EKV_ATTN(16);
#undef EKV_ATTN
    if (e != hipSuccess) return e;
  }
  if (a.stages & 4) {
    const dim3 grid((p.d_u + 255) / 256, n_h, B);
    const auto merge = (int64_t)grid.x * n_h * B <= kTmFewGroups ? merge_tiled_kernel<kTmAhead> : merge_tiled_kernel<0>;
    merge<<<grid, 256, sizeof(float) * (size_t)(1024 + 8 + p.n_splits), stream>>>(pm, pl, pu, ubar, p.ubar_rows, n_h, p.d_u,
                                                                                 p.n_splits);
#define EKV_UP(BT)                                                                                              \
  {                                                                                                             \
    static LdsLimit limit;                                                                                      \
    const size_t lds = sizeof(float) * (size_t)(BT * p.d_u + 16 * BT * kTuCols);                                \
    e = raise_lds_limit(limit, (const void*)upproj_tiled_kernel<T, BT>, lds);                                   \
    if (e != hipSuccess) return e;                                                                              \
    upproj_tiled_kernel<T, BT><<<dim3(d_h / kTuCols, n_h, (B + BT - 1) / BT), 1024, lds, stream>>>(             \
        ubar, p.ubar_rows, (const T*)a.W_uv, (T*)a.out, B, n_h, d_h, p.d_u);                                    \
  }
    if (B == 1) EKV_UP(1)
    else if (B == 2) EKV_UP(2)
    else EKV_UP(4)
#undef EKV_UP
  }
  return hipGetLastError();
}

// (fp32 only: bf16 shapes of this path may have a faster append of their own.  Also where the append alone would be the
// serial kernel's: one launch less is worth more; 64 rows, three sequences of 300 tokens: a step 21.1 us, in two launches 26.5.)
bool front_tiled_supported(const AppendArgs& ap, const DecodeArgs& a, const DecodePlan& p) {
  return p.tiled && a.dims.dtype == ELITEKV_FP32 && a.B <= 8 && append_tiled_covers(a.dims, ap.d_ck);
}

hipError_t launch_front_tiled(const AppendArgs& ap, const DecodeArgs& a, const DecodePlan& p, hipStream_t stream) {
  using T = float;
  const elitekv_dims& d = a.dims;
  TiledFrontArgs A;
  A.plane_rows = ap.plane_rows; A.B = (int)a.B; A.d = d.d_model; A.n_h = d.n_heads; A.d_h = d.head_dim; A.r = d.r;
  A.d_c = d.d_c; A.d_ck = ap.d_ck; A.d_q = p.d_q; A.n_slices = (2 * d.r * d.n_heads + d.d_c) / kTaCols;
  A.q_blocks = (p.d_q + kTaThreads / 4 - 1) / (kTaThreads / 4);
  A.scale_log2e = kLog2e / sqrtf((float)d.head_dim);
#define EKV_FRONT(BT)                                                                                           \
  front_tiled_kernel<T, BT><<<A.n_slices + A.q_blocks * d.n_heads, kTaThreads, 0, stream>>>(                    \
      (const T*)ap.x, (const T*)a.q, a.q_pos, ap.slot, (const T*)ap.W_ke, (const T*)ap.W_dkv,                   \
      (const T*)ap.W_dkv2, (const T*)a.W_uk, a.elite_idx, (T*)ap.ke_plane, (T*)ap.c_plane,                      \
      (float*)(a.ws + p.off_qe), (float*)(a.ws + p.off_qt), A, rope_table(d.rope_base, d.head_dim))
  if (a.B == 1) EKV_FRONT(1);
  else if (a.B == 2) EKV_FRONT(2);
  else if (a.B <= 4) EKV_FRONT(4);
  else EKV_FRONT(8);
#undef EKV_FRONT
  return hipGetLastError();
}

hipError_t launch_decode_tiled(const DecodeArgs& a, const DecodePlan& p, hipStream_t stream) {
  if (a.dims.dtype == ELITEKV_FP32) return launch_decode_tiled_t<float>(a, p, stream);
  return launch_decode_tiled_t<bf16_t>(a, p, stream);
}

}  // namespace ekv
