// RoPElite search (Section 3.1, Algorithm 1): the greedy choice of every head's elite chunks from a
// sample of un-rotated queries and keys of one layer.
//
// With D_i[t, j] = q_{t,i} R((t - j) theta_i) k_{j,i}^T - q_{t,i} k_{j,i}^T (what rotating chunk i adds to
// the score of the causal pair j <= t; Section 3.1 score equation), the scores with elite set E
// differ from the scores of full RoPE by the residual R_E = sum_{i not in E} D_i, and trying chunk c
// as the one addition leaves R_E - D_c.  A round of the algorithm therefore is
//     distance[c] = sum over causal pairs of | R_E[t, j] - D_c[t, j] |   for every c not in E,
// followed by the arg-min (lowest index on ties).  A D_i is recomputed from the fully rotated and
// the un-rotated vectors where it is needed (q^_i . k^_i - q_i . k_i, eq. 1a = 1b); what a round keeps for the next one is
// the residual R_E of every causal pair (one float), from which the next round takes off the chunk that was chosen.
//
//   search_pack   : every token's chunks rotated at its position (angle reduced in double) and laid out as the
//                   operands of the round kernel: per (token, head) four rows of 64 chunk values,
//                   query side (-q^.x, -q^.y, q.x, q.y) / sqrt(d_h), key side (k^.x, k^.y, k.x, k.y),
//                   so that -D_i[t, j] is the 4-term dot product of row-pairs: a rank-4 contraction per chunk
//   search_round  : per (head, 32 queries, range of key tiles): the 64 distances over its causal pairs; R - D_i of a
//                   16 x 16 tile of pairs is one v_mfma_f32_16x16x4_f32 (fp32 in, fp32 out) with the residual as its third
//                   operand.  The last work-group of a head to arrive adds up the head's distances in a fixed order and
//                   takes the arg-min.
//   search_blocks : the same on products of bf16 parts, eight to a term, whose sum is as exact as the fp32 product: 64 x 64 pairs by
//                   a work-group whose waves have a quarter of the chunks each; sb_faster (search_plan.hpp) says which samples take it
// All state (packed copies, residuals, partial distances, elite masks) lives in the caller's workspace; a search is
// 1 + r launches on the caller's stream with no host synchronisation in between.
#include <algorithm>

#include "common.hpp"
#include "launch.hpp"
#include "search_plan.hpp"

namespace ekv {

typedef __attribute__((ext_vector_type(4))) float sr_f32x4;

// Operand order: the four rows x 64 chunks of the 16 tokens of a tile (tiles start at multiples of 16) lie as
// [quad of chunks c4 (16)][lane (64)][4 chunks], lane = 16 * row + token % 16: one 16-byte load per lane and
// instruction, 1 KiB contiguous per wave instruction, 16 instructions per operand.  Tokens beyond T are zeros.

// An fp32 value as the exact sum (from 2^-103 on; of smaller values the last part may be denormal or fall away) of three bf16 parts,
// each rounded to the nearest (ties away from zero; cut off where rounding would leave the range): hm = the first (low half) and
// the second, ll = the third, twice.  Rounded and not cut off: the matrix
// instruction drops the last bits of every product of a group of eight, and the products of parts of one sign would all lose
// in the same direction (measured on normal factors: 6.6e-8 of the sum, against 1e-10 with rounded parts).
struct SrParts { uint32_t hm, ll; };
__device__ __forceinline__ uint32_t sr_top(float x) {
  const uint32_t u = __float_as_uint(x), up = u + 0x8000u;
  return ((u & 0x7f800000u) < 0x7f000000u ? up : u) & 0xffff0000u;
}
__device__ __forceinline__ SrParts sr_parts(float x) {
  const uint32_t h = sr_top(x);
  const float xm = x - __uint_as_float(h);
  const uint32_t m = sr_top(xm);
  const uint32_t l = __float_as_uint(xm - __uint_as_float(m)) & 0xffff0000u;
  return {(h >> 16) | m, (l >> 16) | l};
}

// Work-group = (tile of 16 tokens, `heads` heads): the tile's 16 x 64 rotations are formed once for all of its heads;
// a thread holds four chunks of one token, so every store is 16 bytes and 16 tokens' stores are contiguous.  A thread per
// (token, head, chunk), with its own rotation and eight 4-byte stores, took 40 us for 1000 tokens of 32 heads; this 25.
template <bool SPLIT>
__global__ __launch_bounds__(256) void search_pack_kernel(const float* __restrict__ q, const float* __restrict__ k,
                                                          const int32_t* __restrict__ pos, void* __restrict__ qp,
                                                          void* __restrict__ kp, uint64_t* __restrict__ emask,
                                                          int32_t* __restrict__ arrived, int64_t T, int n_h, int d_h,
                                                          int heads, float scale, RopeTable rope) {
  __shared__ float2 turn[kSrMaxChunks][kSrTile + 1];
  const int tid = threadIdx.x, half = d_h / 2;
  const int64_t tile = blockIdx.x;
  const int h0 = blockIdx.y * heads;
  for (int e = tid; e < kSrTile * kSrMaxChunks; e += 256) {
    const int t = e % kSrTile, i = e / kSrTile;
    float sn = 0.f, cs = 1.f;
    if (i < half && tile * kSrTile + t < T) rope_sincos(pos[tile * kSrTile + t], rope.theta[i], &sn, &cs);
    turn[i][t] = make_float2(sn, cs);
  }
  if (tile == 0 && tid < heads && h0 + tid < n_h) {     // the heads' state, before the first round
    emask[h0 + tid] = 0ull;
    arrived[h0 + tid] = 0;
  }
  __syncthreads();
  const int t = tid % kSrTile, c4 = tid / kSrTile;
  const int64_t token = tile * kSrTile + t;
  for (int h = h0; h < min(h0 + heads, n_h); ++h) {
    sr_f32x4 qo[4], ko[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = 4 * c4 + e;
      float qu = 0.f, qv = 0.f, ku = 0.f, kv = 0.f;
      if (i < half && token < T) {
        const int64_t o = (token * n_h + h) * d_h + 2 * i;
        qu = q[o] * scale; qv = q[o + 1] * scale; ku = k[o]; kv = k[o + 1];
      }
      const float2 r = turn[i][t];
      qo[0][e] = -(qu * r.y - qv * r.x);
      qo[1][e] = -(qu * r.x + qv * r.y);
      qo[2][e] = qu;
      qo[3][e] = qv;
      ko[0][e] = ku * r.y - kv * r.x;
      ko[1][e] = ku * r.x + kv * r.y;
      ko[2][e] = ku;
      ko[3][e] = kv;
    }
    if constexpr (SPLIT) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int row = 0; row < 4; ++row) {
          const int64_t o = (((int64_t)h * kSrMaxChunks + 4 * c4 + e) * gridDim.x + tile) * 64 + 16 * row + t;
          const SrParts a = sr_parts(qo[row][e]), b = sr_parts(ko[row][e]);
          reinterpret_cast<uint2*>(qp)[o] = make_uint2(a.hm, a.ll);
          reinterpret_cast<uint2*>(kp)[o] = make_uint2(b.ll, b.hm);
        }
      continue;
    }
    const int64_t o = ((tile * n_h + h) * (kSrMaxChunks / 4) + c4) * 64 + t;      // 16-byte units
#pragma unroll
    for (int row = 0; row < 4; ++row) {
      reinterpret_cast<sr_f32x4*>(qp)[o + 16 * row] = qo[row];
      reinterpret_cast<sr_f32x4*>(kp)[o + 16 * row] = ko[row];
    }
  }
}

// acc[c] += sum over the lane's pairs of w |R - D_c| for all chunks: a product per chunk, its absolute sums taken while the
// next four products are on the matrix cores.  PREFETCH: a group's key operand is replaced by the next tile's as soon as
// this (the last) query tile has used it.  FUSED: the residual is the product's third operand; else it is added afterwards.
template <bool FUSED, bool PREFETCH>
__device__ __forceinline__ void sr_distances(const sr_f32x4 (*A)[64], int lane, float (&B)[kSrMaxChunks], const sr_f32x4& R,
                                             const float (&w)[4], float (&acc)[kSrMaxChunks], const sr_f32x4* next) {
  sr_f32x4 D[2][4], a4 = A[0][lane], a4_next = a4;
#pragma unroll
  for (int c4 = 0; c4 <= kSrMaxChunks / 4; ++c4) {
    if (c4 + 1 < kSrMaxChunks / 4) a4_next = A[c4 + 1][lane];
    if (c4 < kSrMaxChunks / 4) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        D[c4 & 1][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a4[u], B[4 * c4 + u], FUSED ? R : (sr_f32x4)(0.f), 0, 0, 0);
    }
    // the order as written: left alone, the compiler sinks the additions behind the next branch, with 64 products kept
    __builtin_amdgcn_sched_barrier(0);
    if (c4 > 0) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          float& a = acc[4 * c4 - 4 + u];
          a = fmaf(w[v], fabsf(FUSED ? D[(c4 - 1) & 1][u][v] : R[v] + D[(c4 - 1) & 1][u][v]), a);
          if (v == 3) asm volatile("" : "+v"(a));
        }
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (PREFETCH) {
      if (c4 < kSrMaxChunks / 4) {
        const sr_f32x4 x = next[c4 * 64];
#pragma unroll
        for (int u = 0; u < 4; ++u) B[4 * c4 + u] = x[u];
      }
    }
    a4 = a4_next;
  }
}

// The end of a round: the last work-group of the head to arrive (device-scope stores, acknowledged before the count) adds up the
// head's distances in a fixed order and takes the arg-min.  red: 2 KiB of LDS.
__device__ __forceinline__ void sr_choose(float* red, int* last, uint64_t* emask, int32_t* arrived, const float* partial,
                                          int32_t* elite_out, float* dist_out, int h, int n_items, int half, int r, int round,
                                          uint64_t elite) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    *last = __hip_atomic_fetch_add(arrived + h, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_items - 1;
    if (*last) __hip_atomic_store(arrived + h, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (!*last) return;
  // in 64 bits: thirty-four sums of a wave, one after the other (136 blocks of 1000 tokens), lost 4e-8 of the distance in 32
  double sum = 0.0;
#pragma unroll 16
  for (int i = wave; i < n_items; i += 4)
    sum += __hip_atomic_load(partial + ((int64_t)h * n_items + i) * kSrMaxChunks + lane, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
  double* sums = reinterpret_cast<double*>(red);
  sums[wave * 64 + lane] = sum;
  __syncthreads();
  if (wave != 0) return;
  const float d = (float)((sums[lane] + sums[64 + lane]) + (sums[128 + lane] + sums[192 + lane]));
  const bool cand = lane < half && !((elite >> lane) & 1ull);
  float best = cand ? d : INFINITY;
  int arg = cand ? lane : kSrMaxChunks;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {                 // arg-min, the lowest index wins a tie
    const float ob = __shfl_xor(best, o, kWave);
    const int oa = __shfl_xor(arg, o, kWave);
    if (ob < best || (ob == best && oa < arg)) { best = ob; arg = oa; }
  }
  if (lane == 0) {
    elite_out[h * r + round] = arg;
    if (dist_out) dist_out[h * r + round] = best;
    emask[h] = elite | (1ull << (arg & 63));
  }
}

// grid (heads, items), four waves; item = (32 queries, up to `keys` key tiles), the key tiles dealt to the waves round-robin.
// A wave holds the key operand B of a tile in registers and uses it for both query tiles (their operands in LDS):
//   residual  LOAD: what the last round left, less the chunk it chose; else the sum over the chunks outside E
//   distances one matrix instruction and four additions of absolute values per chunk
// (lane l of a result tile holds queries 4 (l / 16) + v, v < 4, against key l % 16).  Chunks in E are computed like the
// others and ignored by the choice.  Bound by the fp32 matrix cores: 64 instructions of 32 cycles per tile of 256 pairs.
// Before (the residual summed again in every round, subtraction and weights on the vector units, 16 queries per
// work-group) a round of 1000 tokens, 32 heads took 302 us and a launch of 6 us for the choice; now 119 to 130
// (less on a cool chip).
// The product and the additions of its four absolute values do not overlap on a SIMD (measured apart: 13.9 ns a product,
// 2 ns an addition, 25 ns for one product and four additions), which leaves 60 % of the measured time for the instructions.
template <bool LOAD, bool FUSED>
__global__ __launch_bounds__(256, 2) void search_round_kernel(
    const float* __restrict__ qp, const float* __restrict__ kp, float* __restrict__ res, uint64_t* __restrict__ emask,
    int32_t* __restrict__ arrived, float* __restrict__ partial, int32_t* __restrict__ elite_out,
    float* __restrict__ dist_out, int n_h, int n_tiles, int keys, int half, int r, int round,
    bool keep) {
  __shared__ sr_f32x4 As[2][kSrMaxChunks / 4][64];
  __shared__ __attribute__((aligned(8))) float red[8][kSrMaxChunks];   // (twice the waves' sums: also the choice's, in 64 bits)
  __shared__ int last;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i16 = lane & 15, kk = lane >> 4;
  const int h = blockIdx.x, n_items = gridDim.y;
  const int item = n_items - 1 - blockIdx.y;                     // the blocks with the most pieces start first
  // item -> (q32, piece): find the group g of blocks that have g + 1 pieces each
  const int per = keys / 2;
  int g = 0;
  while ((int64_t)per * (g + 1) * (g + 2) / 2 <= item) ++g;
  const int in_group = item - per * g * (g + 1) / 2;
  const int q32 = g * per + in_group / (g + 1), piece = in_group % (g + 1);

  const sr_f32x4* kp4 = reinterpret_cast<const sr_f32x4*>(kp);
  auto key_src = [&](int kt) { return kp4 + (((int64_t)kt * n_h + h) * (kSrMaxChunks / 4)) * 64 + lane; };
  const int kt_end = min(min(2 * q32 + 2, n_tiles), (piece + 1) * keys);
  int kt = piece * keys + wave;
  float B[kSrMaxChunks], acc[kSrMaxChunks];
  if (kt < kt_end) {
    const sr_f32x4* src = key_src(kt);
#pragma unroll
    for (int c4 = 0; c4 < kSrMaxChunks / 4; ++c4) {
      const sr_f32x4 x = src[c4 * 64];
#pragma unroll
      for (int u = 0; u < 4; ++u) B[4 * c4 + u] = x[u];
    }
  }
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int e = u * 256 + tid, qi = e / (64 * kSrMaxChunks / 4), rest = e % (64 * kSrMaxChunks / 4);
    const int qt = min(2 * q32 + qi, n_tiles - 1);               // an odd last tile is read twice, used once
    (&As[0][0][0])[e] = reinterpret_cast<const sr_f32x4*>(qp)[((int64_t)qt * n_h + h) * (64 * kSrMaxChunks / 4) + rest];
  }
#pragma unroll
  for (int c = 0; c < kSrMaxChunks; ++c) acc[c] = 0.f;
  const uint64_t elite = emask[h];
  const int chosen = LOAD ? elite_out[h * r + round - 1] : kSrMaxChunks;
  __syncthreads();

  // -D_c of a (query tile, key tile) added to x, for a chunk known only at run time
  auto less_chunk = [&](int qi, int kt_, int c, const sr_f32x4& x) {
    const float a = reinterpret_cast<const float*>(&As[qi][c >> 2][lane])[c & 3];
    const float b = reinterpret_cast<const float*>(key_src(kt_) + (c >> 2) * 64)[c & 3];
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, x, 0, 0, 0);
  };

  // query tile qi against key tile kt: the residual and its pairs' weights (0 above the diagonal, or where no such tile is)
  auto residual = [&](int qi, int kt_, float (&w)[4]) -> sr_f32x4 {
    const int qt = 2 * q32 + qi;
    const bool there = kt_ <= qt && qt < n_tiles;
#pragma unroll
    for (int v = 0; v < 4; ++v) w[v] = there && (kt_ < qt || i16 <= 4 * kk + v) ? 1.f : 0.f;
    if (!there) return (sr_f32x4)(0.f);
    sr_f32x4* mem = reinterpret_cast<sr_f32x4*>(res) + (((int64_t)qt * (qt + 1) / 2 + kt_) * n_h + h) * 64 + lane;
    sr_f32x4 R;
    if constexpr (LOAD) {
      R = *mem;
      if (chosen >= 0 && chosen < kSrMaxChunks) R = less_chunk(qi, kt_, chosen, R);
    } else {
      sr_f32x4 Rc[4] = {(sr_f32x4)(0.f), (sr_f32x4)(0.f), (sr_f32x4)(0.f), (sr_f32x4)(0.f)};   // -D summed, four chains
#pragma unroll
      for (int c4 = 0; c4 < kSrMaxChunks / 4; ++c4) {
        const sr_f32x4 a4 = As[qi][c4][lane];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (!((elite >> (4 * c4 + u)) & 1ull))
            Rc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a4[u], B[4 * c4 + u], Rc[u], 0, 0, 0);
      }
      R = -((Rc[0] + Rc[1]) + (Rc[2] + Rc[3]));
    }
    if (keep) *mem = R;
    return R;
  };
  for (; kt < kt_end; kt += 4) {
    asm volatile("" ::: "memory");     // the query operands are re-read from LDS for every tile, not kept in registers
    float w[4];
    const sr_f32x4 R0 = residual(0, kt, w);
    sr_distances<FUSED, false>(As[0], lane, B, R0, w, acc, nullptr);
    const sr_f32x4 R1 = residual(1, kt, w);
    sr_distances<FUSED, true>(As[1], lane, B, R1, w, acc, key_src(min(kt + 4, kt_end - 1)));
  }

  // lane c gets the wave's sum of chunk c: at every step a lane keeps half of its chunks and passes on the other half
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
    for (int i = 0; i < o; ++i) {
      const bool up = lane & o;
      const float keep = up ? acc[i + o] : acc[i], pass = up ? acc[i] : acc[i + o];
      acc[i] = keep + __shfl_xor(pass, o, kWave);
    }
  }
  red[wave][lane] = acc[0];
  __syncthreads();
  if (wave == 0)
    __hip_atomic_store(partial + ((int64_t)h * n_items + item) * kSrMaxChunks + lane,
                       (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  sr_choose(&red[0][0], &last, emask, arrived, partial, elite_out, dist_out, h, n_items, half, r, round, elite);
}

// ---- the round on products of bf16 parts -------------------------------------------------------------------------------
//
// A factor of the 4-term product is the exact sum of three bf16 parts (SrParts), and v_mfma_f32_16x16x32_bf16 has room for
// eight products of every term: all pairs of parts but the two last ones' (2^-32 of the term).  A lane holds one term (row) of
// one token: query side {hm, ll, hm, hm}, key side {ll, hm, hm, mh}, of which {hm, ll} and {ll, hm} lie in memory as
// [head][chunk][tile of 16 tokens][lane] (tiles padded to whole blocks, zeros beyond T).

typedef __attribute__((ext_vector_type(8))) __bf16 sr_bf16x8;
typedef __attribute__((ext_vector_type(4))) uint32_t sr_u32x4;

constexpr int kSbChunks = kSrMaxChunks / 4;                 // chunks of a wave
constexpr int kSbLag = 3;                                   // products between a product and the sums of its values

struct SbOperands {
  sr_u32x4 a[kSbTiles], b[kSbTiles];
  __device__ __forceinline__ void load(const uint2* q, const uint2* k) {
#pragma unroll
    for (int i = 0; i < kSbTiles; ++i) {
      const uint2 x = q[i * 64], y = k[i * 64];
      a[i].x = x.x; a[i].y = x.y;
      b[i].x = y.x; b[i].y = y.y;
    }
  }
  __device__ __forceinline__ void expand() {
#pragma unroll
    for (int i = 0; i < kSbTiles; ++i) {
      a[i].z = a[i].x; a[i].w = a[i].x;
      b[i].z = b[i].y; b[i].w = __builtin_amdgcn_alignbit(b[i].y, b[i].y, 16);
    }
  }
  __device__ __forceinline__ sr_f32x4 product(int qi, int ki, const sr_f32x4& c) const {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(sr_bf16x8, a[qi]), __builtin_bit_cast(sr_bf16x8, b[ki]),
                                                   c, 0, 0, 0);
  }
};

// red[c][lane] = the lane's sum over the block's pairs of |R - D_c|, for the wave's chunks c.  DIAG: the block on the
// diagonal: tiles above it are left out, those on it weighted by w (0 above the diagonal).
template <bool DIAG, bool FUSED>
__device__ __forceinline__ void sb_distances(const uint2* q, const uint2* k, int64_t step, const sr_f32x4 (&R)[kSbTiles][kSbTiles],
                                             const float (&w)[4], float* red) {
  constexpr int kPairs = kSbTiles * kSbTiles;
  SbOperands op[2];
  op[0].load(q, k);
  op[0].expand();
#pragma unroll 2
  for (int c = 0; c < kSbChunks; ++c) {
    SbOperands& now = op[c & 1];
    SbOperands& next = op[(c + 1) & 1];
    const int64_t ahead = (c + 1 < kSbChunks ? c + 1 : c) * step;
    next.load(q + ahead, k + ahead);
    float a[4] = {0.f, 0.f, 0.f, 0.f};
    sr_f32x4 D[kSbLag + 1];
#pragma unroll
    for (int i = 0; i < kPairs + kSbLag; ++i) {
      if (i < kPairs) {
        const int qi = i / kSbTiles, ki = i % kSbTiles;
        if (!DIAG || ki <= qi) D[i % (kSbLag + 1)] = now.product(qi, ki, FUSED ? R[qi][ki] : (sr_f32x4)(0.f));
      }
      if (i >= kSbLag) {
        const int j = i - kSbLag, qi = j / kSbTiles, ki = j % kSbTiles;
        if (!DIAG || ki <= qi) {
          const sr_f32x4& d = D[j % (kSbLag + 1)];
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float e = fabsf(FUSED ? d[v] : R[qi][ki][v] + d[v]);
            a[v] = DIAG && ki == qi ? fmaf(w[v], e, a[v]) : a[v] + e;
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    next.expand();
    red[c * 64] = (a[0] + a[1]) + (a[2] + a[3]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// What bounds it: the chip's power.  With every SIMD at work a product of 16 x 16 x 32 bf16 takes 12 ns (16 cycles at the 1.35 GHz
// that are left of 2.4), 18 with its four additions and the operands' copies; the fp32 instruction takes 14, and 25 with the additions,
// for the two do not overlap.  1000 tokens of 32 heads: 75 us of products in a round of 95 to 113
// (search_round_kernel: 119 to 130; both the slower the longer the chip has been at work).  Block size and
// split: a block of 64 x 64 needs half an operand per product and twelve waves of it fit a compute unit; the chunks and not the
// pairs divided among its waves, so that 128 tokens already make 96 work-groups.  Not kept: the queries' operands of all chunks in LDS (1030
// against 900 us a search), both sides through a ring of LDS for 128 x 128 pairs (1325), the work-group's next blocks one after
// the other (two: 940).
// grid n_h x blocks, four waves: a work-group has a block of 64 queries x 64 keys, its waves sixteen chunks each; every wave
// holds the block's residuals in registers:
//   LOAD  what the last round left, less the chunk it chose; else the sum over the chunks outside E, a quarter by each wave
template <bool LOAD, bool FUSED>
__global__ __launch_bounds__(256, 2) void search_blocks_kernel(
    const uint2* __restrict__ qp, const uint2* __restrict__ kp, float* __restrict__ res, uint64_t* __restrict__ emask,
    int32_t* __restrict__ arrived, float* __restrict__ partial, int32_t* __restrict__ elite_out,
    float* __restrict__ dist_out, int n_h, int n_blocks, int half, int r, int round, bool keep) {
  __shared__ __attribute__((aligned(8))) float red[kSrMaxChunks * 64];
  __shared__ sr_f32x4 part[LOAD ? 1 : 4][LOAD ? 1 : 2 * kSbTiles][64];
  __shared__ int last;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, kk = lane >> 4;
  // the blocks of a head on one XCD where the heads can be dealt evenly (their operands in its L2); the lighter ones on the
  // diagonal last
  const int n_items = n_blocks * (n_blocks + 1) / 2, n_full = n_items - n_blocks;
  const int h = n_h % 8 == 0 ? blockIdx.x % 8 + 8 * (blockIdx.x / 8 / n_items) : blockIdx.x % n_h;
  const int item = n_h % 8 == 0 ? blockIdx.x / 8 % n_items : blockIdx.x / n_h;
  int qb = item - n_full, kb = qb;
  if (item < n_full) {
    qb = 1;
    while (qb * (qb + 1) / 2 <= item) ++qb;
    kb = item - qb * (qb - 1) / 2;
  }

  const int64_t step = (int64_t)n_blocks * kSbTiles * 64;        // from chunk to chunk
  const int c0 = wave * kSbChunks;
  const uint2* qt = qp + (int64_t)h * kSrMaxChunks * step + qb * kSbTiles * 64 + lane;
  const uint2* kt = kp + (int64_t)h * kSrMaxChunks * step + kb * kSbTiles * 64 + lane;
  float* mine = red + c0 * 64 + lane;
  float w[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) w[v] = i16 <= 4 * kk + v ? 1.f : 0.f;
  const uint64_t elite = emask[h];
  const int chosen = LOAD ? elite_out[h * r + round - 1] : kSrMaxChunks;

  sr_f32x4* mem = reinterpret_cast<sr_f32x4*>(res) + ((int64_t)h * n_items + item) * kSbTiles * kSbTiles * 64 + lane;
  sr_f32x4 R[kSbTiles][kSbTiles];
  if constexpr (LOAD) {
#pragma unroll
    for (int e = 0; e < kSbTiles * kSbTiles; ++e) R[e / kSbTiles][e % kSbTiles] = mem[e * 64];
    if (chosen >= 0 && chosen < kSrMaxChunks) {
      SbOperands op;
      op.load(qt + chosen * step, kt + chosen * step);
      op.expand();
#pragma unroll
      for (int i = 0; i < kSbTiles; ++i)
#pragma unroll
        for (int j = 0; j < kSbTiles; ++j) R[i][j] = op.product(i, j, R[i][j]);
    }
  } else {
#pragma unroll
    for (int e = 0; e < kSbTiles * kSbTiles; ++e) R[e / kSbTiles][e % kSbTiles] = (sr_f32x4)(0.f);
    SbOperands op[2];
    op[0].load(qt + c0 * step, kt + c0 * step);
#pragma unroll 2
    for (int c = c0; c < c0 + kSbChunks; ++c) {
      SbOperands& now = op[c & 1];
      const int64_t ahead = (c + 1 < c0 + kSbChunks ? c + 1 : c) * step;
      op[(c + 1) & 1].load(qt + ahead, kt + ahead);
      if ((elite >> c) & 1ull) continue;
      now.expand();
#pragma unroll
      for (int i = 0; i < kSbTiles; ++i)
#pragma unroll
        for (int j = 0; j < kSbTiles; ++j) R[i][j] = now.product(i, j, R[i][j]);
    }
    // the waves' sums through LDS, half a block at a time
#pragma unroll
    for (int i0 = 0; i0 < kSbTiles; i0 += 2) {
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 2 * kSbTiles; ++e) part[wave][e][lane] = R[i0 + e / kSbTiles][e % kSbTiles];
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 2 * kSbTiles; ++e)
        R[i0 + e / kSbTiles][e % kSbTiles] = -((part[0][e][lane] + part[1][e][lane]) + (part[2][e][lane] + part[3][e][lane]));
    }
  }
  // waited for here, not wherever they are used below
#pragma unroll
  for (int e = 0; e < kSbTiles * kSbTiles; ++e) asm volatile("" : "+v"(R[e / kSbTiles][e % kSbTiles]));
  if (keep) {
    if constexpr (LOAD) __syncthreads();                         // every wave has read the last round's residuals
#pragma unroll
    for (int e = 0; e < kSbTiles * kSbTiles; ++e)
      if (e / kSbTiles == wave) mem[e * 64] = R[e / kSbTiles][e % kSbTiles];
  }
  if (kb == qb) sb_distances<true, FUSED>(qt + c0 * step, kt + c0 * step, step, R, w, mine);
  else sb_distances<false, FUSED>(qt + c0 * step, kt + c0 * step, step, R, w, mine);

  // four threads to a chunk, sixteen lanes' sums each
  __syncthreads();
  float d = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) d += red[(tid >> 2) * 64 + (tid & 3) * 16 + ((i + (tid >> 2)) & 15)];
  d += __shfl_xor(d, 1, kWave);
  d += __shfl_xor(d, 2, kWave);
  if ((tid & 3) == 0)
    __hip_atomic_store(partial + ((int64_t)h * n_items + item) * kSrMaxChunks + (tid >> 2), d, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  sr_choose(red, &last, emask, arrived, partial, elite_out, dist_out, h, n_items, half, r, round, elite);
}

size_t search_workspace_bytes(int64_t T, int n_h) { return search_layout(T, n_h, 0).total; }
size_t search_min_workspace_bytes(int64_t T, int n_h) { return search_layout(T, n_h, 0).least; }

hipError_t launch_ropelite_search(const float* q, const float* k, const int32_t* pos, int64_t T, int n_h, int d_h,
                                  int r, double rope_base, int32_t* elite_out, float* dist_out, char* ws,
                                  size_t ws_bytes, hipStream_t stream) {
  const SearchLayout L = search_layout(T, n_h, ws_bytes);
  char *qp = ws, *kp = ws + L.kp;
  float* partial = (float*)(ws + L.partial);
  uint64_t* emask = (uint64_t*)(ws + L.emask);
  int32_t* arrived = (int32_t*)(ws + L.arrived);
  float* res = L.blocks || L.keep ? (float*)(ws + L.res) : nullptr;
  const int half = d_h / 2;
  const float scale = 1.f / sqrtf((float)d_h);
  // heads of a work-group: as many as leave a few hundred work-groups, for they share the rotations
  const int heads = std::max<int64_t>(1, std::min<int64_t>(4, (int64_t)L.n_tiles * n_h / 512));
  const dim3 pack_grid(L.n_tiles, (n_h + heads - 1) / heads);
  if (L.blocks)
    search_pack_kernel<true><<<pack_grid, 256, 0, stream>>>(q, k, pos, qp, kp, emask, arrived, T, n_h, d_h, heads, scale,
                                                            rope_table(rope_base, d_h));
  else
    search_pack_kernel<false><<<pack_grid, 256, 0, stream>>>(q, k, pos, qp, kp, emask, arrived, T, n_h, d_h, heads, scale,
                                                             rope_table(rope_base, d_h));
  // A residual carries the rounding errors of the full sum along, while it shrinks as chunks leave it: once more than a
  // quarter of the chunks are chosen it is summed afresh and the products are rounded before they are taken off it, so
  // that the last chunk's distance vanishes exactly.
  for (int round = 0; round < r; ++round) {
    const bool early = 4 * round <= half, keep = res && 4 * (round + 1) <= half && round + 1 < r;
    if (L.blocks) {
      auto kernel = !early  ? search_blocks_kernel<false, false>
                    : round ? search_blocks_kernel<true, true>
                            : search_blocks_kernel<false, true>;
      kernel<<<(unsigned)(n_h * L.n_items), 256, 0, stream>>>((const uint2*)qp, (const uint2*)kp, res, emask, arrived, partial,
                                                              elite_out, dist_out, n_h, L.n_tiles / kSbTiles, half, r, round,
                                                              keep);
    } else {
      auto kernel = !early           ? search_round_kernel<false, false>
                    : round && res   ? search_round_kernel<true, true>
                                     : search_round_kernel<false, true>;
      kernel<<<dim3(n_h, L.n_items), 256, 0, stream>>>((const float*)qp, (const float*)kp, res, emask, arrived, partial, elite_out,
                                                       dist_out, n_h, L.n_tiles, L.keys, half, r, round, keep);
    }
  }
  return hipGetLastError();
}

}  // namespace ekv
