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
// All state (packed copies, residuals, partial distances, elite masks) lives in the caller's workspace; a search is
// 1 + r launches on the caller's stream with no host synchronisation in between.
#include <algorithm>

#include "common.hpp"
#include "launch.hpp"

namespace ekv {

constexpr int kSrTile = 16;      // queries (and keys) per tile
constexpr int kSrMaxChunks = 64; // head_dim <= 128; the packed rows always hold 64 chunks (zeros beyond d_h / 2)
constexpr int kSrRow = 4 * kSrMaxChunks;   // floats per (token, head) of a packed operand

typedef __attribute__((ext_vector_type(4))) float sr_f32x4;

// Operand order: the four rows x 64 chunks of the 16 tokens of a tile (tiles start at multiples of 16) lie as
// [quad of chunks c4 (16)][lane (64)][4 chunks], lane = 16 * row + token % 16: one 16-byte load per lane and
// instruction, 1 KiB contiguous per wave instruction, 16 instructions per operand.  Tokens beyond T are zeros.

// Work-group = (tile of 16 tokens, kSrPackHeads heads): the tile's 16 x 64 rotations are formed once for all of its heads;
// a thread holds four chunks of one token, so every store is 16 bytes and 16 tokens' stores are contiguous.  A thread per
// (token, head, chunk), with its own rotation and eight 4-byte stores, took 40 us for 1000 tokens of 32 heads; this 25.
constexpr int kSrPackHeads = 4;
__global__ __launch_bounds__(256) void search_pack_kernel(const float* __restrict__ q, const float* __restrict__ k,
                                                          const int32_t* __restrict__ pos, float* __restrict__ qp,
                                                          float* __restrict__ kp, uint64_t* __restrict__ emask,
                                                          int32_t* __restrict__ arrived, int64_t T, int n_h, int d_h,
                                                          float scale, RopeTable rope) {
  __shared__ float2 turn[kSrMaxChunks][kSrTile + 1];
  const int tid = threadIdx.x, half = d_h / 2;
  const int64_t tile = blockIdx.x;
  const int h0 = blockIdx.y * kSrPackHeads;
  for (int e = tid; e < kSrTile * kSrMaxChunks; e += 256) {
    const int t = e % kSrTile, i = e / kSrTile;
    float sn = 0.f, cs = 1.f;
    if (i < half && tile * kSrTile + t < T) rope_sincos(pos[tile * kSrTile + t], rope.theta[i], &sn, &cs);
    turn[i][t] = make_float2(sn, cs);
  }
  if (tile == 0 && tid < kSrPackHeads && h0 + tid < n_h) {     // the heads' state, before the first round
    emask[h0 + tid] = 0ull;
    arrived[h0 + tid] = 0;
  }
  __syncthreads();
  const int t = tid % kSrTile, c4 = tid / kSrTile;
  const int64_t token = tile * kSrTile + t;
  for (int h = h0; h < min(h0 + kSrPackHeads, n_h); ++h) {
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
    const int64_t o = ((tile * n_h + h) * (kSrMaxChunks / 4) + c4) * 64 + t;      // 16-byte units
#pragma unroll
    for (int row = 0; row < 4; ++row) {
      reinterpret_cast<sr_f32x4*>(qp)[o + 16 * row] = qo[row];
      reinterpret_cast<sr_f32x4*>(kp)[o + 16 * row] = ko[row];
    }
  }
}

// Key tiles per work-group (a power of two, at least one per wave) and the work-groups ("items") per head: 32-query block Q
// has 2 Q + 2 key tiles, cut into pieces of that many.  A search's launches have about a thousand work-groups (two to four
// rounds of the chip: 512 / 1024 / 2048 / 4096 wanted: 1103 / 1060 / 1145 / 1233 us (before the products were grouped) at 1000 tokens of 32 heads, 205 / 235 /
// 235 / 235 at 300), and a head at most about a thousand or one per 32-query block, since one work-group adds up their
// distances (a piece of 2 n_q32 tiles is a whole block: nothing is gained by longer ones).
inline int sr_keys_per_item(int64_t n_q32, int64_t n_h) {
  int k = 4;
  while (k < 2 * n_q32 && (n_q32 * n_q32 / k > 1024 || n_h * n_q32 * n_q32 / k > 1024)) k *= 2;
  return k;
}
inline int64_t sr_items_before(int q32, int keys) {      // items of the 32-query blocks below q32
  const int64_t per = keys / 2, g = q32 / per;
  return per * g * (g + 1) / 2 + (q32 % per) * (g + 1);
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

// grid (heads, items), four waves; item = (32 queries, up to `keys` key tiles), the key tiles dealt to the waves round-robin.
// A wave holds the key operand B of a tile in registers and uses it for both query tiles (their operands in LDS):
//   residual  LOAD: what the last round left, less the chunk it chose; else the sum over the chunks outside E
//   distances one matrix instruction and four additions of absolute values per chunk
// (lane l of a result tile holds queries 4 (l / 16) + v, v < 4, against key l % 16).  Chunks in E are computed like the
// others and ignored by the choice.  Bound by the fp32 matrix cores: 64 instructions of 32 cycles per tile of 256 pairs.
// Before (the residual summed again in every round, subtraction and weights on the vector units, 16 queries per
// work-group) a round of 1000 tokens, 32 heads took 302 us and a launch of 6 us for the choice; now 127.
// The product and the additions of its four absolute values do not overlap on a SIMD (measured apart: 13.9 ns a product,
// 2 ns an addition, 25 ns for one product and four additions), which leaves 60 % of the measured time for the instructions.
template <bool LOAD, bool FUSED>
__global__ __launch_bounds__(256, 2) void search_round_kernel(
    const float* __restrict__ qp, const float* __restrict__ kp, float* __restrict__ res, uint64_t* __restrict__ emask,
    int32_t* __restrict__ arrived, float* __restrict__ partial, int32_t* __restrict__ elite_out,
    float* __restrict__ dist_out, int n_h, int n_tiles, int keys, int half, int r, int round,
    bool keep) {
  __shared__ sr_f32x4 As[2][kSrMaxChunks / 4][64];
  __shared__ float red[4][kSrMaxChunks];
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
  // the last work-group of the head to arrive makes the choice (device-scope stores, acknowledged before the count)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    last = __hip_atomic_fetch_add(arrived + h, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_items - 1;
    if (last) __hip_atomic_store(arrived + h, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (!last) return;
  float d = 0.f;
#pragma unroll 16
  for (int i = wave; i < n_items; i += 4)
    d += __hip_atomic_load(partial + ((int64_t)h * n_items + i) * kSrMaxChunks + lane, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
  red[wave][lane] = d;
  __syncthreads();
  if (wave != 0) return;
  d = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
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

// Samples of up to this many tokens keep the residuals where the caller's workspace has room for them (n_h (T / 16)^2 / 2
// KiB: 66 MB for 1000 tokens of 32 heads, 1.1 GB for 4096) and the size function asks for that room up to this many bytes.
// The other searches sum the residuals again in every round, at twice the matrix instructions (32 heads, r = 8, 128 / 1000 / 4096
// tokens: 0.128 / 1.56 / 20.9 ms instead of 0.108 / 1.07 / 14.3).
constexpr int64_t kSrKeepTokens = 4096;
constexpr size_t kSrKeepBytes = (size_t)4 << 30;

// least: bytes a search needs, which never falls as T grows (the pieces per head do, wherever a piece gets longer: the
// partial distances are laid out for the most that a shorter sample has); total: with the residuals, if they are kept
struct SearchLayout { size_t kp, partial, emask, arrived, res, least, total; int n_tiles, keys, n_items; };
static SearchLayout search_layout(int64_t T, int n_h) {
  SearchLayout L;
  L.n_tiles = (int)((T + kSrTile - 1) / kSrTile);
  const int n_q32 = (L.n_tiles + 1) / 2;
  L.keys = sr_keys_per_item(n_q32, n_h);
  L.n_items = (int)sr_items_before(n_q32, L.keys);
  auto up = [](size_t v) { return (v + 255) / 256 * 256; };
  const size_t vec = up((size_t)L.n_tiles * kSrTile * n_h * kSrRow * sizeof(float));      // one packed operand (whole tiles)
  L.kp = vec;
  L.partial = L.kp + vec;
  const int64_t most_items = std::min<int64_t>(sr_items_before(n_q32, 4), 1024 + n_q32);
  L.emask = L.partial + up((size_t)n_h * most_items * kSrMaxChunks * sizeof(float));
  L.arrived = L.emask + up((size_t)n_h * sizeof(uint64_t));
  L.res = L.arrived + up((size_t)n_h * sizeof(int32_t));
  L.least = L.total = L.res;
  const size_t kept = (size_t)L.n_tiles * (L.n_tiles + 1) / 2 * n_h * 1024;
  if (T <= kSrKeepTokens && kept <= kSrKeepBytes) L.total += kept;
  return L;
}

size_t search_workspace_bytes(int64_t T, int n_h) { return search_layout(T, n_h).total; }
size_t search_min_workspace_bytes(int64_t T, int n_h) { return search_layout(T, n_h).least; }

hipError_t launch_ropelite_search(const float* q, const float* k, const int32_t* pos, int64_t T, int n_h, int d_h,
                                  int r, double rope_base, int32_t* elite_out, float* dist_out, char* ws,
                                  size_t ws_bytes, hipStream_t stream) {
  const SearchLayout L = search_layout(T, n_h);
  float* qp = (float*)ws;
  float* kp = (float*)(ws + L.kp);
  float* partial = (float*)(ws + L.partial);
  uint64_t* emask = (uint64_t*)(ws + L.emask);
  int32_t* arrived = (int32_t*)(ws + L.arrived);
  float* res = L.total > L.least && ws_bytes >= L.total ? (float*)(ws + L.res) : nullptr;
  const int half = d_h / 2;
  const float scale = 1.f / sqrtf((float)d_h);
  search_pack_kernel<<<dim3(L.n_tiles, (n_h + kSrPackHeads - 1) / kSrPackHeads), 256, 0, stream>>>(
      q, k, pos, qp, kp, emask, arrived, T, n_h, d_h, scale, rope_table(rope_base, d_h));
  const dim3 grid(n_h, L.n_items);
  // A residual carries the rounding errors of the full sum along, while it shrinks as chunks leave it: once more than a
  // quarter of the chunks are chosen it is summed afresh and the products are rounded before they are taken off it, so
  // that the last chunk's distance vanishes exactly.
  for (int round = 0; round < r; ++round) {
    const bool early = 4 * round <= half, keep = res && 4 * (round + 1) <= half && round + 1 < r;
    auto kernel = !early           ? search_round_kernel<false, false>
                  : round && res   ? search_round_kernel<true, true>
                                   : search_round_kernel<false, true>;
    kernel<<<grid, 256, 0, stream>>>(qp, kp, res, emask, arrived, partial, elite_out, dist_out, n_h, L.n_tiles, L.keys, half,
                                     r, round, keep);
  }
  return hipGetLastError();
}

}  // namespace ekv
