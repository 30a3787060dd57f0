// Attention of MANY queries per sequence over the EliteKV cache (a prefill, a long prompt chunk):
// bf16 on the gfx950 matrix cores, fp32 accumulation.
//
// With one query the cheapest order of the multiplications absorbs B^k into the query and applies
// B^v after the attention sum (Section 5), at 4 d_c flops per (query, cached token, head).  With T
// queries it is cheaper to undo the low-rank compression ONCE per cached token and let every query
// use the result: keys  k_j,h = [ke_j,h (stored rotated, Section 3.1) | c_j B^k_J,h]  and values
// v_j,h = c_j B^v_J,h  (Section 3.2, J-LRD), 2 d_c (2 d_h - 2r) flops per (token, head), then
// ordinary attention (Section 2.1) at 4 d_h flops per (query, token, head).  Three steps:
//
//   1. the matrix-core GEMM of the cache append (launch_append_gemm) run on the latent rows:
//                          KV[j, :] = c_j [B^k_J | B^v_J]   (no elite columns, no rotation)
//   2. prefill_attn_kernel (here; prefill_pairs.hip has another for blocks of few tiles and launches of many of them) flash attention: S^T = K Q^T, online softmax, O^T += V^T P^T, with the
//                          query packed on the way in: q^ = [R(pos theta_i) q_i for i in I_h (slot
//                          order) | q's non-elite dims, ascending], scaled by log2(e)/sqrt(d_h)
//                          (Section 3.1 score equation)
//
// Step 2, one work-group (4 waves, one per SIMD; 131 KB of LDS, so one per compute unit) = 128 or 256 queries of one
// (sequence, head), 32 or 64 per wave; 64-key tiles of K and V come in by direct global->LDS loads into a ring of four.
// Per wave and tile:
//   S^T[key, query]   32x32x16 MFMA, A = key rows from LDS (16-byte reads), B = the wave's queries,
//                     held in registers for the whole pass;
//   softmax           a lane owns ONE query (the MFMA output column) and 16 keys per 32-key block,
//                     its partner lane (l ^ 32) the other 16.  No maximum is taken per tile: the running one stays until
//                     a lane's 16 probabilities add up to more than 2^8 (none of them can then be larger), and only such
//                     a block is formed again with a raised maximum;
//   O^T[dim, query]   32x32x16 MFMA, B = the probabilities straight from the score registers (the
//                     keys of a k-step are taken in the order the score tile leaves them in a lane),
//                     A = V read transposed from LDS (ds_read_b64_tr_b16) in that same key order.
// What bounds it: the matrix cores' power.  The loop alone, on zeros, takes 2800 cycles for the 64 MFMAs (2110 cycles) of 64
// queries per wave; in a launch on all compute units a tile of 256 queries takes 1.9 us = 1120 TFLOP/s, where a library
// product of 8192^3 reaches 1206.  To get there every vector instruction and LDS read stands behind an MFMA of its wave by hand
// (left to the compiler they follow each other), 64 queries per wave halve the LDS reads per MFMA, and the accumulators of
// the values live in AGPRs, the scores in VGPRs.  Before: 1.35 - 1.6 us per tile of 128 queries, from maxima, addresses
// multiplied out per load, and MFMAs that waited for all of it; 7B 25 %, 2048 tokens 74 -> 63 us, 13B, 2 x 1021 over 8000 rows
// 590 - 690 -> 350 - 420.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "prefill_common.hpp"

namespace ekv {

constexpr int kPfRing = 4;                       // stages
constexpr int kPfLds = kPfRing * kPfStage + 64 + 256;   // stages + the block's reduction scratch + the head's chunk order

// Work-groups of a launch (one per compute unit), and the state that a work-group leaves of an unfinished block: (maximum, sum)
// of every query, its accumulators
constexpr int kPfGroups = 256;
constexpr size_t kPfPartBytes = (size_t)256 * 16 * (2 + 2 * (kPfDh / 32) * 4);
constexpr size_t kPfStates = 2 * kPfGroups * kPfPartBytes, kPfCounts = kPfGroups * sizeof(int);

#define EKV_INLINE __attribute__((always_inline))
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// a query's running maximum is raised when a lane's 16 probabilities of a 32-key block add up to more than this: none is larger
constexpr float kPfSumLimit = 256.f;

// QB: 32-query blocks per wave; a work-group (one per compute unit, one wave per SIMD) has 128 QB queries of one head.
template <int TWO_R, int QB>
__global__ __launch_bounds__(256, 1) void prefill_attn_kernel(const PrefillParams p) {
  constexpr int KCH = TWO_R / 8;                 // leading 16-byte chunks of a key row that come from the elite plane
  constexpr int R = TWO_R / 2;
  constexpr int QBLK = 128 * QB;                 // queries per work-group
  constexpr int KS = kPfDh / 16, DT = kPfDh / 32;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  int* red = reinterpret_cast<int*>(smem + kPfRing * kPfStage);
  int* order = red + 16;                         // order[pp]: the chunk of q that is pair pp of the packed query
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n32 = lane & 31, g = lane >> 5, i16 = lane & 15, q16 = lane >> 4;

  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem);

  // Work-groups go to the eight XCDs round-robin by linear index.  Divided: an XCD gets one stretch of the line of all tiles,
  // a work-group a part of it.  A work-group per block: the blocks of a head on one XCD, those that see the most keys first.
  int wg, at, line_end;
  if (p.groups > 0) {
    const int per_xcd = (p.groups + 7) / 8;
    wg = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (wg >= p.groups) return;
    at = wg * p.stretch + min(wg, p.longer);
    line_end = at + p.stretch + (wg < p.longer ? 1 : 0);
  } else {
    const int heads8 = (p.B * p.n_h + 7) / 8 * 8;
    wg = blockIdx.x / heads8;                    // place among the head's blocks
    const int head = blockIdx.x % heads8;
    if (head >= p.B * p.n_h) return;
    at = head * p.head_tiles;
    for (int i = 0; i < wg; ++i) at += pf_block_tiles(p.S, p.T, p.nqb - 1 - i, QBLK, p.shift);
    line_end = at + 1;                           // (the block's tiles follow below)
  }
  auto owner = [&](int t) EKV_INLINE {           // of tile t of the line
    const int split = p.longer * (p.stretch + 1);
    return t < split ? t / (p.stretch + 1) : p.longer + (t - split) / p.stretch;
  };
  while (at < line_end) {
  // the next block of the stretch (a head's blocks lie in falling order), its tiles lo .. hi - 1 of `tiles`
  const int ph = at / p.head_tiles;
  int first = ph * p.head_tiles;                 // of the block, on the line
  int qblk = p.nqb - 1, tiles = pf_block_tiles(p.S, p.T, qblk, QBLK, p.shift);
  while (first + tiles <= at) {
    first += tiles;
    tiles = pf_block_tiles(p.S, p.T, --qblk, QBLK, p.shift);
  }
  const int lo = at - first, hi = p.groups > 0 ? min(tiles, line_end - first) : tiles;
  at = first + hi;
  int piece = 0, pieces = 1;
  if (hi - lo < tiles) {
    piece = wg - owner(first);
    pieces = owner(first + tiles - 1) - owner(first) + 1;
  }
  const int b = ph / p.n_h, h = ph % p.n_h;
  const int64_t row0 = (int64_t)b * p.batch_stride_rows;
  __syncthreads();                               // the block before is done with the LDS

  // ---- the wave's rows of q, as the caller holds them, into the last stages (four rows of 16 chunks per load; chunk c of
  // row i lies at chunk c ^ (i & 15): the gather below reads one chunk of 32 rows at a time)
  const int tq0 = qblk * QBLK + wave * (32 * QB);
#pragma unroll
  for (int a = 0; a < QB; ++a)
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = u * 4 + (lane >> 4);
      const int t = min(tq0 + a * 32 + i, p.T - 1);           // past the last query: computed like it, never stored
      const bf16_t* src = p.q + (((int64_t)b * p.T + t) * p.n_h + h) * kPfDh + ((lane & 15) ^ (i & 15)) * 8;
      pf_dma16(src, lds0 + (kPfRing - 1 - a) * kPfStage + wave * 8192 + u * 1024);
    }
  int len[QB];
  int32_t q_at[QB];
  float m_run[QB], l_run[QB];
  // the block's largest visible length bounds the key loop; keys below the wave's smallest need no mask
  int wmax = 0, wmin = 0x7fffffff;
#pragma unroll
  for (int a = 0; a < QB; ++a) {
    const int tq = tq0 + a * 32 + n32;
    const int64_t qrow = (int64_t)b * p.T + min(tq, p.T - 1);
    int64_t len64 = p.kv_len[qrow];
    q_at[a] = p.q_pos[qrow];
    len64 = min(len64, p.max_seq_len);
    len64 = min(len64, p.plane_rows - row0);
    len64 = min(len64, p.S);
    len[a] = (int)max(len64, (int64_t)0);
    wmax = max(wmax, len[a]);
    wmin = min(wmin, len[a]);
    l_run[a] = 0.f;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    wmax = max(wmax, __shfl_xor(wmax, o, kWave));
    wmin = min(wmin, __shfl_xor(wmin, o, kWave));
  }
  wmin = __builtin_amdgcn_readfirstlane(wmin);
  if (lane == 0) red[wave] = wmax;

  // ---- the packed query's dim order (Section 3.1 score equation): the head's elite chunks in slot
  // order, then the other chunks ascending -- the order of a rebuilt key row [ke | c B^k]
  if (wave == 0) {
    int slot = -1;
    for (int j = 0; j < R; ++j)
      if (p.elite_idx[h * R + j] == lane) slot = j;
    const unsigned long long elite = __ballot(slot >= 0);
    const int rank = __popcll(~elite & ((1ull << lane) - 1ull));   // non-elite chunks below this one
    const int pp = slot >= 0 ? slot : R + rank;
    order[lane] = 0;                                               // (repeated elite indices leave holes: keep them in range)
    if (pp < kPfDh / 2) order[pp] = lane;
  }
  __syncthreads();
  const int kv_hi = __builtin_amdgcn_readfirstlane(max(max(red[0], red[1]), max(red[2], red[3])));
  // this work-group's tiles: the same share of the block's real ones
  const int real = (kv_hi + kPfTile - 1) / kPfTile;
  const int tile0 = real == tiles ? lo : (int)((int64_t)lo * real / tiles);
  const int ntiles = (real == tiles ? hi : (int)((int64_t)hi * real / tiles)) - tile0;
#pragma unroll
  for (int a = 0; a < QB; ++a) m_run[a] = len[a] > tile0 * kPfTile ? -INFINITY : 0.f;   // (sees nothing: all its probabilities are 0)

  // ---- loader: load u of wave w fills rows 16u + 4w .. + 3 of the K tile and of the V tile; lane l fills (row l/16, chunk
  // position l%16) and fetches the logical chunk the swizzle puts there: the same one for every u, so a lane has one
  // running pointer into the keys (elite plane or rebuilt rows) and one into the values, moved on by 16 rows per load
  const int ld_row = wave * 4 + (lane >> 4);
  const int lc = (lane & 15) ^ pf_swz(ld_row);
  const char* kv_seq = reinterpret_cast<const char*>(p.kv) + (int64_t)b * p.S * p.NKV * 2;
  const char* ke_seq = reinterpret_cast<const char*>(p.ke_plane) + (row0 * p.n_h + h) * (int64_t)(TWO_R * 2);
  const bool from_ke = KCH > 0 && lc < KCH;
  const int v_step = (int)p.NKV * 2, k_step = from_ke ? p.n_h * (TWO_R * 2) : v_step;        // bytes per row
  const int64_t row_first = (int64_t)tile0 * kPfTile + ld_row;
  const char* k_ptr = (from_ke ? ke_seq + lc * 16 : kv_seq + ((int64_t)h * (kPfDh - TWO_R) + (lc - KCH) * 8) * 2) +
                      row_first * k_step;
  const char* v_ptr = kv_seq + (p.NK + (int64_t)h * kPfDh + lc * 8) * 2 + row_first * v_step;
  // the loads of a tile (e = 2 u: keys, 2 u + 1: values), in this order, tile after tile.  WHOLE: all of its rows are visible
  auto issue_load = [&](int tile, int e, auto whole) EKV_INLINE {
    const int u = e >> 1;
    const uint32_t dst = lds0 + (tile & (kPfRing - 1)) * kPfStage + wave * 1024 + u * 4096 + (e & 1) * kPfPlane;
    const char*& ptr = e & 1 ? v_ptr : k_ptr;
    const int step = e & 1 ? v_step : k_step;
    const char* src = ptr;
    if constexpr (!decltype(whole)::value)                    // rows past the end repeat the last visible one
      src += min(kv_hi - 1 - ((tile0 + tile) * kPfTile + u * 16 + ld_row), 0) * step;
    pf_dma16(src, dst);
    ptr += 16 * step;
  };
  // tile t is requested from the middle of iteration t - 3 to the middle of iteration t - 2, the first ones here
  constexpr int NU = 2 * QB, NG = 2 * NU, kPerGroup = 8 / NG; // units and groups of MFMAs of a tile, loads per group (below)
  constexpr int kAhead = kPfRing - QB;                        // tiles requested while the last stages hold the queries
  auto request = [&](int t) EKV_INLINE {
    const int n = t == kPfRing - 2 ? 2 * kPerGroup : 8;
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (e < n) issue_load(t, e, std::false_type{});
  };
#pragma unroll
  for (int t = 0; t < kAhead; ++t)
    if (t < ntiles && t < kPfRing - 1) request(t);
  // the queries have landed (the tiles' loads are behind them)
  constexpr int kBehind = (kAhead - 1) * 8 + (kAhead == kPfRing - 1 ? 2 * kPerGroup : 8);
  if (ntiles >= kAhead) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kBehind) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  // the wave's queries as the B operand: lane = query n32, packed dims 16*ks + 8*g .. of block a, gathered pair by
  // pair in the packed order; elite pairs (the first R) rotated to the query's position (Section 2.2, eq. 1a);
  // everything scaled by log2(e)/sqrt(d_h)
  pf_bf16x8 Qb[QB][KS];
#pragma unroll
  for (int a = 0; a < QB; ++a) {
    const char* raw_row = smem + (kPfRing - 1 - a) * kPfStage + wave * 8192 + n32 * 256;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint32_t w[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int pp = 8 * ks + 4 * g + j;
        const int ch = order[pp];
        const uint32_t raw = *reinterpret_cast<const uint32_t*>(raw_row + (((ch >> 2) ^ (n32 & 15)) << 4) + (ch & 3) * 4);
        float x = bf16_bits_to_f32(raw & 0xffffu), y = bf16_bits_to_f32(raw >> 16);
        if (8 * ks < R) {                                     // k-steps that can hold elite pairs (compile-time)
          if (pp < R) {
            float sn, cs;
            rope_sincos_poly(q_at[a], p.rope.theta[ch], &sn, &cs);
            const float x2 = x * cs - y * sn, y2 = x * sn + y * cs;
            x = x2; y = y2;
          }
        }
        w[j] = pf_pack2(x * p.scale, y * p.scale);
      }
      Qb[a][ks] = __builtin_bit_cast(pf_bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
    }
  }

  // ---- LDS read offsets
  // keys as the A operand of S^T: row kb*32 + n32, logical chunk 2*ks + g
  const int k_row_off = n32 * kPfRow;
  const int k_swz = pf_swz(n32);                 // the same for row n32 + 32
  // values, transposed: for a k-step (kb, s2) the lane's 16-lane group supplies keys
  // kb*32 + 16*s2 + 4*g + i16/4 (+ 8 for the upper half) and dims 32*dt + 16*(q16%2) + 4*(i16%4) ..
  const int v_r = 4 * g + (i16 >> 2);
  const int v_ch = ((q16 & 1) << 1) | ((i16 & 3) >> 1);
  const int v_lo_swz = ((i16 >> 2) << 2) | g;
  const int v_hi_swz = ((i16 >> 2) << 2) | ((g + 2) & 3);
  const int v_byte = (i16 & 1) << 3;

  pf_f32x16 oacc[QB][DT];
#pragma unroll
  for (int a = 0; a < QB; ++a)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) oacc[a][dt] = (pf_f32x16)(0.f);

  // register v of a score block (32 keys from key_blk on) is key key_blk + 8*(v/4) + 4*g + v%4 for this lane's query
  auto mask = [&](pf_f32x16& s, int a, int key_blk) EKV_INLINE {
    const int rest = len[a] - key_blk - 4 * g;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 8 * (v >> 2) + (v & 3) < rest ? s[v] : -INFINITY;
  };
  // two probabilities of a block (log2 domain: the packed query carries log2(e)/sqrt(d_h))
  auto soft2 = [&](const pf_f32x16& s, int i, float m, uint32_t (&w)[8], float& psum) EKV_INLINE {
    const float p0 = __builtin_amdgcn_exp2f(s[2 * i] - m), p1 = __builtin_amdgcn_exp2f(s[2 * i + 1] - m);
    psum += p0;
    psum += p1;
    w[i] = pf_pack2(p0, p1);
  };
  // a block whose probabilities grew too large for the running maximum (the first one always): raised, and formed again
  auto raise = [&](const pf_f32x16& s, int a, uint32_t (&w)[8], float& psum) EKV_INLINE {
    float t = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) t = fmaxf(t, s[v]);
    t = fmaxf(t, __shfl_xor(t, 32, kWave));
    const float other = __shfl_xor(psum, 32, kWave);          // the other sixteen keys of this lane's query
    const float m_new = psum <= kPfSumLimit && other <= kPfSumLimit ? m_run[a] : fmaxf(m_run[a], t);
    const float m_use = m_new == -INFINITY ? 0.f : m_new;     // nothing visible yet: every exponential below is 0
    const float alpha = __builtin_amdgcn_exp2f(m_run[a] - m_use);
    m_run[a] = m_new;
    l_run[a] *= alpha;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      // the accumulators stay in the AGPRs on both sides of the branch (left alone, the compiler moves them to VGPRs around
      // it in every tile); the wait states are those between an MFMA and a read of its result, and a write and the next MFMA
      asm volatile("s_nop 15\n\ts_nop 7" : "+a"(oacc[a][dt]));
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        float y, z;
        asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(y) : "a"(oacc[a][dt][j]));
        y *= alpha;
        asm volatile("v_accvgpr_write_b32 %0, %1\n\ts_nop 2" : "=a"(z) : "v"(y));
        oacc[a][dt][j] = z;
      }
      asm volatile("" : "+a"(oacc[a][dt]));
    }
    psum = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) soft2(s, i, m_use, w, psum);
  };

  pf_bf16x8 kf[2][KS], vf[2][8];
  auto read_k = [&](const char* Kt, int kb, int ks) EKV_INLINE {
    kf[kb][ks] = *reinterpret_cast<const pf_bf16x8*>(Kt + k_row_off + (((2 * ks + g) ^ k_swz) << 4) + kb * 32 * kPfRow);
  };
  // a value fragment of a block: k-slot (g, j) of k-step s2 is key 16*s2 + 8*(j/4) + 4*g + j%4
  auto read_v = [&](const char* Vt, int kb, int i) EKV_INLINE {
    const int s2 = i >> 2, ch = 4 * (i & 3) + v_ch;
    const char* vlo = Vt + (kb * 32 + 16 * s2 + v_r) * kPfRow + v_byte;
    const pf_s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((pf_lds_s16x4_t*)(vlo + ((ch ^ v_lo_swz) << 4)));
    const pf_s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((pf_lds_s16x4_t*)(vlo + 8 * kPfRow + ((ch ^ v_hi_swz) << 4)));
    vf[kb][i] = __builtin_bit_cast(pf_bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  if (ntiles > 0) {
    if (ntiles >= kAhead) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kBehind - 8) : "memory");   // tile 0 has landed
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                                          // ... everyone's; and everyone's queries are in registers
#pragma unroll
    for (int t = kAhead; t < kPfRing - 1; ++t)
      if (t < ntiles) request(t);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) read_k(smem, 0, ks);
  }

  // A tile is 4 QB groups of eight MFMAs: the scores of the units (32 keys, 32 queries) u = kb QB + a, then their values.  The
  // order is written out (the asm statements and barriers keep it): a wave's vector instructions and LDS reads stand
  // behind MFMAs of the same wave, which they overlap.
  constexpr int kPairs = 8 * NU, kSlots = 8 * (QB == 1 ? 2 : 6);   // pairs of probabilities, spread over the groups 1 ..
  // Tiles count from this work-group's first.  CLEAN: every key is visible to the wave, and tile it + 3 is there and whole
  auto tile = [&](int it, auto clean) EKV_INLINE {
    constexpr bool CLEAN = decltype(clean)::value;
    const char* Kt = smem + (it & (kPfRing - 1)) * kPfStage;
    const char* Vt = Kt + kPfPlane;
    const char* Kn = smem + ((it + 1) & (kPfRing - 1)) * kPfStage;
    const int key0 = (tile0 + it) * kPfTile;
    pf_f32x16 s[NU];
    uint32_t w[NU][8];
    float ps[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) { s[u] = (pf_f32x16)(0.f); ps[u] = 0.f; }
#pragma unroll
    for (int a = 0; a < QB; ++a)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(Qb[a][ks]));
    static_for<NG>([&](auto gic) EKV_INLINE {
      constexpr int gi = decltype(gic)::value, u = gi % NU, kb = u / QB, a = u % QB;
      if constexpr (gi == NG - 2) {
        // tile it + 1 has landed (eight loads of tile it + 2 may be out); everyone is done with tile it - 1
        if (CLEAN || it + 2 < ntiles) asm volatile("s_waitcnt vmcnt(8)\n\ts_barrier" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
      }
      static_for<8>([&](auto ic) EKV_INLINE {
        constexpr int i = decltype(ic)::value;
        if constexpr (gi < NU) {
          s[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kb][i], Qb[a][i], s[u], 0, 0, 0);
          asm volatile("" : "+v"(s[u]));
        } else {
          constexpr int s2 = i >> 2, dt = i & 3;
          const pf_bf16x8 P = __builtin_bit_cast(pf_bf16x8, make_uint4(w[u][4 * s2], w[u][4 * s2 + 1], w[u][4 * s2 + 2], w[u][4 * s2 + 3]));
          // (a group's probabilities may have been formed again just before it: two wait states ahead of the first read)
          if constexpr (i == 0) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(oacc[a][dt]) : "v"(vf[kb][i]), "v"(P));
          else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(oacc[a][dt]) : "v"(vf[kb][i]), "v"(P));
        }
        // the operands of the next group that needs new ones
        if constexpr (gi == QB - 1) read_k(Kt, 1, i);
        if constexpr (gi == 2 * QB - 1) read_v(Vt, 0, i);
        if constexpr (gi == 3 * QB - 1) read_v(Vt, 1, i);
        if constexpr (gi == 4 * QB - 1) read_k(Kn, 0, i);     // (behind the last tile: whatever lies there, unused)
        // one load at a time, from the barrier on: the first of tile it + 3 here, the rest of tile it + 2 before it
        if constexpr (i % (8 / kPerGroup) == 0) {
          constexpr int e = ((gi + 2) % NG) * kPerGroup + i / (8 / kPerGroup);
          const int t = it + kPfRing - (gi >= NG - 2 ? 1 : 2);
          if (CLEAN || t < ntiles) issue_load(t, e, clean);
        }
        constexpr int slot = (gi - 1) * 8 + i;
        if constexpr (slot >= 0 && slot < kSlots) {
          constexpr int from = slot * kPairs / kSlots, to = (slot + 1) * kPairs / kSlots;
          static_for<to - from>([&](auto pc) EKV_INLINE {
            constexpr int pp = from + decltype(pc)::value, u2 = pp / 8, a2 = u2 % QB;
            soft2(s[u2], pp % 8, m_run[a2], w[u2], ps[u2]);
            asm volatile("" : "+v"(w[u2][pp % 8]), "+v"(ps[u2]));
            // units complete: those of the first 32 keys are looked at together, of the others each before its values' turn
            constexpr bool first = u2 < QB;
            if constexpr (first ? pp == 8 * QB - 1 : pp % 8 == 7) {
              constexpr int u0 = first ? 0 : u2, n = first ? QB : 1, a0 = u0 % QB;
              bool fits = true;
#pragma unroll
              for (int x = 0; x < n; ++x) fits &= ps[u0 + x] <= kPfSumLimit;
              if (__builtin_expect(__any(!fits), 0)) {
#pragma unroll
                for (int x = 0; x < n; ++x) raise(s[u0 + x], a0 + x, w[u0 + x], ps[u0 + x]);
              }
#pragma unroll
              for (int x = 0; x < n; ++x) l_run[a0 + x] += ps[u0 + x];
            }
          });
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      if constexpr (gi < NU && !CLEAN) {
        if (key0 + (gi / QB + 1) * 32 > wmin) mask(s[gi], gi % QB, key0 + gi / QB * 32);
      }
    });
    // The compiler does not know the value products for MFMAs: their last results are complete before it may move them.
    asm volatile("s_nop 15");
  };
  const int n_clean = min(min(wmin / kPfTile, kv_hi / kPfTile - (kPfRing - 1)) - tile0, ntiles - (kPfRing - 1));
  int it = 0;
  for (; it < n_clean; ++it) tile(it, std::true_type{});
  for (; it < ntiles; ++it) tile(it, std::false_type{});

  float l_tot[QB];
#pragma unroll
  for (int a = 0; a < QB; ++a) l_tot[a] = l_run[a] + __shfl_xor(l_run[a], 32, kWave);

  // ---- a block of several work-groups: each leaves its state (maximum, sum, accumulators), the last one to arrive adds them
  // up in the order of the pieces.  Device-scope stores, acknowledged before the count.
  if (pieces > 1) {
    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
    constexpr int kDevice = 16;                  // sc1: device scope
    const __amdgpu_buffer_rsrc_t part = __builtin_amdgcn_make_buffer_rsrc(p.part, 0, (uint32_t)kPfStates, 0x00020000);
    const uint32_t mine = (uint32_t)(2 * wg + (piece == 0)) * (uint32_t)kPfPartBytes;
    auto put = [&](int i, float x, float y, float z, float t) EKV_INLINE {
      const u32x4 v = {__float_as_uint(x), __float_as_uint(y), __float_as_uint(z), __float_as_uint(t)};
      __builtin_amdgcn_raw_buffer_store_b128(v, part, tid * 16, mine + i * 4096, kDevice);
    };
#pragma unroll
    for (int a = 0; a < QB; ++a) {
      put(a, l_tot[a] > 0.f ? m_run[a] : -INFINITY, l_tot[a], 0.f, 0.f);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          put(2 + (a * DT + dt) * 4 + j, oacc[a][dt][4 * j], oacc[a][dt][4 * j + 1], oacc[a][dt][4 * j + 2], oacc[a][dt][4 * j + 3]);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0)
      red[0] = __hip_atomic_fetch_add(p.arrived + (wg - piece), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(red[0]) != pieces - 1) continue;
    float m_all[QB];
#pragma unroll
    for (int a = 0; a < QB; ++a) {
      m_all[a] = -INFINITY;
      l_tot[a] = 0.f;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) oacc[a][dt] = (pf_f32x16)(0.f);
    }
    auto get = [&](int j, int i) EKV_INLINE {    // of piece j of the block
      const uint32_t theirs = (uint32_t)(2 * (wg - piece + j) + (j == 0)) * (uint32_t)kPfPartBytes;
      return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(part, tid * 16, theirs + i * 4096, kDevice));
    };
    for (int j = 0; j < pieces; ++j) {
#pragma unroll
      for (int a = 0; a < QB; ++a) m_all[a] = fmaxf(m_all[a], get(j, a).x);
    }
    for (int j = 0; j < pieces; ++j) {
#pragma unroll
      for (int a = 0; a < QB; ++a) {
        float4 o[DT * 4];                        // all requested before the first is used
        const float4 ml = get(j, a);
#pragma unroll
        for (int i = 0; i < DT * 4; ++i) o[i] = get(j, 2 + a * DT * 4 + i);
        __builtin_amdgcn_sched_barrier(0);
        const float w = ml.y > 0.f ? __builtin_amdgcn_exp2f(ml.x - m_all[a]) : ml.y;    // (a sum that is not a number stays one)
        l_tot[a] += w * ml.y;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            oacc[a][dt][4 * i] = fmaf(w, o[dt * 4 + i].x, oacc[a][dt][4 * i]);
            oacc[a][dt][4 * i + 1] = fmaf(w, o[dt * 4 + i].y, oacc[a][dt][4 * i + 1]);
            oacc[a][dt][4 * i + 2] = fmaf(w, o[dt * 4 + i].z, oacc[a][dt][4 * i + 2]);
            oacc[a][dt][4 * i + 3] = fmaf(w, o[dt * 4 + i].w, oacc[a][dt][4 * i + 3]);
          }
      }
    }
  }

  // ---- normalise and store, whole rows at a time: register 4*j + i of tile dt is dim 32*dt + 8*j + 4*g + i of the lane's
  // query.  Through the wave's part of two stages that nobody reads any more (8-byte stores to 32 rows at once took 4 us).
#pragma unroll
  for (int a = 0; a < QB; ++a) {
    char* rows = smem + ((ntiles + 1 + a) & (kPfRing - 1)) * kPfStage + wave * 8192;
    const float inv = l_tot[a] > 0.f ? 1.f / l_tot[a] : 0.f;  // a query that sees nothing gets a zero row
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        uint2 pk;
        pk.x = pf_pack2(oacc[a][dt][4 * j] * inv, oacc[a][dt][4 * j + 1] * inv);
        pk.y = pf_pack2(oacc[a][dt][4 * j + 2] * inv, oacc[a][dt][4 * j + 3] * inv);
        *reinterpret_cast<uint2*>(rows + n32 * 256 + (((4 * dt + j) ^ (n32 & 15)) << 4) + g * 8) = pk;
      }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = u * 4 + (lane >> 4), tq = tq0 + a * 32 + i;
      const uint4 v = *reinterpret_cast<const uint4*>(rows + i * 256 + (((lane & 15) ^ (i & 15)) << 4));
      if (tq < p.T) *reinterpret_cast<uint4*>(p.out + (((int64_t)b * p.T + tq) * p.n_h + h) * kPfDh + (lane & 15) * 8) = v;
    }
  }
  }
}

// ---------------------------------------------------------------------------------------------
static elitekv_dims rebuild_dims(const elitekv_dims& d) {
  elitekv_dims g = d;
  g.d_model = d.d_c;                                         // contraction over the latent
  g.r = 0;                                                   // no elite columns, nothing is rotated
  g.d_c = d.n_heads * (2 * d.head_dim - 2 * d.r);            // [non-elite key dims | values] of every head
  return g;
}

// Below this many queries per sequence the absorbed form (every query through the decode kernels) is the
// cheaper order: rebuilding a row costs 2 d_c (2 d_h - 2r) flops per head, about what 60-70 absorbed queries
// cost on it at their measured rates.
constexpr int kPfMinQueries = 48;

bool prefill_flash_supported(const elitekv_dims& d, int d_ck, int64_t T, int64_t max_seq_len) {
  if (d.dtype != ELITEKV_BF16 || d.head_dim != kPfDh) return false;
  // separated latents: keys are rebuilt from the first d_ck columns of a latent row and values from the rest,
  // each slice in whole contraction stages, and no 128-column block of the rebuilt row lies across the two
  if (d_ck < 0 || d_ck >= d.d_c || d_ck % kGdStage) return false;
  if (d_ck > 0 && (d.n_heads * (d.head_dim - 2 * d.r)) % 128) return false;
  if (T < kPfMinQueries) return false;
  if (2 * d.r != 8 && 2 * d.r != 16) return false;
  if (d.d_c % kGdStage || T < 1 || max_seq_len <= 64 || max_seq_len > (1 << 30)) return false;
  const elitekv_dims g = rebuild_dims(d);
  return append_gemm_supported(g, max_seq_len, d.n_heads * (d.head_dim - 2 * d.r));
}

AppendArgs prefill_rebuild_args(const elitekv_dims& d, int d_ck, int64_t rows) {
  AppendArgs g{};
  g.dims = rebuild_dims(d); g.d_ck = d.n_heads * (d.head_dim - 2 * d.r); g.T = rows;
  if (d_ck > 0) {                                              // [c^k | c^v] rows: keys from c^k, values from c^v
    g.dims.d_model = d_ck; g.x_ld = d.d_c; g.x_off2 = d_ck; g.d2 = d.d_c - d_ck;
  }
  return g;
}

static size_t pf_align(size_t v) { return (v + 255) / 256 * 256; }

// Blocks of 128 or 256 queries, and a work-group per block or the tiles of all blocks divided evenly (in stretches of at
// least eight).
static void pf_line(PrefillParams& p, int block) {
  p.nqb = (p.T + block - 1) / block;
  const int64_t heads = (int64_t)p.B * p.n_h;
  int64_t line;
  for (p.shift = 0;; ++p.shift) {
    int64_t n = 0;
    for (int i = 0; i < p.nqb; ++i) n += pf_block_tiles(p.S, p.T, i, block, p.shift);
    p.head_tiles = (int)n;
    line = heads * n;
    if (line < (1LL << 30)) break;
  }
  p.groups = (int)std::min<int64_t>(kPfGroups, std::max<int64_t>(heads * p.nqb, line / 8));
  p.stretch = (int)(line / p.groups);
  p.longer = (int)(line % p.groups);
}

// us a launch takes with a work-group per block: the compute units that are free first take the next heads' blocks
static double pf_time_blocks(const PrefillParams& p, int block, double tile_us, double block_us) {
  constexpr int kMost = 256;                                 // steps followed; of longer launches the mean will do
  struct { double until; int64_t units; } busy[kMost + 2] = {{0.0, kPfGroups}};   // ascending
  int n = 1;
  const int64_t heads = (int64_t)p.B * p.n_h;
  double all = 0, last = 0;
  int64_t steps = 0;
  for (int i = p.nqb - 1; i >= 0; --i) {
    const double t = block_us + tile_us * (double)((int64_t)pf_block_tiles(p.S, p.T, i, block, p.shift) << p.shift);
    all += t * heads;
    if ((steps += heads / kPfGroups + 2) > kMost) continue;
    for (int64_t left = heads; left > 0;) {
      const int64_t k = std::min(left, busy[0].units);
      const double until = busy[0].until + t;
      left -= k;
      if ((busy[0].units -= k) == 0) std::copy(busy + 1, busy + n--, busy);
      int at = 0;
      while (at < n && busy[at].until < until) ++at;
      if (at < n && busy[at].until == until) {
        busy[at].units += k;
      } else {
        std::copy_backward(busy + at, busy + n, busy + n + 1);
        busy[at] = {until, k};
        ++n;
      }
      last = std::max(last, until);
    }
  }
  return std::max(last, all / kPfGroups);
}

// Rows from which on blocks are divided: a stretch is eight tiles at least, so there must be longer blocks than that.
constexpr int64_t kPfDividedRows = 8 * kPfTile + 1;

// What a launch takes, us: a tile of a block, a block's first and last steps, a piece of a divided block to be added up
struct PfCosts { double tile, block, piece; };

static double pf_launch_us(const PrefillParams& c, int block, const PfCosts& k) {
  if (c.groups == 0) return 3 + pf_time_blocks(c, block, k.tile, k.block);
  const double stretch = (double)((int64_t)(c.stretch + 1) << c.shift);
  const double most = (double)((int64_t)pf_block_tiles(c.S, c.T, c.nqb - 1, block, c.shift) << c.shift);
  return 6 + stretch * k.tile + k.block * (1.0 + (double)c.B * c.n_h * c.nqb / c.groups) + k.piece * std::ceil(most / stretch);
}

// The way a launch goes: the block's width, and p.groups; 0: the kernel of prefill_pairs.hip.
// Of this file's kernel, measured alone (us, 7B 25 % and 13B 25 % shapes, 128 to 2048 queries over up to 8000 rows), blocks of
// 128 / 256 queries: a tile 1.15 / 1.9 with all compute units at work, a block's first and last steps 9 / 14, a piece 2.5 / 4.
// The four ways, queries x rows:
//   128 x 8000, 32 heads: 57 divided, 132 a work-group per block; 86 / 192 with 256-query blocks
//   2048 x 2048: 93 / 63, 87 / 70;  2 sequences: 151 / 125, 144 / 105
//   2 x 1021 x 8000, 40 heads: 474 / 492, 407 / 464
// Against the other kernel by what passes one after the other take, where the chip is warm and another tile's products cost
// power: 0.95 / 1.5 a tile, 13.8 / 25.4 a block, fitted together with that kernel's to their difference (pf_pairs_us).  The
// choice costs more than 1 % of a pass in 31 of 862 (an append and its queries), at most 5.5; this file's kernel
// alone would cost up to 7 % in batches of short prompts, the other one alone up to 56 % over long contexts:
//   queries x rows, this kernel / pairs: 64 x 128 44.2 / 41.8, 2048 x 2048 161 / 171, 8 x 512 x 512 332 / 320,
//   32 x 300 x 600 1403 / 1336, 128 x 8000 289 / 412; 13B 8 x 1024 x 1024 933 / 872, 2 x 1021 x 8000 1055 / 1259
static int pf_plan(PrefillParams& p, bool room) {
  constexpr PfCosts kAlone[2] = {{1.15, 9, 2.5}, {1.9, 14, 4}}, kWarm[2] = {{0.95, 13.8, 2.5}, {1.5, 25.4, 4}};
  double best = 0;
  PrefillParams q = p;
  int width = 0;
  for (int block = 128; block <= 256; block += 128) {
    const PfCosts& k = kAlone[block == 256];
    PrefillParams c = p;
    pf_line(c, block);
    const double divided = pf_launch_us(c, block, k);
    PrefillParams s = c;
    s.groups = 0;
    const double single = pf_launch_us(s, block, k);
    if (!room || p.S < kPfDividedRows || single <= divided) c = s;
    const double us = c.groups > 0 ? divided : single;
    if (width == 0 || us < best) {
      best = us;
      q = c;
      width = block;
    }
  }
  if (pf_pairs_us(p) < pf_launch_us(q, width, kWarm[width == 256])) {
    p.groups = 0;
    return 0;
  }
  p = q;
  return width;
}

// Workspace: the rebuilt K/V rows of all sequences; behind them, where blocks may be divided, the states of unfinished ones and
// the arrival counts.  A call without room for those has no block divided.  The size asks for the room from kPfDividedRows on
// whatever the other sizes are (fewer queries or sequences are divided rather than more), so that it never falls as any of
// them grows: a workspace for the longest chunk serves every shorter one as well.
static size_t pf_rows_bytes(const elitekv_dims& d, int64_t B, int64_t max_seq_len) {
  return pf_align((size_t)B * (size_t)max_seq_len * (size_t)rebuild_dims(d).d_c * 2);
}
size_t prefill_flash_min_workspace(const elitekv_dims& d, int64_t B, int64_t max_seq_len) {
  return pf_rows_bytes(d, B, max_seq_len);
}
size_t prefill_flash_workspace(const elitekv_dims& d, int64_t B, int64_t max_seq_len) {
  return pf_rows_bytes(d, B, max_seq_len) + (max_seq_len >= kPfDividedRows ? kPfStates + kPfCounts : 0);
}

template <int TWO_R, int QB>
static hipError_t launch_pf(const PrefillParams& p, hipStream_t stream) {
  static LdsLimit lim;
  const hipError_t e = raise_lds_limit(lim, reinterpret_cast<const void*>(&prefill_attn_kernel<TWO_R, QB>), kPfLds);
  if (e != hipSuccess) return e;
  const int64_t grid = p.groups > 0 ? (p.groups + 7) / 8 * 8 : ((int64_t)p.B * p.n_h + 7) / 8 * 8 * p.nqb;
  prefill_attn_kernel<TWO_R, QB><<<(unsigned)grid, 256, kPfLds, stream>>>(p);
  return hipGetLastError();
}

hipError_t launch_prefill_flash(const DecodeArgs& a, int64_t B, int64_t T, size_t ws_bytes, hipStream_t stream) {
  const elitekv_dims& d = a.dims;
  const int64_t S = a.max_seq_len;
  const elitekv_dims gd = rebuild_dims(d);
  const int64_t NK = (int64_t)d.n_heads * (d.head_dim - 2 * d.r), NKV = gd.d_c;
  const size_t rows_bytes = pf_rows_bytes(d, B, S);
  const bool room = ws_bytes >= rows_bytes + kPfStates + kPfCounts;
  bf16_t* kv = reinterpret_cast<bf16_t*>(a.ws);

  PrefillParams p{};
  p.q = (const bf16_t*)a.q; p.q_pos = a.q_pos; p.elite_idx = a.elite_idx;
  p.ke_plane = (const bf16_t*)a.ke_plane; p.kv = kv; p.kv_len = a.seq_len; p.out = (bf16_t*)a.out;
  p.n_h = d.n_heads; p.T = (int)T; p.B = (int)B;
  p.scale = kLog2e / sqrtf((float)d.head_dim);
  p.S = a.plane_rows > 0 ? S : 0;                            // planes without rows: nothing to see, every block one empty tile
  p.NKV = NKV; p.NK = NK;
  p.batch_stride_rows = a.batch_stride_rows; p.plane_rows = a.plane_rows; p.max_seq_len = a.max_seq_len;
  p.rope = rope_table(d.rope_base, d.head_dim);
  const int width = pf_plan(p, room);
  p.part = reinterpret_cast<float*>(a.ws + rows_bytes);
  p.arrived = p.groups > 0 ? reinterpret_cast<int*>(a.ws + rows_bytes + kPfStates) : nullptr;

  // K/V of every sequence's first S rows (rows past the end of the planes are left out)
  // Sequences that lie back to back in the planes (stride == max_seq_len) are one GEMM over all their rows;
  // otherwise one launch per sequence.
  const bool packed = a.batch_stride_rows == S && B > 1;
  hipError_t e = hipSuccess;
  for (int64_t b = 0; b < (packed ? 1 : B); ++b) {
    const int64_t row0 = b * a.batch_stride_rows;
    const int64_t want = packed ? B * S : S;
    const int64_t rows = want < a.plane_rows - row0 ? want : a.plane_rows - row0;
    if (rows <= 0) continue;
    AppendArgs g = prefill_rebuild_args(d, a.d_ck, rows);
    g.W_dkv = a.W_uk; g.W_dkv2 = a.W_uv;
    g.x = (const bf16_t*)a.c_plane + row0 * d.d_c;             // (no slots: rows written in place)
    g.c_plane = kv + b * S * NKV; g.plane_rows = want;
    g.clear = p.arrived; g.n_clear = p.groups > 0 ? kPfGroups : 0;
    e = launch_append_gemm(g, stream);
    if (e != hipSuccess) return e;
  }
  if (width == 0) return launch_prefill_pairs(p, 2 * d.r, stream);
  if (width == 256) return 2 * d.r == 16 ? launch_pf<16, 2>(p, stream) : launch_pf<8, 2>(p, stream);
  return 2 * d.r == 16 ? launch_pf<16, 1>(p, stream) : launch_pf<8, 1>(p, stream);
}

int prefill_flash_plan(const elitekv_dims& d, int64_t B, int64_t T, int64_t max_seq_len, size_t ws_bytes) {
  PrefillParams p{};
  p.n_h = d.n_heads; p.T = (int)T; p.B = (int)B; p.S = max_seq_len;
  const int width = pf_plan(p, ws_bytes >= pf_rows_bytes(d, B, max_seq_len) + kPfStates + kPfCounts);
  if (width == 0) return ELITEKV_PREFILL_PAIRS;
  return width == 256 ? (p.groups > 0 ? ELITEKV_PREFILL_256_DIVIDED : ELITEKV_PREFILL_256)
                      : (p.groups > 0 ? ELITEKV_PREFILL_128_DIVIDED : ELITEKV_PREFILL_128);
}

}  // namespace ekv
