// Flash attention of a prefill, two work-groups per compute unit: where prefill_attn.hip's kernel (one work-group per compute
// unit, which follows its matrix products) takes longer, i.e. for blocks of few tiles and launches of many of them.
//
// One work-group = 4 waves x 32 queries of one (sequence, head); a 64-key tile of K and V comes in by direct global->LDS loads,
// double-buffered.  Per wave and tile:
//   S^T[key, query]   32x32x16 MFMA, A = key rows from LDS (16-byte reads), B = the wave's queries,
//                     held in registers for the whole pass;
//   softmax           a lane owns ONE query (the MFMA output column) and 16 keys per 32-key block,
//                     its partner lane (l ^ 32) the other 16: the row maximum is an in-lane
//                     reduction plus one shuffle;
//   O^T[dim, query]   32x32x16 MFMA, B = the probabilities straight from the score registers (the
//                     keys of a k-step are taken in the order the score tile leaves them in a lane),
//                     A = V read transposed from LDS (ds_read_b64_tr_b16) in that same key order.
// Query blocks are handed out in pairs (i, last - i): under a causal mask every work-group then
// has the same number of key tiles.  Work-groups of one (sequence, head) share an XCD, so the
// tiles the later query blocks re-read come from that XCD's L2.
// What bounds it: a tile's chain of products, softmax and products, beside which the other work-group's runs; a block's first
// and last steps (lengths, queries, stores) stand beside the other's tiles.  10 KB of code, where the other kernel's 31 or 51
// KB are fetched for two tiles of a short prompt as for two hundred.  us of an append and its queries, the other kernel / this
// one: 7B 25 % 64 queries over 128 rows 44.2 / 41.8, 8 x 512 332 / 320, 16 x 700 921 / 861; 13B 8 x 1024 933 / 872.
#include <algorithm>

#include "prefill_common.hpp"

namespace ekv {

constexpr int kPpLds = 2 * kPfStage + 64 + 256;  // two stages + the block's reduction scratch + the head's chunk order

// log2-domain slack before a query's running maximum is raised: probabilities stay below 2^8
constexpr float kPpSlack = 8.f;

template <int TWO_R>
__global__ __launch_bounds__(256, 2) void prefill_pairs_kernel(const PrefillParams p) {
  constexpr int KCH = TWO_R / 8;                 // leading 16-byte chunks of a key row that come from the elite plane
  constexpr int R = TWO_R / 2;
  constexpr int QBLK = 128;                      // queries per work-group pass
  extern __shared__ __attribute__((aligned(16))) char smem[];
  int* red = reinterpret_cast<int*>(smem + 2 * kPfStage);
  int* order = red + 16;                         // order[pp]: the chunk of q that is pair pp of the packed query
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n32 = lane & 31, g = lane >> 5, i16 = lane & 15, q16 = lane >> 4;

  // work-groups go to the eight XCDs round-robin by linear index: all query blocks of one
  // (sequence, head) get indices that are equal modulo 8
  const int xcd = blockIdx.x & 7, seqi = blockIdx.x >> 3;
  const int ph = (seqi / p.npair) * 8 + xcd;
  if (ph >= p.B * p.n_h) return;
  const int pr = seqi % p.npair;
  const int b = ph / p.n_h, h = ph % p.n_h;
  const int64_t row0 = (int64_t)b * p.batch_stride_rows;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem);

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

  // ---- loader: wave w fills rows 16w .. 16w+15 of the K tile and of the V tile, four rows per load;
  // lane l fills (row l/16, chunk position l%16) and fetches the logical chunk the swizzle puts there
  const int ld_r = lane >> 4;
  const char* kv_seq = reinterpret_cast<const char*>(p.kv) + (int64_t)b * p.S * p.NKV * 2;
  const char* ke_seq = reinterpret_cast<const char*>(p.ke_plane) + (row0 * p.n_h + h) * (int64_t)(TWO_R * 2);

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

  for (int half = 0; half < 2; ++half) {
    const int qblk = half == 0 ? p.nqb - 1 - pr : pr;
    if (half == 1 && (!p.paired || qblk == p.nqb - 1 - pr)) break;   // single blocks; the middle block of an odd count
    const int tq = qblk * QBLK + wave * 32 + n32;             // this lane's query
    const bool q_ok = tq < p.T;
    const int64_t qrow = (int64_t)b * p.T + (q_ok ? tq : p.T - 1);
    int64_t len64 = q_ok ? (int64_t)p.kv_len[qrow] : 0;
    len64 = min(len64, p.max_seq_len);
    len64 = min(len64, p.plane_rows - row0);
    len64 = min(len64, p.S);
    const int len = (int)max(len64, (int64_t)0);
    int wmax = len;
    // the block's largest visible length bounds the key loop
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) wmax = max(wmax, __shfl_xor(wmax, o, kWave));
    __syncthreads();                                          // the previous block is done with red[] and the tiles
    if (lane == 0) red[wave] = wmax;
    __syncthreads();                                          // (also: order[] is complete)
    const int kv_hi = max(max(red[0], red[1]), max(red[2], red[3]));
    const int ntiles = (kv_hi + kPfTile - 1) / kPfTile;

    // the loads of a tile in four parts (u = 0..3: four rows of K and of V per wave each); a tile index past the
    // last one stands for the last one (such copies are never read)
    auto issue_part = [&](int tile, int buf, int u) {
      const uint32_t kl = __builtin_amdgcn_readfirstlane(lds0 + buf * kPfStage + wave * 4096);
      tile = min(tile, ntiles - 1);
      {
        const int row = wave * 16 + u * 4 + ld_r;
        const int lc = (lane & 15) ^ pf_swz(row);
        const int64_t t = min(tile * kPfTile + row, kv_hi - 1);   // rows past the end repeat the last visible one
        const char* krow = kv_seq + t * p.NKV * 2 + ((int64_t)h * (kPfDh - TWO_R) + (lc - KCH) * 8) * 2;
        const char* erow = ke_seq + t * (int64_t)p.n_h * (TWO_R * 2) + lc * 16;
        pf_dma16((KCH > 0 && lc < KCH) ? erow : krow, kl + u * 1024);
        const char* vrow = kv_seq + t * p.NKV * 2 + (p.NK + (int64_t)h * kPfDh + lc * 8) * 2;
        pf_dma16(vrow, kl + kPfPlane + u * 1024);
      }
    };
    auto issue = [&](int tile, int buf) {
#pragma unroll
      for (int u = 0; u < 4; ++u) issue_part(tile, buf, u);
    };
    if (ntiles > 0) issue(0, 0);                              // in flight while the queries are prepared

    // the wave's queries as the B operand: lane = query n32, packed dims 16*ks + 8*g ..,
    // gathered pair by pair from q in the packed order; elite pairs (the first R) rotated to the
    // query's position (Section 2.2, eq. 1a); everything scaled by log2(e)/sqrt(d_h)
    pf_bf16x8 Qb[kPfDh / 16];
    const bf16_t* qsrc = p.q + (qrow * p.n_h + h) * kPfDh;
    const int32_t qp = p.q_pos[qrow];
#pragma unroll
    for (int ks = 0; ks < kPfDh / 16; ++ks) {
      uint32_t w[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int pp = 8 * ks + 4 * g + j;
        const int ch = order[pp];
        const uint32_t raw = *reinterpret_cast<const uint32_t*>(qsrc + 2 * ch);
        float a = bf16_bits_to_f32(raw & 0xffffu), c = bf16_bits_to_f32(raw >> 16);
        if (8 * ks < R) {                                     // k-steps that can hold elite pairs (compile-time)
          if (pp < R) {
            float sn, cs;
            rope_sincos_poly(qp, p.rope.theta[ch], &sn, &cs);
            const float a2 = a * cs - c * sn, c2 = a * sn + c * cs;
            a = a2; c = c2;
          }
        }
        w[j] = pf_pack2(a * p.scale, c * p.scale);
      }
      Qb[ks] = __builtin_bit_cast(pf_bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
    }

    pf_f32x16 oacc[kPfDh / 32];
#pragma unroll
    for (int dt = 0; dt < kPfDh / 32; ++dt) oacc[dt] = (pf_f32x16)(0.f);
    float m_run = -INFINITY, l_run = 0.f;

    for (int it = 0; it < ntiles; ++it) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // this wave's part of tile `it` has landed
      __syncthreads();                                        // ... everyone's; and tile it-1 has been read by all
      const char* Kt = smem + (it & 1) * kPfStage;
      const char* Vt = Kt + kPfPlane;
      const int key0 = it * kPfTile;

      // ---- scores: two 32-key blocks.  All key fragments of the tile are requested
      // before the first MFMA (the compiler would otherwise read each one right before its use and
      // expose the LDS latency sixteen times); sched_barrier keeps the requests where they are.
      pf_bf16x8 kf[kPfDh / 16][2];
#pragma unroll
      for (int ks = 0; ks < kPfDh / 16; ++ks) {
        const int off = k_row_off + (((2 * ks + g) ^ k_swz) << 4);
        kf[ks][0] = *reinterpret_cast<const pf_bf16x8*>(Kt + off);
        kf[ks][1] = *reinterpret_cast<const pf_bf16x8*>(Kt + off + 32 * kPfRow);
      }
      __builtin_amdgcn_sched_barrier(0);
      pf_f32x16 sacc[2] = {(pf_f32x16)(0.f), (pf_f32x16)(0.f)};
      // The next tile's loads are requested BEHIND the first score MFMAs: vector work (here the address
      // arithmetic) overlaps MFMAs of the same wave that were issued before it, not those of the other wave.
#pragma unroll
      for (int ks = 0; ks < kPfDh / 16; ++ks) {
        sacc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks][0], Qb[ks], sacc[0], 0, 0, 0);
        sacc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks][1], Qb[ks], sacc[1], 0, 0, 0);
        if (ks < 4) {
          asm volatile("" : "+v"(sacc[1]));                // (keeps the MFMAs above the requests below)
          issue_part(it + 1, (it + 1) & 1, ks);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // ---- value fragments of the first 32 keys, requested ahead of the softmax arithmetic.
      // k-slot (g, j) of k-step (kb, s2) is key kb*32 + 16*s2 + 8*(j/4) + 4*g + j%4
      pf_bf16x8 vf[2][2][kPfDh / 32];
      auto read_v = [&](int kb) {
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          const char* vlo = Vt + (kb * 32 + 16 * s2 + v_r) * kPfRow + v_byte;
#pragma unroll
          for (int dt = 0; dt < kPfDh / 32; ++dt) {
            const int ch = 4 * dt + v_ch;
            const pf_s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((pf_lds_s16x4_t*)(vlo + ((ch ^ v_lo_swz) << 4)));
            const pf_s16x4 hi =
                __builtin_amdgcn_ds_read_tr16_b64_v4i16((pf_lds_s16x4_t*)(vlo + 8 * kPfRow + ((ch ^ v_hi_swz) << 4)));
            vf[kb][s2][dt] = __builtin_bit_cast(pf_bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
          }
        }
      };
      read_v(0);
      __builtin_amdgcn_sched_barrier(0);
      pf_bf16x8 Pb[2][2];
      // register v of block kb is key key0 + kb*32 + 8*(v/4) + 4*g + v%4 for this lane's query
      if (__any(key0 + kPfTile > len)) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int key = key0 + kb * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
            sacc[kb][v] = key < len ? sacc[kb][v] : -INFINITY;
          }
      }
      // ---- online softmax (log2 domain: the packed query carries log2(e)/sqrt(d_h))
      float t0 = fmaxf(sacc[0][0], sacc[1][0]);
#pragma unroll
      for (int v = 1; v < 16; ++v) t0 = fmaxf(t0, fmaxf(sacc[0][v], sacc[1][v]));
      const float tmax = fmaxf(t0, __shfl_xor(t0, 32, kWave));
      // the reference maximum is raised only when a score exceeds it by more than the slack
      const float m_new = (tmax > m_run + kPpSlack || m_run == -INFINITY) ? tmax : m_run;
      const float m_use = m_new == -INFINITY ? 0.f : m_new;    // nothing visible yet: every exponential below is 0
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);
      m_run = m_new;
      float psum = 0.f;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const float pv = __builtin_amdgcn_exp2f(sacc[kb][8 * s2 + j] - m_use);
            psum += pv;
            Pb[kb][s2][j] = (__bf16)pv;
          }
      l_run = l_run * alpha + psum;
      if (__any(alpha != 1.f)) {
#pragma unroll
        for (int dt = 0; dt < kPfDh / 32; ++dt) oacc[dt] *= alpha;
      }
      // ---- values: the fragments of the second 32 keys are requested before the first MFMAs
      read_v(1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
          for (int dt = 0; dt < kPfDh / 32; ++dt)
            oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[kb][s2][dt], Pb[kb][s2], oacc[dt], 0, 0, 0);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // the spare copy of the last tile has landed before the stages are reused

    // ---- normalise and store: register 4*j + i of tile dt is dim 32*dt + 8*j + 4*g + i of the lane's query
    const float l_tot = l_run + __shfl_xor(l_run, 32, kWave);
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;         // a query that sees nothing gets a zero row
    if (q_ok) {
      bf16_t* orow = p.out + (qrow * p.n_h + h) * kPfDh + 4 * g;
#pragma unroll
      for (int dt = 0; dt < kPfDh / 32; ++dt)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          uint2 pk;
          pk.x = pf_pack2(oacc[dt][4 * j] * inv, oacc[dt][4 * j + 1] * inv);
          pk.y = pf_pack2(oacc[dt][4 * j + 2] * inv, oacc[dt][4 * j + 3] * inv);
          *reinterpret_cast<uint2*>(orow + 32 * dt + 8 * j) = pk;
        }
    }
  }
}

// Pairs of blocks give every work-group the same number of key tiles, but a work-group runs its two blocks one after the
// other.  When single blocks still make at most one work-group per compute unit, the pairs would leave half of them idle: then
// every block gets a work-group of its own, heaviest first (0.085 -> 0.073 ms at 1024 tokens, 7B 25 %).  With more blocks than
// compute units the pairs are faster (2048 tokens: 0.138 against 0.153 ms with single blocks, whose heaviest two share a
// compute unit and set the launch's length).
static int64_t pp_blocks(const PrefillParams& p) { return ((int64_t)p.T + 127) / 128; }
static int64_t pp_heads(const PrefillParams& p) { return ((int64_t)p.B * p.n_h + 7) / 8 * 8; }   // whole rounds of the XCDs
static bool pp_paired(const PrefillParams& p) { return pp_heads(p) * pp_blocks(p) > 256; }

// us a launch takes.  A block: its first and last steps, its tiles, the stores of its rows; alone on a compute unit 9.2 +
// 1.28 a tile + 3.8 for 128 rows, of two that share one 20.3 + 1.74 (and 0.003 more per tile of the longest block, as less of
// the keys and values stays in the L2s) + 0.87.  Pairs are counted as rounds of 512 work-groups, the last one of 256 and fewer
// at the speed of a work-group that is alone, by a share of 0.82, and as evenly divided work by the rest.  Fitted, with the
// other kernel's times (pf_plan), to the difference of both in 862 passes (an append and its queries, one after the other; 32
// and 40 heads, 1 to 32 sequences, 48 to 2048 queries over up to 8000 rows).
double pf_pairs_us(const PrefillParams& p) {
  const int64_t n = pp_blocks(p), heads = (int64_t)p.B * p.n_h;
  auto tiles = [&](int64_t i) { return (double)pf_block_tiles(p.S, p.T, (int)i, 128, 0); };
  auto rows = [&](int64_t i) { return (double)(std::min<int64_t>(p.T, (i + 1) * 128) - i * 128) / 128; };
  auto alone = [&](int64_t i) { return 9.2 + 1.28 * tiles(i) + 3.8 * rows(i); };
  const double tile_us = 1.74 + 0.003 * tiles(n - 1);
  auto shared = [&](int64_t i) { return 20.3 + tile_us * tiles(i) + 0.87 * rows(i); };
  if (!pp_paired(p)) {
    double most = 0;
    for (int64_t i = 0; i < n; ++i) most = std::max(most, alone(i));
    return 3.5 + most;
  }
  const int64_t groups = heads * ((n + 1) / 2), rest = groups % 512;
  double work = 0;
  for (int64_t i = 0; i < n; ++i) work += shared(i) * heads;
  const double one = alone(n - 1) + (n > 1 ? alone(0) : 0), two = shared(n - 1) + (n > 1 ? shared(0) : 0);
  const double rounds = (double)(groups / 512) * (work / groups) + (rest == 0 ? 0 : rest <= 256 ? one : two);
  return 3.5 + 0.82 * rounds + 0.18 * std::max(work / 512, one);
}

template <int TWO_R>
static hipError_t launch_pp(const PrefillParams& p, hipStream_t stream) {
  static LdsLimit lim;
  const hipError_t e = raise_lds_limit(lim, reinterpret_cast<const void*>(&prefill_pairs_kernel<TWO_R>), kPpLds);
  if (e != hipSuccess) return e;
  prefill_pairs_kernel<TWO_R><<<(unsigned)(pp_heads(p) * p.npair), 256, kPpLds, stream>>>(p);
  return hipGetLastError();
}

hipError_t launch_prefill_pairs(PrefillParams& p, int two_r, hipStream_t stream) {
  p.nqb = (int)pp_blocks(p);
  p.paired = pp_paired(p) ? 1 : 0;
  p.npair = p.paired ? (p.nqb + 1) / 2 : p.nqb;
  return two_r == 16 ? launch_pp<16>(p, stream) : launch_pp<8>(p, stream);
}

}  // namespace ekv
