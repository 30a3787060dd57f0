// What the two flash-attention kernels of a prefill share (prefill_attn.hip, prefill_pairs.hip): the staged tiles' shape and
// swizzle, the launch's arguments, and the lengths that the host plans with.
#pragma once
#include "common.hpp"
#include "launch.hpp"

namespace ekv {

typedef __attribute__((ext_vector_type(8))) __bf16 pf_bf16x8;
typedef __attribute__((ext_vector_type(16))) float pf_f32x16;
typedef __attribute__((ext_vector_type(4))) short pf_s16x4;
typedef __attribute__((ext_vector_type(8))) short pf_s16x8;
typedef __attribute__((address_space(3))) pf_s16x4 pf_lds_s16x4_t;

constexpr int kPfDh = 128;                       // head dim of the compiled kernel
constexpr int kPfTile = 64;                      // keys per tile
constexpr int kPfRow = kPfDh * 2;                // bytes of a staged K or V row
constexpr int kPfPlane = kPfTile * kPfRow;       // one K (or V) tile: 16 KiB
constexpr int kPfStage = 2 * kPfPlane;           // K + V

struct PrefillParams {
  const bf16_t* q;           // [B * T, n_h, d_h]  queries as the caller holds them (un-rotated)
  const int32_t* q_pos;      // [B * T]
  const int32_t* elite_idx;  // [n_h, r]
  const bf16_t* ke_plane;    // [plane_rows, n_h, 2r]
  const bf16_t* kv;          // [B, S, NKV]  rebuilt [non-elite key dims of every head | values of every head]
  const int32_t* kv_len;     // [B * T] rows of its sequence each query attends to
  bf16_t* out;               // [B * T, n_h, d_h]
  int n_h, T, B;
  int nqb;                   // query blocks per sequence
  int npair, paired;         // prefill_pairs.hip: work-groups per (sequence, head); 1: a work-group takes two query blocks
  int groups;                // work-groups among which the tiles are divided; 0: a work-group per block
  int head_tiles;            // key tiles of a (sequence, head)'s query blocks, as pf_block_tiles counts them
  int stretch, longer;       // tiles per work-group, and how many (the first ones) have one more
  int shift;                 // (a line of 2^30 tiles and more is counted in larger units)
  float* part;               // two states of an unfinished block per work-group
  int* arrived;              // per work-group: pieces left of the divided block that it has the first one of; cleared by the rebuild
  float scale;               // log2(e) / sqrt(d_h)
  int64_t S;                 // rows per sequence in kv
  int64_t NKV, NK;           // row width of kv; first value column
  int64_t batch_stride_rows, plane_rows, max_seq_len;
  RopeTable rope;
};

// Key tiles of query block i (of `block` queries) of a sequence whose last T of S rows the queries are: what the host, which
// does not see the lengths, divides among the work-groups
__host__ __device__ inline int pf_block_tiles(int64_t S, int64_t T, int i, int block, int shift) {
  int64_t end = (int64_t)(i + 1) * block;
  if (end > T) end = T;
  int64_t seen = S - T + end;
  if (seen < 1) seen = 1;
  return (int)((seen + kPfTile - 1) / kPfTile >> shift) + (shift > 0);
}

// staged rows are 16 chunks of 16 bytes; chunk c of row `row` sits at chunk c ^ pf_swz(row): 16 rows read at
// one logical chunk cover all 64 banks, and the 4 rows x 32 bytes of a transposed read cover 4 different
// 64-byte windows
__device__ __forceinline__ int pf_swz(int row) { return ((row & 3) << 2) | ((row >> 2) & 3); }

// (M0 is read one wait state after its write: the s_nop, which the compiler does not put into inline assembly)
__device__ __forceinline__ void pf_dma16(const void* gptr, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_base), "v"(gptr) : "memory", "m0");
}

__device__ __forceinline__ uint32_t pf_pack2(float lo, float hi) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  bf16x2 v;
  v[0] = (__bf16)lo;
  v[1] = (__bf16)hi;
  return __builtin_bit_cast(uint32_t, v);
}

double pf_pairs_us(const PrefillParams& p);                    // what a launch of prefill_pairs.hip takes
hipError_t launch_prefill_pairs(PrefillParams& p, int two_r, hipStream_t stream);

}  // namespace ekv
