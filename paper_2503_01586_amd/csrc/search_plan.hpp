// The plan of a RoPElite search: the pieces of its launches, the workspace, which kernel runs a round.  Plain C++: the host
// can run it without a GPU.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace ekv {

constexpr int kSrTile = 16;      // queries (and keys) per tile
constexpr int kSrMaxChunks = 64; // head_dim <= 128; the packed rows always hold 64 chunks (zeros beyond d_h / 2)
constexpr int kSrRow = 4 * kSrMaxChunks;   // floats per (token, head) of a packed operand
constexpr int kSbTiles = 4;                                 // tiles of queries (and of keys) in a block: 64 x 64 pairs

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

// Samples of up to this many tokens keep the residuals where the caller's workspace has room for them (n_h (T / 16)^2 / 2
// KiB: 66 MB for 1000 tokens of 32 heads, 1.1 GB for 4096) and the size function asks for that room up to this many bytes.
// The other searches sum the residuals again in every round, at twice the matrix instructions (search_round_kernel, 32 heads, r = 8, 128
// / 1000 / 4096 tokens: 0.128 / 1.56 / 20.9 ms instead of 0.098 / 1.05 / 14.3; in blocks, where those are taken, 0.90 at 1000).
constexpr int64_t kSrKeepTokens = 4096;
constexpr size_t kSrKeepBytes = (size_t)4 << 30;

// Operands and residuals of the samples that search_blocks_kernel takes: what the 256 MB cache behind the L2s holds but for a little
// (us a search of 128 dims, r = 8, blocks against search_round_kernel: 64 heads x 640 tokens, 216 MiB, 807 against 881; 32 x 1280,
// 267 MiB, 1493 / 1572; 64 x 768, 271 MiB, 1194 / 1171; 32 x 1536, 344 MiB, 2281 / 2132; 64 x 1000, 394 MiB, 2090 / 1943).
constexpr size_t kSbBytes = (size_t)280 << 20;

// Which of them (us a search of 128 dims, r = 8, blocks / search_round_kernel): 15 tiles and more (32 heads x 240 tokens 143 / 190, 512
// 332 / 419, 1000 949 / 1052; one head x 240 94.0 / 97.7, 1000 112 / 136; a step below 10 % the other way only for one to five
// heads of 512 tokens, 106 / 97).  Of the shorter ones, whose blocks of 64 x 64 are partly empty and whose operands take more to
// pack, those
//   whose round launch has more work-groups than the chip holds at once (two a compute unit: 64 x 144 150 / 173, 40 x 200 154 / 195),
//   or more than compute units where the same pairs are at most half as many blocks (32 x 176 106 / 123, 48 x 112 103 / 114,
//   28 x 176 117 / 125, 64 x 128 118 / 124),
//   or more than compute units where there is a block for each of them at most and the heads are dealt to the XCDs evenly, a
//   head's operands to one L2 (32 x 160 106 / 115, x 144 105 / 105, 24 x 200 112 / 125, 40 x 144 120 / 121; not so 20 x 200 135 /
//   125, 28 x 160 117 / 107, 36 x 144 125 / 119).  A search of fewer rounds gains less, for the packing is the same: r = 4, 64
//   dims, 24 x 200 64.4 / 68.0, 32 x 160 63.0 / 63.2, 40 x 160 70.1 / 68.0; r = 2, 16 dims, 32 x 160 39.5 / 37.5.
// The others lose by it or gain nothing: 32 x 128 102 / 97, x 200 144 / 135; 48 x 144 139 / 124; 44 x 144 142 / 127; 28 x 200 150 / 136; 8 x 128 91 / 89; 24 x 160
// 103 / 103; 16 x 192 (100 / 107) has the work-groups of 32 x 128 and is given up for the rule.  Below seven tiles no sample gains but
// by what two runs differ.
constexpr int kSrComputeUnits = 256;
inline bool sb_faster(int64_t tiles, int64_t n_h) {
  if (tiles < 7 || tiles >= 15) return tiles >= 15;
  const int64_t n_q32 = (tiles + 1) / 2, n_blocks = (tiles + kSbTiles - 1) / kSbTiles;
  const int64_t round_groups = n_h * sr_items_before((int)n_q32, sr_keys_per_item(n_q32, n_h));
  const int64_t block_groups = n_h * (n_blocks * (n_blocks + 1) / 2);
  if (round_groups <= kSrComputeUnits) return false;
  return round_groups > 2 * kSrComputeUnits || round_groups >= 2 * block_groups || (n_h % 8 == 0 && block_groups <= kSrComputeUnits);
}

// least: bytes a search needs, which never falls as T grows (the pieces per head do, wherever a piece gets longer: the
// partial distances are laid out for the most that a shorter sample has); total: with what it is faster with, for every
// shorter sample too.  room: what a caller has; decides what the search keeps
struct SearchLayout { size_t kp, partial, emask, arrived, res, least, total; int n_tiles, keys, n_items; bool blocks, keep; };
inline SearchLayout search_layout(int64_t T, int n_h, size_t room) {
  SearchLayout L;
  auto up = [](size_t v) { return (v + 255) / 256 * 256; };
  auto lay = [&](size_t vec, int64_t items) {                    // one packed operand, partial distances: returns the bytes
    L.kp = up(vec);
    L.partial = 2 * L.kp;
    L.emask = L.partial + up((size_t)n_h * items * kSrMaxChunks * sizeof(float));
    L.arrived = L.emask + up((size_t)n_h * sizeof(uint64_t));
    return L.res = L.arrived + up((size_t)n_h * sizeof(int32_t));
  };
  auto lay_blocks = [&](int64_t n_blocks) {
    const int64_t items = n_blocks * (n_blocks + 1) / 2;
    L.n_tiles = (int)n_blocks * kSbTiles;
    L.n_items = (int)items;
    return lay((size_t)L.n_tiles * kSrTile * n_h * kSrRow * 8, items) + (size_t)items * n_h * kSbTiles * kSbTiles * 1024;
  };
  const int64_t tiles = (T + kSrTile - 1) / kSrTile, n_q32 = (tiles + 1) / 2, blocks = (tiles + kSbTiles - 1) / kSbTiles;
  int64_t fast_blocks = std::min<int64_t>(blocks, kSrKeepTokens / (kSbTiles * kSrTile));
  while (fast_blocks > 0 && lay_blocks(fast_blocks) > kSbBytes) --fast_blocks;
  const size_t fast = lay_blocks(fast_blocks);
  L.n_tiles = (int)tiles;
  L.keys = sr_keys_per_item(n_q32, n_h);
  L.n_items = (int)sr_items_before(n_q32, L.keys);
  const int64_t most_items = std::min<int64_t>(sr_items_before(n_q32, 4), 1024 + n_q32);
  L.least = L.total = lay((size_t)tiles * kSrTile * n_h * kSrRow * sizeof(float), most_items);
  const size_t kept = (size_t)tiles * (tiles + 1) / 2 * n_h * 1024;
  if (T <= kSrKeepTokens && kept <= kSrKeepBytes) L.total += kept;
  L.keep = L.total > L.least && room >= L.total;
  L.blocks = blocks == fast_blocks && sb_faster(tiles, n_h) && room >= fast;
  if (tiles >= 7) L.total = std::max(L.total, fast);             // (a shorter sample may take the blocks where this one does not)
  if (L.blocks) lay_blocks(blocks);
  return L;
}

}  // namespace ekv
