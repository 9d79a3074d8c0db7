// Internal representation of the tile map (host side) and the device view handed to kernels.
//
// Geometry (see include/peagle.h): a row tile is A = 128/K anchors at all K depths (dense map) or a
// run of anchors whose kept positions fill 128 rows (sampled / packed maps), its rows ordered anchor by
// anchor; key tiles are 64 wide and come from two streams (depth-0 anchors, and the chain positions of a
// row tile's own anchors, each in the slot of its row).  The classification follows the parallel-prediction mask of Sec. 3 of the paper.
#pragma once

#include <cstdint>
#include <vector>

#include "peagle.h"

namespace peagle {

constexpr int kRowsPerTile = 128;
constexpr int kKeysPerTile = 64;
constexpr int kMaskWordsPerRow = kKeysPerTile / 32;                   // 2 x u32 per row
constexpr int kMaskWords = kRowsPerTile * kMaskWordsPerRow;           // 256 x u32 = 1 KiB per mask

// Quotients by a number that is the same for a whole launch, without a division: the compiler's takes 20 to 40 instructions,
// one after the other; they stood at the start of every workgroup, in front of every row's token and twice in front of every
// chain key's.  With them gone, and the products of Delta two at a time, a forward wave at L = 1,391 executes 3,470 vector
// instructions instead of 3,710 and a dQ wave 2,345 instead of 2,604.  us per step, with / without: 4 heads L = 128 27.2 / 25.2,
// 64 heads L = 1,391 691 / 684, L = 4,096 4,745 / 4,724, eight packed sequences 3,041 / 3,020.
struct Divisor {  // of numbers below 2^31, by wave-uniform arithmetic
  uint32_t d, mul, shift;
};
inline Divisor make_divisor(uint32_t d) {
  uint32_t l = 0;
  while ((1ull << l) < d) ++l;
  // mul = ceil(2^(31 + l) / d) < 2^32, and n * mul / 2^(31 + l) exceeds n / d by less than n / 2^(31 + l) <= 1 / d
  return Divisor{d, (uint32_t)(((1ull << (31 + l)) + d - 1) / d), 31 + l};
}
// of a row or slot of a row tile (x < 128) by d <= 128: x * ceil(2^16 / d) / 2^16 exceeds x / d by less than x / 2^16 < 1 / d
inline uint32_t small_reciprocal(uint32_t d) { return d ? ((1u << 16) + d - 1) / d : 0; }

struct TileEntry {
  int32_t tile;     // key-tile id in the row-tile lists, row-tile id in the key-tile lists
  int32_t mask_id;  // -1: every element of the pair is visible; >= 0: index into the mask pool.  Key-tile lists
                    // of packed maps also use INT32_MIN (listed for the pair's other tile only: nothing to do)
                    // and -2 - a (visible for keys with anchor >= a: the row tile's sequence starts at a)
};

// Pointers into device memory; passed to kernels by value.
struct DeviceTileMap {
  const int32_t* row_ptr;     // [n_row_tiles + 1]  offsets into row_entries
  const TileEntry* row_entries;
  const int32_t* row_lead;    // [n_row_tiles]  length of the leading run of full entries in each row tile's list
  const int32_t* key_ptr;     // [n_key_tiles + 1]  offsets into key_entries (row tiles ascending)
  const TileEntry* key_entries;
  const int32_t* key_seg_ptr; // [n_key_tiles][S + 1]  offsets into key_entries: where each segment's row tiles start
  const uint32_t* masks;      // [n_masks][128][2]: bit k%32 of word k/32 of row r: row r sees key k
  const uint32_t* masks_by_key;  // [n_masks][64][4]: the same bits key-major (bit r%32 of word r/32 of key k)
  const void* zeros;          // 256 zero bytes: source of rows that do not exist, for direct-to-LDS loads
  const void* no_row;         // -infinity (fp32): -lse/scale of a row that does not exist
  const int32_t* row_tok;     // sampled maps only (else null): [n_row_tiles][128] token of each row; of a row that does not
                              // exist the complement of the tile's last token (negative)
  const int32_t* chain_tok;   // sampled maps only: [n_row_tiles * n_csub][64] token of each chain key, -1 = none
  const int32_t* tok_posid;   // sampled maps only: [T] sequence position (anchor - sequence start + depth) of each token
  int32_t A, K, S, n_row_tiles, n_d0, n_csub, n_key_tiles;
  int32_t chain_slots, chain_first;  // dense maps: chain slot ck of a row tile is anchor ck / chain_slots of the tile,
                                     // depth chain_first + ck % chain_slots (depth 0: the slot is unused)
  uint32_t k_reciprocal, slots_reciprocal;  // small_reciprocal() of K and of chain_slots
};

}  // namespace peagle

struct peagle_tilemap {
  int32_t L_max = 0, K = 0, S = 0, A = 0;       // A = 0 for a sampled map (anchors per row tile vary)
  int32_t sampled = 0;                           // built from a drop-token sampled position set
  int64_t T_tokens = 0;                          // stored tokens of a length-L_max sequence
  std::vector<int32_t> seg_rt;                   // [S+1] first row tile of each segment
  std::vector<int32_t> seg_key_lo;               // [S] first depth-0 key (anchor) a segment's rows can see (packed batches)
  std::vector<int32_t> row_tok, chain_tok;       // explicit token lists of a sampled map (empty for a dense one)
  std::vector<int32_t> key_side_id;              // per row entry, packed maps only: the id the key tile -> row tile
                                                 // list carries when it differs from the row side (see finish_map)
  std::vector<int64_t> tok_pos;                  // sampled map, host only: token -> row tile * 128 + row
  std::vector<int32_t> tok_posid;                // sampled map: token -> sequence position (rotary embedding)
  int32_t max_posid = 0;                         // largest entry of tok_posid
  int32_t n_row_tiles = 0, n_d0 = 0, n_csub = 0, n_key_tiles = 0;
  int32_t chain_slots = 0, chain_first = 0;      // dense map, see DeviceTileMap
  std::vector<int32_t> seg_bounds;               // [S+1] anchors
  std::vector<int32_t> row_ptr;
  std::vector<int32_t> row_lead;                 // leading full entries per row tile
  std::vector<peagle::TileEntry> row_entries;
  std::vector<int32_t> key_ptr;
  std::vector<peagle::TileEntry> key_entries;
  std::vector<int32_t> key_seg_ptr;              // n_key_tiles * (S+1)
  bool rows_follow = false;                      // the row tiles of each depth-0 key tile's list follow one another
  std::vector<uint32_t> masks;                   // n_masks * kMaskWords
  int64_t n_full = 0, n_partial = 0;
  int32_t n_masks = 0;
  int32_t device = -1;
  void* dev_blob = nullptr;                      // one allocation holding all device arrays
  void* staging = nullptr;                       // pinned host image of the blob (source of the upload copy)
  void* copy_done = nullptr;                     // hipEvent_t recorded after the last upload copy
  int64_t dev_capacity = 0;                      // bytes allocated for dev_blob and staging
  int64_t dev_bytes = 0;                         // bytes in use
  peagle::DeviceTileMap dview{};
};

namespace peagle {

// Anchor range [lo, hi) of a segment clipped to a length-L problem, and the row tiles covering it.
struct SegRange {
  int32_t a_lo, a_hi, rt_lo, rt_hi;
  int32_t key_lo;      // first depth-0 key any of the rows can see (0 unless the map packs several sequences)
  int32_t s_lo, s_hi;  // segment boundary indices spanned: [bounds[s_lo], bounds[s_hi])
  int32_t cropped;     // the range ends before bounds[s_hi] (L < L_max cuts it short)
};
int resolve_segment(const peagle_tilemap* tm, int32_t L, int32_t seg, SegRange* out);

}  // namespace peagle
