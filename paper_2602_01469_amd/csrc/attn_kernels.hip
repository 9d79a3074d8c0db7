// Block-sparse flash attention forward / backward for the parallel-prediction mask (Sec. 3 of
// the paper), gfx950 only.  Work is organised by the tile map: a row tile is A anchors at all K
// depths (128 rows), key tiles are 64 wide; full pairs skip masking, partial pairs apply a
// bitmask from the pool, empty pairs are never listed.
//
// All score matrices are produced transposed where that keeps the softmax reduction inside a
// lane: in the forward and dQ kernels a lane owns one query row (S^T = K Q^T, lane <-> row,
// registers <-> keys); in the dK/dV kernel a lane owns one key (S = Q K^T, lane <-> key,
// registers <-> rows).  Operands whose contraction index is not contiguous in memory are read
// from LDS with ds_read_b64_tr_b16.
#include "attn_kernels.h"
#include "mfma_util.h"
#include "rope_util.h"

#include <climits>
#include <type_traits>

namespace peagle {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
// How far the running reference max may lag, log2 units (moving it costs a pass over the accumulators).  A drafting step keeps
// it closer: the key that is the reference has a probability of exactly 1, unrounded, and the fewer pieces a context is cut
// into, the fewer references it starts.  Error against 64 bits, rel-L2, mean of 31 batches (and the worst of them against the
// cut for a thousand workgroups with a lag of 8, 2.255e-3): lag 8 2.265e-3 (+2.9 %), 2 2.223e-3 (+1.4 %, batches of one piece
// only), 1 2.178e-3 (-0.7 %).  us at a lag of 8 / 2 / 1: 4 requests of 2,048 - 4,096 tokens 12.4 / 12.7 / 13.0, 64 of 512 -
// 8,192 119.7 / 119.8 / 120.2, D = 128 35 of 2,137 - 3,838 46.0 / 47.3 / 48.0; one piece, 64 of 100 - 1,000 18.8 / 19.7 / 19.9.
constexpr int kLag = 8, kDraftLag = 2, kDraftLagOnePiece = 1;
constexpr float kNegInit = -1.0e30f;
// Bits of a 32-key mask word (already shifted right by 4g) that belong to the keys a lane holds in the
// C layout of a transposed score block: keys 8*(i/4) + 4g + i%4, i = 0..15.
constexpr uint32_t kLaneKeyBits = 0x0f0f0f0fu;

// n / d and, in its place, n % d; n wave-uniform and below 2^31 (see Divisor).
__device__ __forceinline__ int split_by(int& n, const Divisor& d) {
  const uint32_t q = (uint32_t)(((uint64_t)(uint32_t)n * d.mul) >> d.shift);
  n -= (int)(q * d.d);
  return (int)q;
}
// x / d for x < 128, r = small_reciprocal(d)
__device__ __forceinline__ int small_quotient(int x, uint32_t r) { return (int)(__umul24((uint32_t)x, r) >> 16); }

// Token (row of the [T, H, D] tensors) of key `row` of key tile `kt`; false if that key does not
// exist in a length-L problem.
__device__ __forceinline__ bool key_token(const DeviceTileMap& tm, int kt, int row, int L, int& tok) {
  if (kt < tm.n_d0) {
    tok = kt * kKeysPerTile + row;
    return tok < L;
  }
  const int cid = kt - tm.n_d0;
  if (tm.row_tok) {  // sampled map: explicit list of the tile's chain keys
    tok = tm.chain_tok[(size_t)cid * kKeysPerTile + row];
    return tok >= 0;
  }
  const int R = cid >> (tm.n_csub - 1);  // (one or two chain tiles a row tile)
  const int ck = (cid - R * tm.n_csub) * kKeysPerTile + row;
  const int a = small_quotient(ck, tm.slots_reciprocal);
  const int e = tm.chain_first + ck - a * tm.chain_slots;
  const int j = R * tm.A + a;
  tok = e * L + j;
  return e >= 1 && a < tm.A && j < L;
}

// Tokens of the keys row0, row0 + step, ... of key tile `kt`, -1 where one does not exist: a listed map's are all on their way
// before the first is waited for.
template <int N>
__device__ __forceinline__ void key_tokens(const DeviceTileMap& tm, int kt, int row0, int step, int L, int (&tok)[N]) {
  if (kt >= tm.n_d0 && tm.row_tok) {
    const int32_t* list = tm.chain_tok + (size_t)(kt - tm.n_d0) * kKeysPerTile + row0;
#pragma unroll
    for (int i = 0; i < N; ++i) tok[i] = list[i * step];
    return;
  }
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (!key_token(tm, kt, row0 + i * step, L, tok[i])) tok[i] = -1;
}

// Token of row `r` of row tile `rt`; false if the row is padding or beyond the sequence.
__device__ __forceinline__ bool row_token(const DeviceTileMap& tm, int rt, int r, int L, int& tok) {
  if (tm.row_tok) {  // sampled map: explicit list of the tile's rows
    tok = tm.row_tok[(size_t)rt * kRowsPerTile + r];
    return tok >= 0;
  }
  const int a = small_quotient(r, tm.k_reciprocal), i = rt * tm.A + a;
  tok = (r - a * tm.K) * L + i;
  return a < tm.A && i < L;
}

__device__ __forceinline__ uint4 ld16(const __bf16* p) { return *reinterpret_cast<const uint4*>(p); }
__device__ __forceinline__ bf16x8 as_frag(uint4 u) { return __builtin_bit_cast(bf16x8, u); }

// Entry `e` of a tile list, made wave-uniform (the index is uniform; this lets branches on the
// entry be scalar).  Lists are read two iterations ahead of their use: fetch_entry() starts the
// load early in an iteration, take_entry() - called after the iteration's barrier - moves the
// value to scalar registers.  The empty assembly statement pins that move below the barrier;
// without it the compiler places it, and the wait for the load, right behind the load.
__device__ __forceinline__ u32x2 fetch_entry(const TileEntry* list, int e) {
  return *reinterpret_cast<const u32x2*>(list + e);
}
__device__ __forceinline__ TileEntry take_entry(u32x2 w) {
  uint32_t w0 = w[0], w1 = w[1];
  asm volatile("" : "+v"(w0), "+v"(w1) : : "memory");
  TileEntry en;
  en.tile = __builtin_amdgcn_readfirstlane((int)w0);
  en.mask_id = __builtin_amdgcn_readfirstlane((int)w1);
  return en;
}
// An entry, or one of the map's integers, through the scalar path (index wave-uniform): what a workgroup starts with is
// looked up without waiting for the vector loads issued before it, and several at a time.
typedef const int32_t __attribute__((address_space(4))) * ConstInts;
__device__ __forceinline__ int32_t const_int(const int32_t* list, int i) { return ((ConstInts)(uintptr_t)list)[i]; }
__device__ __forceinline__ TileEntry const_entry(const TileEntry* list, int e) {
  static_assert(sizeof(TileEntry) == 8, "an entry is two words");
  const ConstInts w = (ConstInts)(uintptr_t)(list + e);
  TileEntry en;
  en.tile = w[0];
  en.mask_id = w[1];
  return en;
}

// LDS addresses of the K/V tile buffers of the row-stationary kernels, [slot][K|V][tile bytes], as plain scalar
// integers: the address of slot 0 is taken once per kernel and everything else is integer arithmetic (taken
// per copy from a pointer, each address costs a null check and two moves to the scalar unit).
template <int D>
struct KeyTileLds {
  uint32_t base;  // address of slot 0's K image + 1024 * wave
  __device__ __forceinline__ KeyTileLds(const char* slot0, int wave)
      : base(lds_scalar_addr(slot0 + wave * 1024)) {}
  __device__ __forceinline__ uint32_t k(int slot) const { return base + (uint32_t)slot * (2u * kKeysPerTile * D * 2); }
  __device__ __forceinline__ uint32_t v(int slot) const { return k(slot) + kKeysPerTile * D * 2; }
};

// The lane's number, computed anew where it stands: what is derived from it takes no register before and after.
__device__ __forceinline__ int lane_id() {
  int l = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  asm volatile("" : "+v"(l));
  return l;
}

// Key tiles straight into their swizzled LDS images (K and V): wave w of NW fills the 1 KiB blocks w, w + NW, ...; lane l of
// block b owns LDS bytes [1024 b + 16 l, +16), i.e. tile row b*(512/D) + l/(D/8) and physical chunk l%(D/8), and fetches the
// logical chunk that lives there.
// kd, vd: LDS byte addresses of this wave's first block of the K and of the V image (tile address + 1024 * wave), as
// wave-uniform integers - see KeyTileLds.
// A tile of depth-0 keys.  The rows a lane copies are NW * 512/D apart (a multiple of the swizzle period), so its byte offset
// from each copy's first row is one value, the same for every whole tile, and the rest of the address is wave-uniform.  Rows
// past the end of the sequence are read from its last row: no row of the problem sees them, and what zero times a NaN of the
// last key reaches, the last key itself has reached (a wave that takes the block of the one takes the block of the other).
template <int D, int NW>
__device__ __forceinline__ void dma_d0_tile(uint32_t kd, uint32_t vd, const __bf16* kbase, const __bf16* vbase, int Hkv, int kvh,
                                            int kt, int L, int wave, int lane) {
  constexpr int kCopies = kKeysPerTile * D * 2 / 1024 / NW, kApart = NW * (512 / D);
  static_assert(kCopies * NW * 1024 == kKeysPerTile * D * 2, "tile must split evenly over the waves");
  const int row0 = wave * (512 / D) + lane / (D / 8);
  const uint32_t chunk = (uint32_t)((lane % (D / 8) ^ swz<D>(row0)) << 4), stride = (uint32_t)(Hkv * D * 2);
  if ((kt + 1) * kKeysPerTile <= L) {
    const uint32_t voff = (uint32_t)row0 * stride + chunk;
#pragma unroll
    for (int i = 0; i < kCopies; ++i) {
      const size_t first = ((size_t)(kt * kKeysPerTile + i * kApart) * Hkv + kvh) * D;
      dma16_untracked(uniform_ptr(kbase + first), voff, kd + i * NW * 1024);
      dma16_untracked(uniform_ptr(vbase + first), voff, vd + i * NW * 1024);
    }
    return;
  }
  const int at = kt * kKeysPerTile < L ? kt * kKeysPerTile : L - 1;  // (a cropped sequence's last row tile may list a tile past it)
  const size_t first = ((size_t)at * Hkv + kvh) * D;
  const int last = L - 1 - at;
#pragma unroll
  for (int i = 0; i < kCopies; ++i) {
    const int row = row0 + i * kApart;
    const uint32_t voff = (uint32_t)(row < last ? row : last) * stride + chunk;
    dma16_untracked(uniform_ptr(kbase + first), voff, kd + i * NW * 1024);
    dma16_untracked(uniform_ptr(vbase + first), voff, vd + i * NW * 1024);
  }
}

// A tile of chain keys.  SV (first-layer form; a template flag: kernels of the ordinary step carry none of this): every key's
// value row is the one shared vector of its KV head.
template <int D, int NW, bool SV>
__device__ __forceinline__ void dma_chain_tile(uint32_t kd, uint32_t vd, const __bf16* kbase, const __bf16* vbase, int Hkv, int kvh,
                                               const DeviceTileMap& tm, int kt, int L, int wave, int lane, const __bf16* v_shared) {
  constexpr int kCopies = kKeysPerTile * D * 2 / 1024 / NW, kApart = NW * (512 / D);
  const int phys = lane % (D / 8), row0 = wave * (512 / D) + lane / (D / 8);
  int tok[kCopies];
  key_tokens(tm, kt, row0, kApart, L, tok);
#pragma unroll
  for (int i = 0; i < kCopies; ++i) {
    const bool ok = tok[i] >= 0;
    const int chunk = (phys ^ swz<D>(row0 + i * kApart)) << 3;
    const size_t off = ((size_t)(ok ? tok[i] : 0) * Hkv + kvh) * D + chunk;
    const __bf16* v = SV ? v_shared + (size_t)kvh * D + chunk : vbase + off;
    dma16_untracked(ok ? (const void*)(kbase + off) : tm.zeros, kd + i * NW * 1024);
    dma16_untracked(ok ? (const void*)v : tm.zeros, vd + i * NW * 1024);
  }
}

// Either.
template <int D, int NW, bool SV>
__device__ __forceinline__ void dma_key_tile(uint32_t kd, uint32_t vd, const __bf16* kbase, const __bf16* vbase, int Hkv, int kvh,
                                             const DeviceTileMap& tm, int kt, int L, int wave, int lane, const __bf16* v_shared) {
  if (kt < tm.n_d0) dma_d0_tile<D, NW>(kd, vd, kbase, vbase, Hkv, kvh, kt, L, wave, lane);
  else dma_chain_tile<D, NW, SV>(kd, vd, kbase, vbase, Hkv, kvh, tm, kt, L, wave, lane, v_shared);
}

// The bitmask of a row tile's key tile, to LDS with the tile's copies: each wave the words of its own 32 rows.  (A mask word
// loaded to a register where the tile is computed is waited for behind the next tile's copies, because a wave's accesses
// complete in order: nothing of them was hidden in a masked tile, three of every row tile, or in any iteration of a chain
// tile in the dK/dV kernel.  us, so / from LDS: packed 203 to 900 anchors, 64 heads 767 / 745, eight sequences 3,138 / 3,111,
// L = 411 120 / 117.5, L = 1,391 722 / 713; L = 20,480 the same, without a test for a mask in the loops over full tiles.)
constexpr int kTileMaskBytes = kRowsPerTile * kMaskWordsPerRow * 4;
__device__ __forceinline__ void dma_tile_mask(uint32_t mask_lds, const DeviceTileMap& tm, const TileEntry& en, int wave) {
  if (en.mask_id < 0) return;
  constexpr int kWords = kTileMaskBytes / 4 / 4;  // of a wave: one per lane
  static_assert(kWords == 64, "a lane copies one word");
  const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane(wave);
  dma4_untracked(uniform_ptr(tm.masks + ((size_t)en.mask_id * 4 + w) * kWords), lane_id() * 4u, mask_lds + w * (kWords * 4));
}
// ... and the words of row `row` (32-key blocks 0 and 1), shifted to the keys of the lane's half.
__device__ __forceinline__ void tile_mask(const char* mask, int row, int g, uint32_t (&mw)[2]) {
  const u32x2 w = *reinterpret_cast<const u32x2*>(mask + row * (kMaskWordsPerRow * 4));
  mw[0] = w[0] >> (4 * g);
  mw[1] = w[1] >> (4 * g);
}

// The chain tiles that end a row tile's list (none to two).  At D = 64 the row-stationary kernels take them first and together:
// a wave sees one block of 32 of the 128 chain slots (or two), so as iterations of their own each was a copy and a barrier for
// half of the workgroup's waves.  Both travel with the first tile of depth-0 keys, which the workgroup waits for anyway, into
// buffers that the loop uses later (one more than it needs, 52 KB in all: still three workgroups a CU; where four are wanted,
// the forward of one head, there are two buffers, see there).  us per step, last / first: L = 1,391 704.9 / 702.5, L = 4,096
// 4,810 / 4,786, eight packed sequences 3,077 / 3,067.  (D = 128: no LDS for two.)
struct ChainTiles {
  int n;
  TileEntry tile[2];
};
__device__ __forceinline__ ChainTiles chain_tiles(const DeviceTileMap& tm, int e0, int e1) {
  const TileEntry a = const_entry(tm.row_entries, e1 - 2 > e0 ? e1 - 2 : e0), b = const_entry(tm.row_entries, e1 - 1);
  ChainTiles c;
  const bool two = e1 - 2 > e0 && a.tile >= tm.n_d0;  // (a list starts with a tile of depth-0 keys)
  c.n = two ? 2 : b.tile >= tm.n_d0 ? 1 : 0;
  c.tile[0] = two ? a : b;
  c.tile[1] = b;
  return c;
}

// Row tile (128 rows of one query head) straight into its swizzled LDS image, same block/lane
// assignment as dma_key_tile; rows that do not exist are filled from the zero page.  The rows a
// lane copies are the same for every row tile, so their (depth, anchor) split - which costs an
// integer division by A - is done once per kernel (RowDmaLane) and a copy only adds rt*A.
template <int D, int NW>
struct RowDmaLane {
  static constexpr int kBlocks = kRowsPerTile * D * 2 / 1024;
  static constexpr int kPer = kBlocks / NW;
  static_assert(kBlocks % NW == 0, "tile must split evenly over the waves");
  int tok0[kPer];    // d*L + a : token of the row in row tile 0 (dense map)
  int a[kPer];       // anchor offset inside the row tile; >= A*K... marks a padding row via a huge value
  int row[kPer];     // row of the tile (index into a sampled map's row list)
  int chunk[kPer];   // element offset of the logical 16-byte chunk this lane fetches
  int stat_tok0, stat_a, stat_row;  // same for the row whose per-row statistic this lane copies (waves 0..3)
};
template <int D, int NW>
__device__ __forceinline__ RowDmaLane<D, NW> row_dma_lane(const DeviceTileMap& tm, int L, int wave, int lane) {
  RowDmaLane<D, NW> r;
  const int row_in_blk = lane / (D / 8), phys = lane % (D / 8);
#pragma unroll
  for (int i = 0; i < RowDmaLane<D, NW>::kPer; ++i) {
    const int row = (i * NW + wave) * (512 / D) + row_in_blk;
    const int a = small_quotient(row, tm.k_reciprocal);  // (a sampled map has no fixed geometry; rows come from its list)
    r.tok0[i] = (row - a * tm.K) * L + a;
    r.a[i] = a < tm.A ? a : (1 << 30);
    r.row[i] = row;
    r.chunk[i] = (phys ^ swz<D>(row)) << 3;
  }
  const int srow = (wave & 1) * 64 + lane;
  const int sa = small_quotient(srow, tm.k_reciprocal);
  r.stat_tok0 = (srow - sa * tm.K) * L + sa;
  r.stat_a = sa < tm.A ? sa : (1 << 30);
  r.stat_row = srow;
  return r;
}
// Dense maps whose tensors span less than 4 GiB: byte offset of each copy's source from the head's row of the tile's
// first anchor, ((d*L + a) * Hq) * D * 2 + 2 * chunk (and 4 * (d*L + a) for the statistic) - the same for every row
// tile and head, so a copy needs only a new scalar base.  (Where the rows a lane copies are a whole number of anchors
// apart, the copies' offsets differ by a scalar step and off[0] is all that is kept.)
template <int D, int NW>
struct RowDmaOffsets {
  uint32_t off[RowDmaLane<D, NW>::kPer], stat_off;
};
template <int D, int NW>
__device__ __forceinline__ RowDmaOffsets<D, NW> row_dma_offsets(const DeviceTileMap& tm, int L, int wave, int lane, int Hq) {
  RowDmaOffsets<D, NW> r;
  const int row_in_blk = lane / (D / 8), phys = lane % (D / 8);
  auto token = [&](int row) {
    const int a = small_quotient(row, tm.k_reciprocal);
    return (uint32_t)((row - a * tm.K) * L + a);
  };
#pragma unroll
  for (int i = 0; i < RowDmaLane<D, NW>::kPer; ++i) {
    const int row = (i * NW + wave) * (512 / D) + row_in_blk;
    r.off[i] = token(row) * (uint32_t)(Hq * D * 2) + (uint32_t)((phys ^ swz<D>(row)) << 4);
  }
  r.stat_off = token((wave & 1) * 64 + lane) * 4u;
  return r;
}
// Tokens of the rows this lane copies for one row tile (-1: the row does not exist).  For a dense map
// they are arithmetic; a sampled / packed map lists them, and the loads are issued an iteration
// before the copy that needs them so that their latency does not add to the copy's.
template <int D, int NW>
struct RowTokens {
  int tok[RowDmaLane<D, NW>::kPer];
  int stat_tok;
};
template <int D, int NW, bool LISTED>
__device__ __forceinline__ RowTokens<D, NW> row_tokens(const DeviceTileMap& tm, const RowDmaLane<D, NW>& rl, int rt,
                                                       int L) {
  RowTokens<D, NW> t;
  if (LISTED) {
    const int32_t* list = tm.row_tok + (size_t)rt * kRowsPerTile;
#pragma unroll
    for (int i = 0; i < RowDmaLane<D, NW>::kPer; ++i) t.tok[i] = list[rl.row[i]];
    t.stat_tok = list[rl.stat_row];
  } else {
    const int i0 = rt * tm.A;
#pragma unroll
    for (int i = 0; i < RowDmaLane<D, NW>::kPer; ++i) t.tok[i] = i0 + rl.a[i] < L ? rl.tok0[i] + i0 : -1;  // padding rows carry a huge anchor offset
    t.stat_tok = i0 + rl.stat_a < L ? rl.stat_tok0 + i0 : -1;
  }
  return t;
}
template <int D, int NW>
__device__ __forceinline__ void dma_row_tile(char* lds_tile, const __bf16* base, int Hq, int h, const DeviceTileMap& tm,
                                             const RowDmaLane<D, NW>& rl, const RowTokens<D, NW>& t, int wave) {
  const uint32_t dst = lds_scalar_addr(lds_tile + wave * 1024);
#pragma unroll
  for (int i = 0; i < RowDmaLane<D, NW>::kPer; ++i) {
    const bool ok = t.tok[i] >= 0;
    const size_t off = ((size_t)(ok ? t.tok[i] : 0) * Hq + h) * D + rl.chunk[i];
    dma16_untracked(ok ? (const void*)(base + off) : tm.zeros, dst + i * NW * 1024);
  }
}

// Per-row fp32 statistic of a row tile (128 values, [Hq, T] array) into LDS: two waves of the
// caller each fill 64 rows (half = wave & 1).
template <int D, int NW>
__device__ __forceinline__ void dma_row_stat(float* lds_stat, const float* base, int T, int h, const DeviceTileMap& tm,
                                             const RowTokens<D, NW>& t, int half) {
  const bool ok = t.stat_tok >= 0;
  dma4_untracked(ok ? (const void*)(base + (size_t)h * T + t.stat_tok) : tm.zeros,
                 lds_scalar_addr(reinterpret_cast<const char*>(lds_stat + half * 64)));
}

// Does any row of the wave see a key of the 32-key block whose (shifted) mask word each lane holds?
__device__ __forceinline__ bool wave_sees_block(uint32_t mw) {
  return __builtin_amdgcn_ballot_w64((mw & kLaneKeyBits) != 0) != 0;
}

// 32 features of a row from the C layout of a transposed block (lane and lane ^ 32 share the row: the lane holds features
// 8*(i/4) + 4g + i%4), times f, rounded to bf16.  The two lanes exchange halves so that each stores 16 bytes at a
// time: half the store instructions of 8-byte pieces, which a row tile's end waits on (forward at 1,391 anchors 171 -> 165
// us, dQ 249 -> 242; at 4,096 forward 1,112 -> 1,085, dQ 1,625 -> 1,603).
__device__ __forceinline__ u32x4 row_piece_bf16(const f32x16& x, int q, float f) {  // features 16q + 8g + 0..7
  u32x4 w;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const uint32_t even = pack_bf16(x[8 * q + 2 * j] * f, x[8 * q + 2 * j + 1] * f);
    const uint32_t odd = pack_bf16(x[8 * q + 4 + 2 * j] * f, x[8 * q + 4 + 2 * j + 1] * f);
    const u32x2 r = __builtin_amdgcn_permlane32_swap(even, odd, false, false);
    w[j] = r[0];
    w[2 + j] = r[1];
  }
  return w;
}
__device__ __forceinline__ void store_row_bf16(__bf16* dst, const f32x16& x, float f, int g) {
#pragma unroll
  for (int q = 0; q < 2; ++q) *reinterpret_cast<u32x4*>(dst + 16 * q + 8 * g) = row_piece_bf16(x, q, f);
}

// Eight more terms of a lane's half of rowsum(dO * O).  Every kernel that forms Delta adds in this order - pieces of 16
// features up, the lane's eight of each pair by pair, the halves last - so that Delta has the same bits wherever it is formed.
// (v_dot2_f32_bf16: the products exact, sums in fp32; against 64 bits 3.4e-8 over 32 features of normal data where
// unpacking and a chain of 32 fused multiply-adds, 96 instructions instead of 16, is off by 3.5e-8.)
__device__ __forceinline__ float add_delta8(float dl, bf16x8 dof, bf16x8 of) {
  const u32x4 a = __builtin_bit_cast(u32x4, dof), b = __builtin_bit_cast(u32x4, of);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t x = a[j], y = b[j];
    dl = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, x), __builtin_bit_cast(bf16x2, y), dl, false);
  }
  return dl;
}

// Bit `pos` of w selects x, otherwise -inf.
__device__ __forceinline__ float mask_sel(float x, uint32_t w, int pos) {
  return ((w >> pos) & 1u) ? x : -__builtin_inff();
}

// x where bit `pos` of w is set, otherwise 0 (whatever x is: the exponential of a score that the row does not see may be infinite).
__device__ __forceinline__ float mask_zero(float x, uint32_t w, int pos) {
  const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe((int)w, pos, 1);
  return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, x) & keep);
}

__device__ __forceinline__ float max16(const f32x16& s) {
  float a = __builtin_fmaxf(__builtin_fmaxf(s[0], s[1]), s[2]);
  float b = __builtin_fmaxf(__builtin_fmaxf(s[3], s[4]), s[5]);
  float c = __builtin_fmaxf(__builtin_fmaxf(s[6], s[7]), s[8]);
  float d = __builtin_fmaxf(__builtin_fmaxf(s[9], s[10]), s[11]);
  float e = __builtin_fmaxf(__builtin_fmaxf(s[12], s[13]), s[14]);
  a = __builtin_fmaxf(__builtin_fmaxf(a, b), c);
  d = __builtin_fmaxf(__builtin_fmaxf(d, e), s[15]);
  return __builtin_fmaxf(a, d);
}

// Online-softmax update for one 32-key block of one head.  On entry s holds raw q.k of the
// lane's row for its 16 keys; on exit pb holds exp2(s*c - m) as two bf16 B-operand fragments.
// The reference max m moves only when the block exceeds it by more than LAG, which
// keeps the accumulator rescale off the common path without affecting the result.
template <int DB, bool MASKED, int LAG>
__device__ __forceinline__ void softmax_block(f32x16& s, uint32_t mw, float c, float& m, float& lsum,
                                              f32x16 (&o)[DB], bf16x8 (&pb)[2]) {
  if (MASKED) {
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = mask_sel(s[i], mw, 8 * (i / 4) + (i % 4));
  }
  const float mx = max_halves(max16(s)) * c;
  const bool need = mx > m + (float)LAG;
  if (__builtin_amdgcn_ballot_w64(need) != 0) {
    const float m_new = need ? mx : m;
    const float alpha = exp2_fast(m - m_new);
    m = m_new;
    lsum *= alpha;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
  }
  const float neg_m = -m;
#pragma unroll
  for (int i = 0; i < 16; ++i) s[i] = exp2_fast(__builtin_fmaf(s[i], c, neg_m));
  pb[0] = pack8_sum(s, 0, lsum);
  pb[1] = pack8_sum(s, 1, lsum);
}

}  // namespace

// =====================================================================================
// Forward: O = softmax(scale Q K^T + mask) V, LSE.  One workgroup (4 waves) per
// (row tile, NH query heads of one KV group); wave w owns rows [32w, 32w+32) of the tile.
// K/V tiles are staged once in LDS per workgroup and serve all NH heads.
// =====================================================================================
template <int D, int NH, bool MASKED, bool SAFE, int LAG = kLag>
__device__ __forceinline__ void fwd_tile(const char* kt_lds, const char* vt_lds, const NatOff<D>& no, const TrOff<D>& to,
                                         const bf16x8 (&qf)[NH][D / 16], f32x16 (&o)[NH][D / 32], float (&m)[NH],
                                         float (&lsum)[NH], const uint32_t (&mw)[2], float c) {
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {  // the tile's two 32-key blocks
    // S^T block: 32 keys x 32 rows, lane <-> row, registers <-> keys 8*(i/4) + 4g + i%4
    f32x16 s[NH];
#pragma unroll
    for (int hh = 0; hh < NH; ++hh) s[hh] = zero16();
#pragma unroll
    for (int st = 0; st < D / 16; ++st) {
      const bf16x8 a = frag_nat<D>(kt_lds, no, kb, st);
#pragma unroll
      for (int hh = 0; hh < NH; ++hh) s[hh] = mfma32(a, qf[hh][st], s[hh]);
    }
    bf16x8 pb[NH][2];
#pragma unroll
    for (int hh = 0; hh < NH; ++hh) {
      if (SAFE) {
        softmax_block<D / 32, MASKED, LAG>(s[hh], mw[kb], c, m[hh], lsum[hh], o[hh], pb[hh]);
      } else {  // reference max fixed at 0: p = 2^(c s); the caller checks the row sums' range
        if (MASKED) {
#pragma unroll
          for (int i = 0; i < 16; ++i) s[hh][i] = mask_sel(s[hh][i], mw[kb], 8 * (i / 4) + (i % 4));
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) s[hh][i] = exp2_fast(s[hh][i] * c);
        pb[hh][0] = pack8_sum(s[hh], 0, lsum[hh]);
        pb[hh][1] = pack8_sum(s[hh], 1, lsum[hh]);
      }
    }
    // O^T += V^T P^T : A = V^T (lane <-> d, contraction over the block's 32 keys)
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const bf16x8 a = frag_tr<D>(vt_lds, to, kb * 32 + t * 16, db);
#pragma unroll
        for (int hh = 0; hh < NH; ++hh) o[hh][db] = mfma32(a, pb[hh][t], o[hh][db]);
      }
  }
}

// Tile that carries a bitmask: 32-key blocks that none of the wave's 32 rows can see are left out (of a row tile's
// chain blocks a wave sees one or two of four; the second half of a diagonal depth-0 tile is often in the future of the
// whole row tile), and the heads are taken one after the other, which needs fewer registers than fwd_tile.  Three of a
// row tile's tiles are of this kind: at L = 1,391, K = 8 (14 tiles per row tile on average) the forward takes 183
// instead of 199 us, at L = 4,096 in four segments 1,236 instead of 1,269.
template <int D, int NH, bool SAFE>
__device__ __forceinline__ void fwd_tile_masked(const char* kt_lds, const char* vt_lds, const NatOff<D>& no, const TrOff<D>& to,
                                                const bf16x8 (&qf)[NH][D / 16], f32x16 (&o)[NH][D / 32], float (&m)[NH],
                                                float (&lsum)[NH], const uint32_t (&mw)[2], float c) {
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    if (!wave_sees_block(mw[kb])) continue;
#pragma unroll
    for (int hh = 0; hh < NH; ++hh) {
      f32x16 s = zero16();
#pragma unroll
      for (int st = 0; st < D / 16; ++st) s = mfma32(frag_nat<D>(kt_lds, no, kb, st), qf[hh][st], s);
      bf16x8 pb[2];
      if (SAFE) {
        softmax_block<D / 32, true, kLag>(s, mw[kb], c, m[hh], lsum[hh], o[hh], pb);
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = exp2_fast(mask_sel(s[i], mw[kb], 8 * (i / 4) + (i % 4)) * c);
        pb[0] = pack8_sum(s, 0, lsum[hh]);
        pb[1] = pack8_sum(s, 1, lsum[hh]);
      }
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int t = 0; t < 2; ++t) o[hh][db] = mfma32(frag_tr<D>(vt_lds, to, kb * 32 + t * 16, db), pb[t], o[hh][db]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// PER_SIMD: workgroups per CU, which registers and LDS both allow.
template <int D, int NH, bool SV, int PER_SIMD>
__global__ __launch_bounds__(256, PER_SIMD) void fwd_kernel(FwdParams p) {
  // Two heads in three workgroups per CU leave 168 registers: what only masked tiles and the last stores need is computed there.
  constexpr bool LEAN = NH == 2 && PER_SIMD == 3;
  constexpr int kTileBytes = kKeysPerTile * D * 2;
  constexpr bool kChainFirst = D == 64;
  // (Four workgroups per CU have two buffers, 37 KB in all: of two chain tiles the first then stands in the buffer that the first
  // tile of depth-0 keys is copied to while the second is computed.)
  constexpr bool kTwoBufs = kChainFirst && PER_SIMD == 4;
  constexpr int kBufs = kChainFirst && !kTwoBufs ? 3 : 2;
  __shared__ __attribute__((aligned(16))) char lds[kBufs][2][kTileBytes];  // [buffer][K|V]
  __shared__ __attribute__((aligned(16))) char lds_mask[kChainFirst ? 4 : 2][kTileMaskBytes];  // of buffers 0 and 1, of the chain tiles

  const int tid = threadIdx.x, wave = LEAN ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6, lane = tid & 63, g = lane >> 5, ln = lane & 31;
  const KeyTileLds<D> kl(&lds[0][0][0], wave);
  const uint32_t mask_lds = lds_scalar_addr(&lds_mask[0][0]);
  const DeviceTileMap& tm = p.tm;
  int kvh = blockIdx.x;
  int hc = split_by(kvh, p.by_kv);
  const int rt = p.rt_hi - 1 - split_by(hc, p.by_heads);  // heaviest row tiles first
  const int h0 = kvh * p.group + hc * NH;

  // The start of a workgroup is a chain of memory round trips - parameters, list bounds, entries, copies; tokens, rows -, and
  // with short lists the other workgroups of the CU do not cover it.  What does not depend on one another is on its way
  // together, here and in the backward's kernels: lookups go through the scalar path (a vector load that is waited for waits
  // for the rows' loads before it), several at a time, and the rows are loaded without a branch for each.  us per step, one by
  // one / so, 64 heads: packed 203 to 517 anchors 322 / 304, 203 to 900 745 / 713, eight packed sequences 3,111 / 3,056,
  // L = 1,391 713 / 709; long lists the same (L = 4,096 4,931 / 4,924, L = 20,480 109.1 / 109.0 ms).
  const int e0 = const_int(tm.row_ptr, rt), e_end = const_int(tm.row_ptr, rt + 1);
  const int e_lead = e0 + const_int(tm.row_lead, rt);  // end of the leading run of full tiles
  const int r = wave * 32 + ln;  // row of the tile owned by this lane (shared with lane^32)
  int tq_held;
  const bool row_ok = row_token(tm, rt, r, p.L, tq_held);

  // (A row that does not exist computes on token 0's: a lane's row meets no other lane's, and it is not stored.)
  bf16x8 qf[NH][D / 16];
  auto load_q = [&]() {
    const __bf16* q = p.q + ((size_t)(row_ok ? tq_held : 0) * p.Hq + h0) * D + g * 8;
#pragma unroll
    for (int hh = 0; hh < NH; ++hh)
#pragma unroll
      for (int st = 0; st < D / 16; ++st) qf[hh][st] = as_frag(ld16(q + hh * D + st * 16));
  };

  f32x16 o[NH][D / 32];
  float m[NH], lsum[NH], l_tot[NH];
  const NatOff<D> no = nat_offsets<D>(lane);
  const TrOff<D> to = tr_offsets<D>(lane);

  auto copy_tile = [&](int buf, int kt) {
    if (kChainFirst) dma_d0_tile<D, 4>(kl.k(buf), kl.v(buf), p.k, p.v, p.Hkv, kvh, kt, p.L, wave, lane);
    else dma_key_tile<D, 4, SV>(kl.k(buf), kl.v(buf), p.k, p.v, p.Hkv, kvh, tm, kt, p.L, wave, lane, p.v_shared);
  };

  // One pass over the row tile's key tiles.  The first pass keeps the softmax reference at 0
  // (no running max: fewer vector instructions per score); it is exact as long as every row
  // sum stays inside the fp32 / bf16 exponent range.  If any row of a head leaves [2^-100, 2^100]
  // (or is not finite) the tile is recomputed with the running-max form, for that head alone: the
  // workgroup's other head keeps its first pass, so that a head's results do not depend on which
  // heads share its workgroup.
  auto pass = [&](auto safe_tag) {
    constexpr bool SAFE = decltype(safe_tag)::value;
#pragma unroll
    for (int hh = 0; hh < NH; ++hh) {
      m[hh] = SAFE ? kNegInit : 0.f;
      lsum[hh] = 0.f;
#pragma unroll
      for (int db = 0; db < D / 32; ++db) o[hh][db] = zero16();
    }
    ChainTiles ch{};
    if (kChainFirst) ch = chain_tiles(tm, e0, e_end);
    const int e1 = e_end - ch.n;  // (the chain tiles come first)
    TileEntry cur = const_entry(tm.row_entries, e0);
    TileEntry nxt = const_entry(tm.row_entries, e0 + 1 < e_end ? e0 + 1 : e0);
    TileEntry masked = const_entry(tm.row_entries, e_lead < e_end ? e_lead : e0);
    if (e_lead >= e1) masked.mask_id = -1;
    if (!SAFE || LEAN) load_q();  // (lean: not held over the stores of the first pass)
    const bool first_waits = kTwoBufs && ch.n == 2;
    const int chain_buf = first_waits ? 0 : 1;
    if (kChainFirst) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (i < ch.n) {
          dma_chain_tile<D, 4, SV>(kl.k(chain_buf + i), kl.v(chain_buf + i), p.k, p.v, p.Hkv, kvh, tm, ch.tile[i].tile, p.L, wave,
                                   LEAN ? lane_id() : lane, p.v_shared);
          dma_tile_mask(mask_lds + (2 + i) * kTileMaskBytes, tm, ch.tile[i], wave);
        }
    }
    if (!first_waits) copy_tile(0, cur.tile);
    // (The first bitmask, if there is one, travels with the first tile, to where its own tile finds it: the loop over full tiles
    // then has no test for one in front of its matrix instructions.  With the test / without, CU busy cycles of 10,816 anchors
    // at D = 128 3.13e9 / 3.09e9; us of 20,480 anchors 23,720 / 23,600.  Not so in dq_item: 4.48e9 / 4.50e9 cycles.)
    dma_tile_mask(mask_lds + ((e_lead - e0) & 1) * kTileMaskBytes, tm, masked, wave);
    dma_publish();
    if (kChainFirst && ch.n > 0) {
      const int l = LEAN ? lane_id() : lane;
#pragma unroll 1
      for (int i = 0; i < ch.n; ++i) {
        if (first_waits && i == 1) {
          __syncthreads();  // buffer 0 may be overwritten
          copy_tile(0, cur.tile);
        }
        uint32_t mw[2];
        tile_mask(lds_mask[2 + i], wave * 32 + (l & 31), l >> 5, mw);
        fwd_tile_masked<D, NH, SAFE>(lds[chain_buf + i][0], lds[chain_buf + i][1], no, to, qf, o, m, lsum, mw, p.c_log2);
      }
      // buffer 1 may be overwritten (two buffers: and tile e0 has landed)
      if (kTwoBufs) dma_publish();
      else __syncthreads();
    }
    // A row tile's list holds its full tiles first, then the partial ones: two loops (accumulators stay in place).
    int e = e0;
    auto full_tile = [&](int buf) {
      const u32x2 ahead = fetch_entry(tm.row_entries, e + 2 < e1 ? e + 2 : e);
      if (e + 1 < e1)
        copy_tile(buf ^ 1, nxt.tile);
      const uint32_t mw[2] = {0xffffffffu, 0xffffffffu};
      fwd_tile<D, NH, false, SAFE>(lds[buf][0], lds[buf][1], no, to, qf, o, m, lsum, mw, p.c_log2);
      dma_publish();
      cur = nxt;
      nxt = take_entry(ahead);
      ++e;
    };
    // (two at a time with the buffer index a constant: every LDS address is then a per-lane register plus an
    // immediate, which saves the eight vector additions per tile that a buffer index in a register costs)
    while (e + 1 < e_lead) {
      full_tile(0);
      full_tile(1);
    }
    if (e < e_lead) full_tile(0);
    for (; e < e1; ++e) {
      const int buf = (e - e0) & 1;
      const u32x2 ahead = fetch_entry(tm.row_entries, e + 2 < e1 ? e + 2 : e);
      if (e + 1 < e1) {
        copy_tile(buf ^ 1, nxt.tile);
        dma_tile_mask(mask_lds + (buf ^ 1) * kTileMaskBytes, tm, nxt, wave);
      }
      const int l = LEAN ? lane_id() : lane;
      uint32_t mw[2];
      tile_mask(lds_mask[buf], wave * 32 + (l & 31), l >> 5, mw);
      fwd_tile_masked<D, NH, SAFE>(lds[buf][0], lds[buf][1], no, to, qf, o, m, lsum, mw, p.c_log2);
      dma_publish();
      cur = nxt;
      nxt = take_entry(ahead);
    }
#pragma unroll
    for (int hh = 0; hh < NH; ++hh) l_tot[hh] = sum_halves(lsum[hh]);
  };
  auto store = [&](int hh) {
    const float inv = 1.0f / l_tot[hh];
    const int l = LEAN ? lane_id() : lane, g = l >> 5;
    int tq = tq_held;
    if (LEAN ? row_token(tm, rt, wave * 32 + (l & 31), p.L, tq) : row_ok) {
      const size_t off = ((size_t)tq * p.Hq + h0 + hh) * D;
      const float lse = (m[hh] + __builtin_log2f(l_tot[hh])) * kLn2;
      if (p.d_o) {  // the backward follows in the same call: leave its per-row terms, in the form it consumes
        bf16x8 dof[D / 16];
#pragma unroll
        for (int st = 0; st < D / 16; ++st) dof[st] = as_frag(ld16(p.d_o + off + st * 16 + g * 8));
        float dl = 0.f;
#pragma unroll
        for (int st = 0; st < D / 16; ++st) {
          const u32x4 w = row_piece_bf16(o[hh][st / 2], st % 2, inv);
          *reinterpret_cast<u32x4*>(p.o + off + st * 16 + g * 8) = w;
          dl = add_delta8(dl, dof[st], __builtin_bit_cast(bf16x8, w));
        }
        dl = sum_halves(dl);
        if (g == 0) {
          p.delta[(size_t)(h0 + hh) * p.T + tq] = -dl;
          p.nlse[(size_t)(h0 + hh) * p.T + tq] = -(lse * kLog2e) / p.c_log2;
        }
      } else {
#pragma unroll
        for (int db = 0; db < D / 32; ++db) store_row_bf16(p.o + off + db * 32, o[hh][db], inv, g);
      }
      if (g == 0) p.lse[(size_t)(h0 + hh) * p.T + tq] = lse;
    }
  };
  pass(std::false_type{});
  int bad = 0;  // a bit per head
#pragma unroll
  for (int hh = 0; hh < NH; ++hh)
    if (row_ok && !(l_tot[hh] > 0x1p-100f && l_tot[hh] < 0x1p100f)) bad |= 1 << hh;
  int redo = 0;
  if (__syncthreads_or(bad)) {
#pragma unroll
    for (int hh = 0; hh < NH; ++hh) redo |= (NH == 1 || __syncthreads_or(bad & (1 << hh))) ? 1 << hh : 0;
  }
#pragma unroll
  for (int hh = 0; hh < NH; ++hh)
    if (!(redo & (1 << hh))) store(hh);
  if (redo) {
    pass(std::true_type{});
#pragma unroll
    for (int hh = 0; hh < NH; ++hh)
      if (redo & (1 << hh)) store(hh);
  }
}

// =====================================================================================
// Backward, part 1: Delta = rowsum(dO * O) and dQ = scale * dS K, row-tile owned (same
// decomposition as the forward).  Writes Delta [Hq, T] for part 2.
// =====================================================================================
// |lse| up to which (log2 units) the D = 64 kernels leave a row's probabilities unnormalised, see dq_pipe_kernel.
constexpr float kDqLseRange = 64.f;

// FROM_DELTA: -Delta is the start value of the dP sum, as in dq_pipe_body, instead of being subtracted at its end.
template <int D, int NH, bool MASKED, bool FROM_DELTA = false>
__device__ __forceinline__ void dq_tile(const char* kt_lds, const char* vt_lds, const NatOff<D>& no, const TrOff<D>& to,
                                        const bf16x8 (&qf)[NH][D / 16], const bf16x8 (&dof)[NH][D / 16],
                                        f32x16 (&dq)[NH][D / 32], const float (&lse2)[NH], const float (&delta)[NH],
                                        const uint32_t (&mw)[2], float c) {
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    // A 32-key block of a masked tile that none of the wave's 32 rows can see contributes exact zeros and is left out
    // (see fwd_tile_masked).
    if (MASKED && !wave_sees_block(mw[kb])) continue;
    f32x16 s[NH], dp[NH];
#pragma unroll
    for (int hh = 0; hh < NH; ++hh) {
      s[hh] = zero16();
#pragma unroll
      for (int i = 0; i < 16; ++i) dp[hh][i] = FROM_DELTA ? -delta[hh] : 0.f;
    }
#pragma unroll
    for (int st = 0; st < D / 16; ++st) {
      const bf16x8 ak = frag_nat<D>(kt_lds, no, kb, st);
      const bf16x8 av = frag_nat<D>(vt_lds, no, kb, st);
#pragma unroll
      for (int hh = 0; hh < NH; ++hh) {
        s[hh] = mfma32(ak, qf[hh][st], s[hh]);     // S^T  = K Q^T
        dp[hh] = mfma32(av, dof[hh][st], dp[hh]);  // dP^T = V dO^T
      }
    }
    bf16x8 dsb[NH][2];
#pragma unroll
    for (int hh = 0; hh < NH; ++hh) {
      const float nl = -lse2[hh], dl = delta[hh];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        float pr = exp2_fast(__builtin_fmaf(s[hh][i], c, nl));
        if (MASKED) pr = mask_zero(pr, mw[kb], 8 * (i / 4) + (i % 4));
        s[hh][i] = pr * (FROM_DELTA ? dp[hh][i] : dp[hh][i] - dl);
      }
      dsb[hh][0] = pack8(s[hh], 0);
      dsb[hh][1] = pack8(s[hh], 1);
    }
    // dQ^T += K^T dS^T : A = K^T (lane <-> d, contraction over the block's keys)
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const bf16x8 a = frag_tr<D>(kt_lds, to, kb * 32 + t * 16, db);
#pragma unroll
        for (int hh = 0; hh < NH; ++hh) dq[hh][db] = mfma32(a, dsb[hh][t], dq[hh][db]);
      }
  }
}

// (One query head per workgroup.  This plain form serves D = 128, and at D = 64 launches of many workgroups with short
// lists, where three per CU cover one another's first loads and last stores; the others run dq_pipe_kernel below.  At
// D = 64 it does the arithmetic of dq_pipe_kernel step for step - unnormalised probabilities where that kernel leaves
// them so, -Delta as the start value of dP in the tiles which that kernel pipelines - so that a row's dQ has the same
// bits from either and the launcher may choose freely.  NH stays a named constant because dq_tile is written for NH
// heads sharing the K / V fragments.)
// TERMS: as in dq_pipe_item.
template <int D>
constexpr int kDqLds = (D == 64 ? 3 : 2) * 2 * kKeysPerTile * D * 2 + (D == 64 ? 4 : 2) * kTileMaskBytes;
template <int D, bool SV, bool TERMS>
__device__ __forceinline__ void dq_item(const BwdParams& p, char* lds_base, int b) {
  constexpr int NH = 1;
  constexpr int kTileBytes = kKeysPerTile * D * 2;
  constexpr bool kAsPipe = D == 64;
  constexpr bool kChainFirst = D == 64;
  constexpr int kBufs = kChainFirst ? 3 : 2, kMasks = kChainFirst ? 4 : 2;  // (see fwd_kernel)
  char (&lds)[kBufs][2][kTileBytes] = *reinterpret_cast<char (*)[kBufs][2][kTileBytes]>(lds_base);  // [buffer][K|V]
  char (&lds_mask)[kMasks][kTileMaskBytes] = *reinterpret_cast<char (*)[kMasks][kTileMaskBytes]>(lds_base + sizeof(lds));

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, g = lane >> 5, ln = lane & 31;
  const KeyTileLds<D> kl(&lds[0][0][0], wave);
  const uint32_t mask_lds = lds_scalar_addr(&lds_mask[0][0]);
  const DeviceTileMap& tm = p.tm;
  static_assert(NH == 1, "by_group counts workgroups of one head");
  int kvh = b;
  int hc = split_by(kvh, p.by_kv);
  const int rt = p.rt_hi - 1 - split_by(hc, p.by_group);
  const int h0 = kvh * p.group + hc;

  const int e0 = const_int(tm.row_ptr, rt), e_end = const_int(tm.row_ptr, rt + 1);  // (see fwd_kernel)
  const int e_lead = e0 + const_int(tm.row_lead, rt);  // end of the leading run of full tiles
  const int r = wave * 32 + ln;
  int tq;
  const bool row_ok = row_token(tm, rt, r, p.L, tq);
  ChainTiles ch{};
  if (kChainFirst) ch = chain_tiles(tm, e0, e_end);
  const int e1 = e_end - ch.n;  // (the chain tiles come first)
  TileEntry cur = const_entry(tm.row_entries, e0);
  TileEntry nxt = const_entry(tm.row_entries, e0 + 1 < e_end ? e0 + 1 : e0);

  bf16x8 qf[NH][D / 16], dof[NH][D / 16], of[NH][D / 16];
  float lse2[NH], delta[NH];
#pragma unroll
  for (int hh = 0; hh < NH; ++hh) {
    const size_t off = ((size_t)(row_ok ? tq : 0) * p.Hq + h0 + hh) * D + g * 8;
    lse2[hh] = p.lse[(size_t)(h0 + hh) * p.T + (row_ok ? tq : 0)] * kLog2e;
    if (!TERMS) delta[hh] = -p.delta[(size_t)(h0 + hh) * p.T + (row_ok ? tq : 0)];
#pragma unroll
    for (int st = 0; st < D / 16; ++st) {
      qf[hh][st] = as_frag(ld16(p.q + off + st * 16));
      dof[hh][st] = as_frag(ld16(p.d_o + off + st * 16));
      if (TERMS) of[hh][st] = as_frag(ld16(p.o + off + st * 16));
    }
  }
  auto copy_tile = [&](int buf, int kt) {
    if (kChainFirst) dma_d0_tile<D, 4>(kl.k(buf), kl.v(buf), p.k, p.v, p.Hkv, kvh, kt, p.L, wave, lane);
    else dma_key_tile<D, 4, SV>(kl.k(buf), kl.v(buf), p.k, p.v, p.Hkv, kvh, tm, kt, p.L, wave, lane, p.v_shared);
  };
  if (kChainFirst) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (i < ch.n) {
        dma_chain_tile<D, 4, SV>(kl.k(1 + i), kl.v(1 + i), p.k, p.v, p.Hkv, kvh, tm, ch.tile[i].tile, p.L, wave, lane, p.v_shared);
        dma_tile_mask(mask_lds + (2 + i) * kTileMaskBytes, tm, ch.tile[i], wave);
      }
  }
  copy_tile(0, cur.tile);
  dma_tile_mask(mask_lds, tm, cur, wave);
#pragma unroll
  for (int hh = 0; TERMS && hh < NH; ++hh) {
    float dl = 0.f;
#pragma unroll
    for (int st = 0; st < D / 16; ++st) dl = add_delta8(dl, dof[hh][st], of[hh][st]);
    dl = sum_halves(dl);
    delta[hh] = dl;
    if (row_ok && g == 0) {  // per-row terms in the form the dK/dV kernel consumes
      p.delta[(size_t)(h0 + hh) * p.T + tq] = -dl;
      p.nlse[(size_t)(h0 + hh) * p.T + tq] = -lse2[hh] / p.c_log2;
    }
  }

  f32x16 dq[NH][D / 32];
#pragma unroll
  for (int hh = 0; hh < NH; ++hh)
#pragma unroll
    for (int db = 0; db < D / 32; ++db) dq[hh][db] = zero16();

  const NatOff<D> no = nat_offsets<D>(lane);
  const TrOff<D> to = tr_offsets<D>(lane);

  float row_factor = p.scale;
  int e_pipe = e0;  // end of the tiles that dq_pipe_kernel would run in its pipeline
  if (kAsPipe) {    // (see there; lse2 is not needed unchanged from here on)
    const bool unnormalised = __syncthreads_or(row_ok && !(__builtin_fabsf(lse2[0]) <= kDqLseRange)) == 0;
    if (unnormalised) {
      row_factor = exp2_fast(-lse2[0]) * p.scale;
      lse2[0] = 0.f;
      e_pipe = e0 + (e_lead - e0) / 3 * 3;
    }
  }
  dma_publish();
  if (kChainFirst && ch.n > 0) {
#pragma unroll 1
    for (int i = 0; i < ch.n; ++i) {
      uint32_t mw[2];
      tile_mask(lds_mask[2 + i], r, g, mw);
      dq_tile<D, NH, true>(lds[1 + i][0], lds[1 + i][1], no, to, qf, dof, dq, lse2, delta, mw, p.c_log2);
    }
    __syncthreads();  // buffer 1 may be overwritten
  }

  int e = e0;
  auto full_tiles = [&](int e_end, auto from_delta_tag) {  // leading full tiles: counted loop, no mask branch
    constexpr bool FROM_DELTA = decltype(from_delta_tag)::value;
    for (; e < e_end; ++e) {
      const int buf = (e - e0) & 1;
      const u32x2 ahead = fetch_entry(tm.row_entries, e + 2 < e1 ? e + 2 : e);
      if (e + 1 < e1) {
        copy_tile(buf ^ 1, nxt.tile);
        dma_tile_mask(mask_lds + (buf ^ 1) * kTileMaskBytes, tm, nxt, wave);
      }
      const uint32_t mw[2] = {0xffffffffu, 0xffffffffu};
      dq_tile<D, NH, false, FROM_DELTA>(lds[buf][0], lds[buf][1], no, to, qf, dof, dq, lse2, delta, mw, p.c_log2);
      dma_publish();
      cur = nxt;
      nxt = take_entry(ahead);
    }
  };
  if (kAsPipe) full_tiles(e_pipe, std::true_type{});
  full_tiles(e_lead, std::false_type{});
  for (; e < e1; ++e) {
    const int buf = (e - e0) & 1;
    const u32x2 ahead = fetch_entry(tm.row_entries, e + 2 < e1 ? e + 2 : e);
    if (e + 1 < e1) {
      copy_tile(buf ^ 1, nxt.tile);
      dma_tile_mask(mask_lds + (buf ^ 1) * kTileMaskBytes, tm, nxt, wave);
    }
    uint32_t mw[2];
    tile_mask(lds_mask[buf], r, g, mw);
    dq_tile<D, NH, true>(lds[buf][0], lds[buf][1], no, to, qf, dof, dq, lse2, delta, mw, p.c_log2);
    dma_publish();
    cur = nxt;
    nxt = take_entry(ahead);
  }

  if (row_ok) {
    if (p.rope_table) {
      // q was the rotated copy: turn dQ back.  The lane holds features db*32 + 8*q4 + 4g + j of its
      // row, so both members of every pair (feature, feature + D/2) are in its own registers.
      const float* rope = p.rope_table + (size_t)token_position(tm, tq, p.L) * D;
#pragma unroll
      for (int db = 0; db < D / 64; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int d0 = db * 32 + 8 * q4 + 4 * g;
          const f32x4 cs = *reinterpret_cast<const f32x4*>(rope + d0);
          const f32x4 sn = *reinterpret_cast<const f32x4*>(rope + D / 2 + d0);
#pragma unroll
          for (int hh = 0; hh < NH; ++hh) {
            f32x4 lo, hi;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              lo[j] = dq[hh][db][4 * q4 + j];
              hi[j] = dq[hh][db + D / 64][4 * q4 + j];
            }
            rope_turn4<true>(lo, hi, cs, sn);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              dq[hh][db][4 * q4 + j] = lo[j];
              dq[hh][db + D / 64][4 * q4 + j] = hi[j];
            }
          }
        }
    }
#pragma unroll
    for (int hh = 0; hh < NH; ++hh) {
      __bf16* drow = p.dq + ((size_t)tq * p.Hq + h0 + hh) * D;
#pragma unroll
      for (int db = 0; db < D / 32; ++db) store_row_bf16(drow + db * 32, dq[hh][db], row_factor, g);
    }
  }
}

template <int D, bool SV>
__global__ __launch_bounds__(256, 2) void dq_kernel(BwdParams p) {
  __shared__ __attribute__((aligned(16))) char lds[kDqLds<D>];
  dq_item<D, SV, true>(p, lds, blockIdx.x);
}

// =====================================================================================
// Backward, part 1 with the leading full tiles of a row tile run as one software pipeline (D = 64; same
// decomposition and results layout as dq_kernel).  The unit of work is a 32-key block, two per key tile.
// A wave that issues a matrix instruction and then independent vector instructions runs the vector work
// in the shadow of the matrix pipe, whereas matrix and vector phases that follow one another - in one wave
// or in several waves of a SIMD - take the sum of their times (see dkdv_rowtile_pipelined).  So while the
// vector unit turns the scores of unit u into dS, the matrix pipe runs dQ += K^T dS of unit u-1 and S, dP
// of unit u+1, across key-tile boundaries: three K/V buffers rotate (tile e of the row tile's list lives in
// buffer e % 3; the pipelined tiles are taken three at a time so that every LDS address is a per-lane
// register plus an immediate), the copy of tile e+2 is issued when every wave has left tile e-1, and one
// barrier per tile - between its two units - both frees that buffer and publishes tile e+1.
//
// Per-row terms cost no vector instruction here: -Delta is the accumulator input of the first dP
// instruction (sixteen equal registers per lane, lane <-> row), and the probabilities are left
// unnormalised, p' = 2^(c s), the factor 2^(-lse) being applied to the row's dQ once at the end.  That is
// exact as long as 2^(c s) cannot leave the fp32 range, which |lse| <= 64 (log2 units) guarantees for
// every key of the row; a workgroup with a row outside that range (or a non-finite lse) takes the plain
// routine with the normalised probabilities for all its tiles.
// Tiles that carry a bitmask (the chain tiles, which are taken first, from the buffer the pipeline reaches last and one
// more, and the diagonal tiles that end a row tile's list) and the up to two full tiles left over by the groups of three go
// through dq_tile.
// =====================================================================================
constexpr int kDqAhead = 2;

template <int D>
struct DqPipe {
  f32x16 sc[2], dpc[2];     // S and dP of the units in flight (index = 32-key block of the unit's tile)
  u32x4 dsb[2][2];          // dS of a unit as bf16 B operands, per 16-key step
  bf16x8 ring[kDqAhead];    // A operands on their way from LDS
};

// A operand of matrix instruction j of a unit's body: first the D/16 transposed K fragments of the unit whose
// dQ is due (j = 16-key step * D/32 + feature block), then the D/8 natural fragments of the unit whose S / dP
// start (even: K, odd: V).
template <int D>
__device__ __forceinline__ bf16x8 dq_pipe_frag(const char* k_dq, int kb_dq, const char* k_s, const char* v_s, int kb_s,
                                               const NatOff<D>& no, const TrOff<D>& to, int j) {
  constexpr int N2 = D / 16;
  if (j < N2) return frag_tr<D>(k_dq, to, kb_dq * 32 + (j / (D / 32)) * 16, j % (D / 32));
  const int i = j - N2;
  return frag_nat<D>((i & 1) ? v_s : k_s, no, kb_s, i >> 1);
}

// Body of the unit (tile e, block KB): its vector work rides on the matrix instructions dQ of the unit before
// it (block 1-KB of k_dq: tile e-1 for KB = 0, tile e for KB = 1) and, unless LAST, S / dP of the unit after it
// (block 1-KB of k_s, v_s: tile e for KB = 0, tile e+1 for KB = 1).  k_self is K of tile e: the next body's
// dQ fragments (this unit's) are prefetched from it.
template <int D, int KB, bool LAST>
__device__ __forceinline__ void dq_pipe_body(DqPipe<D>& P, const char* k_dq, const char* k_s, const char* v_s,
                                             const char* k_self, const NatOff<D>& no, const TrOff<D>& to,
                                             const bf16x8 (&qf)[1][D / 16], const bf16x8 (&dof)[1][D / 16],
                                             f32x16 (&dq)[1][D / 32], const f32x16& ndelta16, float c) {
  constexpr int N2 = D / 16, NM = LAST ? N2 : N2 + D / 8, O = 1 - KB;
  static_assert(N2 % kDqAhead == 0 && (D / 8) % kDqAhead == 0, "fragment slots must repeat from body to body");
#pragma unroll
  for (int j = 0; j < NM; ++j) {
    const int slot = j % kDqAhead;
    const bf16x8 a = P.ring[slot];
    if (j < N2) {
      dq[0][j % (D / 32)] = mfma32(a, __builtin_bit_cast(bf16x8, P.dsb[O][j / (D / 32)]), dq[0][j % (D / 32)]);
    } else {
      const int i = j - N2, st = i >> 1;
      if (i & 1) P.dpc[O] = mfma32(a, dof[0][st], st == 0 ? ndelta16 : P.dpc[O]);
      else P.sc[O] = mfma32(a, qf[0][st], st == 0 ? zero16() : P.sc[O]);
    }
    if (j + kDqAhead < NM) {
      P.ring[slot] = dq_pipe_frag<D>(k_dq, O, k_s, v_s, O, no, to, j + kDqAhead);
    } else {
      const int jn = j + kDqAhead - NM;
      P.ring[slot] = frag_tr<D>(k_self, to, KB * 32 + (jn / (D / 32)) * 16, jn % (D / 32));
    }
    // Vector work of the unit, skewed by one matrix instruction: p' = 2^(c s) of a few scores here, their
    // products with dP and the rounding to bf16 behind the next instruction, so that neighbouring vector
    // instructions do not depend on one another (registers <-> keys 8*(i/4) + 4g + i%4 of the block).
    // The empty assembly statements keep each value's computation where it is written: without them the
    // compiler moves it to the first use, which for dS is the next body.
    if (j > 0) {
#pragma unroll
      for (int i = 16 * (j - 1) / (NM - 1); i < 16 * j / (NM - 1); ++i) {
        P.sc[KB][i] *= P.dpc[KB][i];
        if (i & 1) {
          uint32_t w = pack_bf16(P.sc[KB][i - 1], P.sc[KB][i]);
          asm volatile("" : "+v"(w));
          P.dsb[KB][i >> 3][(i & 7) >> 1] = w;
        }
      }
    }
    if (j + 1 < NM) {
#pragma unroll
      for (int i = 16 * j / (NM - 1); i < 16 * (j + 1) / (NM - 1); ++i) {
        float e = exp2_fast(P.sc[KB][i] * c);
        asm volatile("" : "+v"(e));
        P.sc[KB][i] = e;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// TERMS: forms the per-row terms from O and writes them for the dK/dV kernel; otherwise they are there already.
template <int D>
constexpr int kDqPipeLds = 4 * 2 * kKeysPerTile * D * 2 + 5 * kTileMaskBytes;
template <int D, bool SV, bool TERMS>
__device__ __forceinline__ void dq_pipe_item(const BwdParams& p, char* lds_base, int b) {
  constexpr int kTileBytes = kKeysPerTile * D * 2;
  constexpr int N2 = D / 16;
  char (&lds)[4][2][kTileBytes] = *reinterpret_cast<char (*)[4][2][kTileBytes]>(lds_base);  // [buffer][K|V]
  const char* lds_mask = lds_base + sizeof(lds);                                                      // [buffer], then the chain tiles'

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, g = lane >> 5, ln = lane & 31;
  const KeyTileLds<D> kl(&lds[0][0][0], wave);
  const uint32_t mask_lds = lds_scalar_addr(lds_mask);
  const DeviceTileMap& tm = p.tm;
  int kvh = b;
  int hc = split_by(kvh, p.by_kv);
  const int rt = p.rt_hi - 1 - split_by(hc, p.by_group);  // heaviest row tiles first
  const int h = kvh * p.group + hc;

  const int e0 = const_int(tm.row_ptr, rt), e_end = const_int(tm.row_ptr, rt + 1);  // (see fwd_kernel)
  const int n_lead = const_int(tm.row_lead, rt);  // leading full tiles
  const int r = wave * 32 + ln;  // row of the tile owned by this lane (shared with lane ^ 32)
  int tq;
  const bool row_ok = row_token(tm, rt, r, p.L, tq);
  const ChainTiles ch = chain_tiles(tm, e0, e_end);
  const int e1 = e_end - ch.n;  // (the chain tiles come first)
  auto entry_at = [&](int e) { return e < e_end ? e : e_end - 1; };
  TileEntry t_cur = const_entry(tm.row_entries, e0);
  TileEntry t_n1 = const_entry(tm.row_entries, entry_at(e0 + 1));
  TileEntry t_n2 = const_entry(tm.row_entries, entry_at(e0 + 2));
  const TileEntry masked0 = const_entry(tm.row_entries, entry_at(e0 + n_lead));  // the first two with a bitmask, if there are any
  const TileEntry masked1 = const_entry(tm.row_entries, entry_at(e0 + n_lead + 1));

  bf16x8 qf[1][D / 16], dof[1][D / 16], of[D / 16];
  const size_t at = (size_t)h * p.T + (row_ok ? tq : 0);
  float lse2 = p.lse[at] * kLog2e, delta = TERMS ? 0.f : -p.delta[at];
  {
    const size_t off = ((size_t)(row_ok ? tq : 0) * p.Hq + h) * D + g * 8;
#pragma unroll
    for (int st = 0; st < D / 16; ++st) {
      qf[0][st] = as_frag(ld16(p.q + off + st * 16));
      dof[0][st] = as_frag(ld16(p.d_o + off + st * 16));
      if (TERMS) of[st] = as_frag(ld16(p.o + off + st * 16));
    }
  }

  // the first two tiles are on their way before anything is computed, and the first two bitmasks, to where their tiles find them:
  // the pipeline then has no test for one (with / without, us: 20,480 anchors 34,970 / 34,780, 8,000 5,690 / 5,657)
  dma_d0_tile<D, 4>(kl.k(0), kl.v(0), p.k, p.v, p.Hkv, kvh, t_cur.tile, p.L, wave, lane);
  if (e0 + 1 < e1) dma_d0_tile<D, 4>(kl.k(1), kl.v(1), p.k, p.v, p.Hkv, kvh, t_n1.tile, p.L, wave, lane);
  dma_tile_mask(mask_lds + n_lead % 3 * kTileMaskBytes, tm, masked0, wave);
  dma_tile_mask(mask_lds + (n_lead + 1) % 3 * kTileMaskBytes, tm, masked1, wave);
#pragma unroll
  for (int i = 0; i < 2; ++i)
    if (i < ch.n) {
      dma_chain_tile<D, 4, SV>(kl.k(2 + i), kl.v(2 + i), p.k, p.v, p.Hkv, kvh, tm, ch.tile[i].tile, p.L, wave, lane, p.v_shared);
      dma_tile_mask(mask_lds + (3 + i) * kTileMaskBytes, tm, ch.tile[i], wave);
    }

  if (TERMS) {
    float dl = 0.f;
#pragma unroll
    for (int st = 0; st < D / 16; ++st) dl = add_delta8(dl, dof[0][st], of[st]);
    delta = sum_halves(dl);
    if (row_ok && g == 0) {  // per-row terms in the form the dK/dV kernel consumes
      p.delta[at] = -delta;
      p.nlse[at] = -lse2 / p.c_log2;
    }
  }

  f32x16 dq[1][D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db) dq[0][db] = zero16();

  const NatOff<D> no = nat_offsets<D>(lane);
  const TrOff<D> to = tr_offsets<D>(lane);
  // unnormalised probabilities for the whole workgroup, or normalised ones for the whole workgroup
  const bool in_range = __builtin_fabsf(lse2) <= kDqLseRange;  // (false for NaN)
  const bool unnormalised = __syncthreads_or(row_ok && !in_range) == 0;
  const float lse_used[1] = {unnormalised ? 0.f : lse2};
  const float delta_used[1] = {delta};
  const float row_factor = (unnormalised ? exp2_fast(-lse2) : 1.f) * p.scale;
  const int n_groups = unnormalised ? n_lead / 3 : 0;  // groups of three pipelined tiles

  dma_publish();  // tiles e0 and e0+1 have landed, and the chain tiles
#pragma unroll 1
  for (int i = 0; i < ch.n; ++i) {
    uint32_t mw[2];
    tile_mask(lds_mask + (3 + i) * kTileMaskBytes, r, g, mw);
    dq_tile<D, 1, true>(lds[2 + i][0], lds[2 + i][1], no, to, qf, dof, dq, lse_used, delta_used, mw, p.c_log2);
  }
  __syncthreads();  // buffer 2 may be overwritten
  if (n_groups > 0) {
    // The K half of the buffer that the first pipelined body reads its (absent) predecessor from: that body multiplies it by
    // dS = 0, so it only has to be finite.
    uint4* z = reinterpret_cast<uint4*>(lds[2][0]);
    for (int i = tid; i < kTileBytes / 16; i += 256) z[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
  }
  int e = e0;

  if (n_groups > 0) {
    f32x16 ndelta16;
#pragma unroll
    for (int i = 0; i < 16; ++i) ndelta16[i] = -delta;
    const float c = p.c_log2;
    DqPipe<D> P;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int t = 0; t < 2; ++t) P.dsb[a][t] = u32x4{0, 0, 0, 0};
    {  // S and dP of the first unit; nothing to overlap them with
      P.sc[0] = zero16();
      P.dpc[0] = ndelta16;
#pragma unroll
      for (int st = 0; st < D / 16; ++st) {
        P.sc[0] = mfma32(frag_nat<D>(lds[0][0], no, 0, st), qf[0][st], P.sc[0]);
        P.dpc[0] = mfma32(frag_nat<D>(lds[0][1], no, 0, st), dof[0][st], P.dpc[0]);
      }
#pragma unroll
      for (int j = 0; j < kDqAhead; ++j) P.ring[j] = dq_pipe_frag<D>(lds[2][0], 1, lds[0][0], lds[0][1], 1, no, to, j);
    }
    // One key tile in buffer B (a compile-time constant).
    auto tile = [&](auto buf_tag, auto last_tag) {
      constexpr int B = decltype(buf_tag)::value, BP = (B + 2) % 3, BN = (B + 1) % 3;
      constexpr bool LAST = decltype(last_tag)::value;
      const u32x2 ahead = fetch_entry(tm.row_entries, entry_at(e + 3));
      dq_pipe_body<D, 0, false>(P, lds[BP][0], lds[B][0], lds[B][1], lds[B][0], no, to, qf, dof, dq, ndelta16, c);
      // Every wave has left tile e-1 (its last reader was the body above) and has waited for its own copies of
      // tile e+1: after the barrier that buffer may be overwritten and tile e+1 may be read.
      dma_publish();
      if (e + 2 < e1) dma_d0_tile<D, 4>(kl.k(BP), kl.v(BP), p.k, p.v, p.Hkv, kvh, t_n2.tile, p.L, wave, lane);
      dq_pipe_body<D, 1, LAST>(P, lds[B][0], lds[BN][0], lds[BN][1], lds[B][0], no, to, qf, dof, dq, ndelta16, c);
      t_cur = t_n1;
      t_n1 = t_n2;
      t_n2 = take_entry(ahead);
      ++e;
    };
    using B0 = std::integral_constant<int, 0>;
    using B1 = std::integral_constant<int, 1>;
    using B2 = std::integral_constant<int, 2>;
    for (int gi = 0; gi < n_groups - 1; ++gi) {
      tile(B0{}, std::false_type{});
      tile(B1{}, std::false_type{});
      tile(B2{}, std::false_type{});
    }
    tile(B0{}, std::false_type{});
    tile(B1{}, std::false_type{});
    tile(B2{}, std::true_type{});  // starts no further unit
    // dQ of the last unit (block 1 of the tile in buffer 2)
#pragma unroll
    for (int j = 0; j < N2; ++j) {
      const bf16x8 a = j < kDqAhead ? P.ring[j] : frag_tr<D>(lds[2][0], to, 32 + (j / (D / 32)) * 16, j % (D / 32));
      dq[0][j % (D / 32)] = mfma32(a, __builtin_bit_cast(bf16x8, P.dsb[1][j / (D / 32)]), dq[0][j % (D / 32)]);
    }
    // tiles e and e+1 have been copied (e+1 perhaps not yet published), and a wave may still be reading tile e-1
    dma_publish();
  }

  // The remaining tiles, one barrier each: tile e sits in buffer (e - e0) % 3, tile e+1 is published, the
  // copy of tile e+2 goes to the buffer tile e-1 has left.
  int buf = 0;  // (e - e0) % 3: the pipelined part ends on a multiple of three
  auto plain = [&](int e_end, auto masked_tag) {
    constexpr bool MASKED = decltype(masked_tag)::value;
    for (; e < e_end; ++e) {
      const u32x2 ahead = fetch_entry(tm.row_entries, entry_at(e + 3));
      const int buf2 = buf == 0 ? 2 : buf - 1;
      if (e + 2 < e1) {
        dma_d0_tile<D, 4>(kl.k(buf2), kl.v(buf2), p.k, p.v, p.Hkv, kvh, t_n2.tile, p.L, wave, lane);
        if (MASKED) dma_tile_mask(mask_lds + buf2 * kTileMaskBytes, tm, t_n2, wave);
      }
      const char* kt_lds = lds[0][0] + buf * (2 * kTileBytes);
      const char* vt_lds = kt_lds + kTileBytes;
      uint32_t mw[2] = {0xffffffffu, 0xffffffffu};
      if (MASKED) tile_mask(lds_mask + buf * kTileMaskBytes, r, g, mw);
      dq_tile<D, 1, MASKED>(kt_lds, vt_lds, no, to, qf, dof, dq, lse_used, delta_used, mw, p.c_log2);
      dma_publish();
      t_cur = t_n1;
      t_n1 = t_n2;
      t_n2 = take_entry(ahead);
      buf = buf == 2 ? 0 : buf + 1;
    }
  };
  plain(e0 + n_lead, std::false_type{});  // full tiles left over
  plain(e1, std::true_type{});            // the tiles that carry a bitmask end the list

  if (row_ok) {
    if (p.rope_table) {
      // q was the rotated copy: turn dQ back.  The lane holds features db*32 + 8*q4 + 4g + j of its
      // row, so both members of every pair (feature, feature + D/2) are in its own registers.
      const float* rope = p.rope_table + (size_t)token_position(tm, tq, p.L) * D;
#pragma unroll
      for (int db = 0; db < D / 64; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int d0 = db * 32 + 8 * q4 + 4 * g;
          const f32x4 cs = *reinterpret_cast<const f32x4*>(rope + d0);
          const f32x4 sn = *reinterpret_cast<const f32x4*>(rope + D / 2 + d0);
          f32x4 lo, hi;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            lo[j] = dq[0][db][4 * q4 + j];
            hi[j] = dq[0][db + D / 64][4 * q4 + j];
          }
          rope_turn4<true>(lo, hi, cs, sn);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            dq[0][db][4 * q4 + j] = lo[j];
            dq[0][db + D / 64][4 * q4 + j] = hi[j];
          }
        }
    }
    __bf16* drow = p.dq + ((size_t)tq * p.Hq + h) * D;
#pragma unroll
    for (int db = 0; db < D / 32; ++db) store_row_bf16(drow + db * 32, dq[0][db], row_factor, g);
  }
}

template <int D>
__global__ __launch_bounds__(256, 2) void dq_pipe_kernel(BwdParams p) {
  __shared__ __attribute__((aligned(16))) char lds[kDqPipeLds<D>];
  dq_pipe_item<D, false, true>(p, lds, blockIdx.x);
}

// =====================================================================================
// Backward, part 2: dK, dV, key-tile owned.  A workgroup holds a PAIR of adjacent key tiles
// (128 keys) of one KV head in registers and loops over the row tiles that see the first of
// them (clipped to the segment) for the query heads [h_lo, h_hi) assigned to it; the second
// tile's list is a suffix of the first's, so its waves idle on the few leading row tiles.
// Wave w owns key block w (32 keys) and all 128 rows of each row tile.
//   depth-0 key tiles: one query head per workgroup, result to the per-head partial buffer;
//   chain key tiles:   all heads of the KV group, result straight to dk_acc / dv_acc.
// =====================================================================================
// ---- one row tile (128 rows of one query head) against the wave's 32 keys, as one software pipeline ----
// MODE 0: every element visible; 1: key-major bitmask; 2: every element visible except for lanes whose key
// belongs to another sequence of a packed batch (lane_off = true): those lanes contribute nothing.
//
// On this chip a wave that issues a matrix instruction and then independent vector instructions runs the
// vector work in the shadow of the matrix pipe (about four plain vector instructions per
// v_mfma_f32_32x32x16_bf16 cost nothing), whereas matrix and vector phases that follow one another - in the
// same wave or in two waves of one SIMD - take the sum of their times.  The row tile's four 32-row units
// are therefore staggered: while the vector unit turns the scores of unit u into P and dS, the matrix
// pipe runs dV / dK of unit u-1 and S / dP of unit u+1.  The 8 groups of D/8 matrix instructions are
//   S,dP(0) | S,dP(1) | dV,dK(0) | S,dP(2) | dV,dK(1) | S,dP(3) | dV,dK(2) | dV,dK(3)
// and the vector work of units 0..3 rides on groups 1 | 2,3 | 4,5 | 6.  Every matrix instruction is
// followed by its share of vector instructions and a scheduling fence, so the interleaving written here
// is the one the hardware sees; operand fragments are fetched from LDS kPipeAhead instructions ahead.
struct PipeGroup {
  int kind;   // 0: S and dP of `unit`; 1: dV and dK of `unit`
  int unit;   // 32-row block of the row tile
  int vunit;  // unit whose vector work rides on this group (-1: none)
  int e0, e1; // ... and which of its 16 score registers
};
constexpr PipeGroup kPipeGroups[8] = {{0, 0, -1, 0, 0}, {0, 1, 0, 0, 16}, {1, 0, 1, 0, 8},  {0, 2, 1, 8, 16},
                                      {1, 1, 2, 0, 8},  {0, 3, 2, 8, 16}, {1, 2, 3, 0, 16}, {1, 3, -1, 0, 0}};
// (Fragments ahead, dK/dV of a step at D = 64, us: one 2,285, two 2,258, three 2,435 - spills.  At D = 128, with one wave per
// SIMD and room for more, L = 10,816: two 13,436, four 13,229; six against four 14,226 and 13,879 on another box.)
template <int D>
constexpr int kPipeAhead = D == 128 ? 4 : 2;
// The copies of the next row tile are issued one after every kCopyEvery-th matrix instruction.  Issued all together, each
// holds its wave for about 100 cycles (the address unit takes 1 KiB of copies in 25, and the other waves issue theirs at
// the same time): 17 copies at D = 128 were 2,085 of an iteration's 9,100 cycles, 9 at D = 64 1,275 of 6,400.  dK/dV, us,
// together / spread: D = 128 L = 10,816 14,650 / 13,820, L = 1,391 354 / 333, K = 7 L = 4,000 2,025 / 1,890; D = 64, where
// another wave of the SIMD covers most of it, L = 4,096 2,160 / 2,130, 4 heads (one workgroup per CU) L = 3,000 395 / 361.
// (Every third or sixth: the same within 0.5 %.)
constexpr int kCopyEvery = 4;

// f(0), f(1), .. f(N-1), the argument a compile-time constant.
template <int J, int N, class F>
__device__ __forceinline__ void unrolled(F&& f) {
  if constexpr (J < N) {
    f(std::integral_constant<int, J>{});
    unrolled<J + 1, N>(f);
  }
}

// The copies that a routine issues between its matrix instructions: none, or this wave's share of the next row tile.
struct NoCopies {
  template <int M>
  __device__ __forceinline__ void after() const {}
};
template <int D, bool WHOLE>
struct NextRowTile {
  const __bf16 *q, *d_o;           // the head's row of the tile's first anchor
  const float* stat;
  const RowDmaOffsets<D, 4>& ro;   // WHOLE: of copy 0 only, copy i reads i * step behind it
  uint32_t step;
  uint32_t dst, stat_dst;          // LDS
  bool last_ok, stat_ok;           // not WHOLE: the lane's row of the last copy, and of the statistic, exists
  const void* zeros;
  static constexpr int kPer = RowDmaLane<D, 4>::kPer;
  static constexpr int kCopies = 2 * kPer + 1;
  template <int C>
  __device__ __forceinline__ void issue() const {
    constexpr int i = C >> 1, kOff = (C & 1) * kRowsPerTile * D * 2 + i * 4096;
    const __bf16* base = C & 1 ? d_o : q;
    if constexpr (C == 2 * kPer) {
      if (WHOLE) dma4_untracked_at<0>(stat, ro.stat_off, stat_dst);
      else dma4_untracked(stat_ok ? (const void*)((const char*)stat + ro.stat_off) : zeros, stat_dst);
    } else if constexpr (WHOLE) {
      dma16_untracked_at<kOff>(base, ro.off[0] + i * step, dst);
    } else if constexpr (i < kPer - 1) {
      dma16_untracked_at<kOff>(base, ro.off[i], dst);
    } else {
      dma16_untracked(last_ok ? (const void*)((const char*)base + ro.off[i]) : zeros, dst + kOff);
    }
  }
  template <int M>
  __device__ __forceinline__ void after() const {  // behind matrix instruction M of the row tile
    if constexpr (M % kCopyEvery == 0 && M / kCopyEvery < kCopies) issue<M / kCopyEvery>();
  }
};

// The same for rows named by token lists.  A row that does not exist is read from the tile's last row and its -lse/scale of
// -infinity makes its probabilities zero: no copy of Q or dO has to choose between two addresses.  (Zero times a NaN of that
// row is a NaN: the last row, because a key that is taken with a unit of missing rows - chain keys at D = 64 are taken unit
// by unit - is taken with the last row's unit anyway.)  FAR: offsets past 4 GiB.  (dK/dV, us, with 64-bit addresses chosen
// per lane and the copies issued together at D = 64 / so: sampled 8,192 4,581 / 4,357, eight packed sequences 1,388 / 1,318;
// D = 128, riding before too, sampled 4,096 1,349 / 1,233, packed 1,556 / 1,417.)
template <int D, bool FAR>
struct NextListedRowTile {
  const __bf16 *q, *d_o;           // the head's row of token 0
  const float* stat;
  const RowTokens<D, 4>& t;
  const RowDmaLane<D, 4>& rl;
  uint32_t stride;                 // bytes from token to token
  uint32_t dst, stat_dst;
  const void* no_row;              // the statistic of a row that does not exist
  static constexpr int kPer = RowDmaLane<D, 4>::kPer;
  static constexpr int kCopies = 2 * kPer + 1;
  template <int C>
  __device__ __forceinline__ void issue() const {
    if constexpr (C == 2 * kPer) {
      dma4_untracked(t.stat_tok >= 0 ? (const void*)(stat + t.stat_tok) : no_row, stat_dst);
    } else {
      constexpr int i = C >> 1, kOff = (C & 1) * kRowsPerTile * D * 2 + i * 4096;
      const uint32_t tok = (uint32_t)(t.tok[i] ^ (t.tok[i] >> 31));
      const __bf16* base = C & 1 ? d_o : q;
      if constexpr (FAR) dma16_untracked((const char*)base + ((size_t)tok * stride + 2 * rl.chunk[i]), dst + kOff);
      else dma16_untracked_at<kOff>(base, tok * stride + 2 * rl.chunk[i], dst);
    }
  }
  template <int M>
  __device__ __forceinline__ void after() const {
    if constexpr (M % kCopyEvery == 0 && M / kCopyEvery < kCopies) issue<M / kCopyEvery>();
  }
};

template <int D>
struct DkdvPipe {
  f32x16 sc[2], dpc[2];        // S and dP accumulators of the units in flight (unit & 1)
  u32x4 pb[2][2], dsb[2][2];   // P and dS of a unit as bf16 B operands, per 16-row step
  bf16x8 ring[kPipeAhead<D>];  // A operands on their way from LDS
};

// A operand of matrix instruction j of a group: S / dP read natural fragments (even j: Q, odd j: dO),
// dV / dK transposed ones (even j: dO^T, odd j: Q^T; j/2 = 16-row step * D/32 + feature block).
template <int D, int KIND>
__device__ __forceinline__ bf16x8 pipe_frag(const char* q_lds, const char* do_lds, const NatOff<D>& no,
                                            const TrOff<D>& to, int r0, int j) {
  if (KIND == 0) return *reinterpret_cast<const bf16x8*>(((j & 1) ? do_lds : q_lds) + no.off[j >> 1] + r0 * (2 * D));
  const int idx = j >> 1, db = idx % (D / 32), tt = idx / (D / 32);
  return frag_tr<D>((j & 1) ? q_lds : do_lds, to, r0 + tt * 16, db);
}

// -lse/scale and -Delta of the unit's rows, straight into the accumulators S and dP start from (C layout).
template <int MODE>
__device__ __forceinline__ void pipe_row_terms(f32x16& s, f32x16& dp, const float* nlse_lds, const float* ndelta_lds,
                                               int r0, int g, bool lane_off) {
#pragma unroll
  for (int q4 = 0; q4 < 4; ++q4) {
    const f32x4 l4 = *reinterpret_cast<const f32x4*>(nlse_lds + r0 + 8 * q4 + 4 * g);
    const f32x4 d4 = *reinterpret_cast<const f32x4*>(ndelta_lds + r0 + 8 * q4 + 4 * g);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      s[4 * q4 + j] = MODE == 2 && lane_off ? -__builtin_inff() : l4[j];
      dp[4 * q4 + j] = d4[j];
    }
  }
}

// The vector work that the group table gives to matrix instruction M, in three stages a matrix instruction apart: scale,
// exponentiate (and mask), multiply with dP and round.  (All three behind the same matrix instruction, each waited for the one
// before it, and a no-op stood between exponential and product: dK/dV at D = 128, one wave per SIMD, L = 10,816 13,376 ->
// 13,072 us, L = 1,391 325 -> 317; D = 64 L = 4,096 2,046 -> 2,018, L = 20,480 46,720 -> 46,090, 4 heads L = 3,000 362 -> 342.)  The last
// two scores of a unit are finished behind the first two matrix instructions of the next group, which needs them only in
// its second half; a unit's per-row terms take the registers of the unit two before it after that.
template <int D, int MODE, int STAGE, int M>
__device__ __forceinline__ void dkdv_vector_work(DkdvPipe<D>& P, float c, const u32x4& cm) {
  constexpr int NG = D / 8;
  if constexpr (M >= 0) {
    constexpr PipeGroup gd = kPipeGroups[M / NG];
    if constexpr (gd.vunit >= 0) {
      constexpr int vu = gd.vunit & 1, j = M % NG, n = gd.e1 - gd.e0;
#pragma unroll
      for (int i = gd.e0 + n * j / NG; i < gd.e0 + n * (j + 1) / NG; ++i) {
        if (STAGE == 1) {
          P.sc[vu][i] *= c;
        } else if (STAGE == 2) {
          float pr = exp2_fast(P.sc[vu][i]);
          if (MODE == 1) {  // the lane's key-major mask word of this unit, shifted down by 4g: bit of row 8*(i/4) + 4g + i%4
            const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe((int)cm[gd.vunit & 3], 8 * (i / 4) + (i % 4), 1);
            pr = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, pr) & keep);
          }
          P.sc[vu][i] = pr;
        } else {
          P.dpc[vu][i] *= P.sc[vu][i];
          if (i & 1) {
            P.pb[vu][i >> 3][(i & 7) >> 1] = pack_bf16(P.sc[vu][i - 1], P.sc[vu][i]);
            P.dsb[vu][i >> 3][(i & 7) >> 1] = pack_bf16(P.dpc[vu][i - 1], P.dpc[vu][i]);
          }
        }
      }
    }
  }
}

template <int D, int MODE, int G, class Copies>
__device__ __forceinline__ void dkdv_pipe_group(const Copies& copies, DkdvPipe<D>& P, const char* q_lds, const char* do_lds,
                                                const float* nlse_lds, const float* ndelta_lds, const NatOff<D>& no,
                                                const TrOff<D>& to, const bf16x8 (&kf)[D / 16],
                                                const bf16x8 (&vf)[D / 16], f32x16 (&dk)[D / 32], f32x16 (&dv)[D / 32],
                                                int g, float c, bool lane_off, const u32x4& cm) {
  constexpr int NG = D / 8;  // matrix instructions per group
  constexpr PipeGroup gd = kPipeGroups[G];
  constexpr PipeGroup gn = kPipeGroups[G + 1 < 8 ? G + 1 : 7];
  constexpr int u = gd.unit & 1;
  unrolled<0, NG>([&](auto j_tag) {
    constexpr int j = decltype(j_tag)::value;
    const int slot = (G * NG + j) % kPipeAhead<D>;  // the instruction kPipeAhead<D> later takes the slot this one frees
    const bf16x8 a = P.ring[slot];
    if (gd.kind == 0) {
      if (j & 1) P.dpc[u] = mfma32(a, vf[j >> 1], P.dpc[u]);
      else P.sc[u] = mfma32(a, kf[j >> 1], P.sc[u]);
    } else {
      const int idx = j >> 1, db = idx % (D / 32), tt = idx / (D / 32);
      if (j & 1) dk[db] = mfma32(a, __builtin_bit_cast(bf16x8, P.dsb[u][tt]), dk[db]);
      else dv[db] = mfma32(a, __builtin_bit_cast(bf16x8, P.pb[u][tt]), dv[db]);
    }
    if (j + kPipeAhead<D> < NG)
      P.ring[slot] = pipe_frag<D, gd.kind>(q_lds, do_lds, no, to, gd.unit * 32, j + kPipeAhead<D>);
    else if (G + 1 < 8)
      P.ring[slot] = pipe_frag<D, gn.kind>(q_lds, do_lds, no, to, gn.unit * 32, j + kPipeAhead<D> - NG);
    constexpr int M = G * NG + j;
    // stage 3 before stage 2 before stage 1: neighbouring instructions do not depend on one another
    dkdv_vector_work<D, MODE, 3, M - 2>(P, c, cm);
    dkdv_vector_work<D, MODE, 2, M - 1>(P, c, cm);
    dkdv_vector_work<D, MODE, 1, M>(P, c, cm);
    if (j == 2 && G + 1 < 8 && gn.kind == 0)  // the next group starts S / dP of a unit: fetch its per-row terms now
      pipe_row_terms<MODE>(P.sc[gn.unit & 1], P.dpc[gn.unit & 1], nlse_lds, ndelta_lds, gn.unit * 32, g, lane_off);
    copies.template after<G * NG + j>();
    __builtin_amdgcn_sched_barrier(0);
  });
}

template <int D, int MODE, class Copies>
__device__ __forceinline__ void dkdv_rowtile_pipelined(const Copies& copies, const char* q_lds, const char* do_lds, const float* nlse_lds,
                                                       const float* ndelta_lds, const NatOff<D>& no, const TrOff<D>& to,
                                                       const bf16x8 (&kf)[D / 16], const bf16x8 (&vf)[D / 16],
                                                       f32x16 (&dk)[D / 32], f32x16 (&dv)[D / 32], int g, float c,
                                                       bool lane_off = false, const u32x4 cm = u32x4{0, 0, 0, 0}) {
  DkdvPipe<D> P;
  pipe_row_terms<MODE>(P.sc[0], P.dpc[0], nlse_lds, ndelta_lds, 0, g, lane_off);
#pragma unroll
  for (int j = 0; j < kPipeAhead<D>; ++j) P.ring[j] = pipe_frag<D, 0>(q_lds, do_lds, no, to, 0, j);
#define PEAGLE_PIPE_GROUP(G) \
  dkdv_pipe_group<D, MODE, G>(copies, P, q_lds, do_lds, nlse_lds, ndelta_lds, no, to, kf, vf, dk, dv, g, c, lane_off, cm)
  PEAGLE_PIPE_GROUP(0);
  PEAGLE_PIPE_GROUP(1);
  PEAGLE_PIPE_GROUP(2);
  PEAGLE_PIPE_GROUP(3);
  PEAGLE_PIPE_GROUP(4);
  PEAGLE_PIPE_GROUP(5);
  PEAGLE_PIPE_GROUP(6);
  PEAGLE_PIPE_GROUP(7);
#undef PEAGLE_PIPE_GROUP
}

// The same row tile against chain keys: rows and chain keys of a tile are ordered alike, so a wave's 32 keys are seen
// by one or two of the four 32-row units (cm: the lane's key-major mask words).  Those are taken one by one, without the
// pipeline above, which would run the matrix instructions of all four: an iteration is then bound by its copies
// (dK/dV of eight packed sequences of 64 to 1,728 anchors: the step 3,600 -> 3,460 us).
template <int D>
__device__ __forceinline__ void dkdv_rowtile_chain(const char* q_lds, const char* do_lds, const float* nlse_lds,
                                                   const float* ndelta_lds, const NatOff<D>& no, const TrOff<D>& to,
                                                   const bf16x8 (&kf)[D / 16], const bf16x8 (&vf)[D / 16],
                                                   f32x16 (&dk)[D / 32], f32x16 (&dv)[D / 32], int g, float c, u32x4 cm) {
#pragma unroll 1
  for (int u = 0; u < 4; ++u) {
    const uint32_t mw = cm[0] >> (4 * g);
    cm = u32x4{cm[1], cm[2], cm[3], 0u};
    if (!wave_sees_block(mw)) continue;
    const char* q = q_lds + u * (32 * 2 * D);
    const char* d_o = do_lds + u * (32 * 2 * D);
    f32x16 s, dp;
    pipe_row_terms<0>(s, dp, nlse_lds + u * 32, ndelta_lds + u * 32, 0, g, false);
#pragma unroll
    for (int st = 0; st < D / 16; ++st) {
      s = mfma32(frag_nat<D>(q, no, 0, st), kf[st], s);
      dp = mfma32(frag_nat<D>(d_o, no, 0, st), vf[st], dp);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe((int)mw, 8 * (i / 4) + (i % 4), 1);
      const float pr = exp2_fast(s[i] * c);
      s[i] = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, pr) & keep);
      dp[i] *= s[i];
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const bf16x8 pb = pack8(s, t), dsb = pack8(dp, t);
#pragma unroll
      for (int db = 0; db < D / 32; ++db) {
        dv[db] = mfma32(frag_tr<D>(d_o, to, t * 16, db), pb, dv[db]);
        dk[db] = mfma32(frag_tr<D>(q, to, t * 16, db), dsb, dk[db]);
      }
    }
  }
}

// How the rows of a row tile are found.
//   kRowsWhole, kRowsMost: dense map, tensors within reach of a 32-bit offset (RowDmaOffsets): every row tile but the
//     sequence's last holds the same rows, and the copies of the next one ride between the matrix instructions
//     (NextRowTile).  Whole: the rows a lane copies are a whole number of anchors apart (K divides kRowsApart, so that
//     A * K = 128): one per-lane offset and a scalar step address every copy.  Most: an offset per copy, and the last copy
//     of a tile holds the rows past A * K (A * K > 128 - kRowsApart).
//   kRowsFar: any other dense map - larger tensors, and the K whose tiles lack more rows than their last copies hold (D = 128:
//     22, 26 to 28, 33 to 37, 43 to 56, 65 to 112; D = 64: 43 to 48, 65 to 96); tokens are computed when a copy is issued, and
//     none rides.
//     (Step of 4 heads, D = 128, in the loops of before copies rode / now: K = 33 957 / 920 us, K = 20, Most, 832 / 710.)
//   kRowsListed, kRowsListedFar: the map names rows by explicit token lists (sampled / packed maps); their tokens are
//     fetched an iteration before the copy that uses them, and the copies ride too (NextListedRowTile).
// (A near loop that carried every row's token and anchor as the far one does reloaded spilled registers behind its own
// copies, and waited for them: dK/dV at L = 4,096 2,226 us, now 2,152.)
enum { kRowsWhole = 0, kRowsFar = 1, kRowsListed = 2, kRowsMost = 3, kRowsListedFar = 4 };
template <int D>
constexpr int kRowsApart = 4 * (512 / D);  // rows of the tile between two copies of a lane
// Partials of a set: dK (which = 0) or dV.
__device__ __forceinline__ float* part_of(const BwdParams& p, int set, int which) {
  return set == 0 ? (which ? p.dv_part : p.dk_part) : p.part_more + (size_t)(2 * (set - 1) + which) * p.part_stride;
}
template <int D>
constexpr int kDkdvLds = 2 * (2 * kRowsPerTile * D * 2 + 2 * kRowsPerTile * 4 + 2 * kMaskWords * 4);  // see kBufBytes
template <int D, int ROWS, bool SV>
__device__ __forceinline__ void dkdv_item(const BwdParams& p, char* lds, const int item) {
  constexpr bool LISTED = ROWS == kRowsListed || ROWS == kRowsListedFar;
  // Blocks that no row sees are left out at D = 64.  At D = 128, with one wave per SIMD, nothing covers the unpipelined
  // chain routine, and the second loop costs the first: dK/dV at 1,391 anchors 378 us with both, 338 with one pipelined
  // loop for all tiles, at 3,000 anchors 1,410 and 1,320.
  constexpr bool kSkips = D == 64;
  constexpr int kTileBytes = kRowsPerTile * D * 2;
  constexpr int kMaskAt = 2 * kTileBytes + 2 * kRowsPerTile * 4;  // Q | dO | lse2 | delta | masks of the pair's key tiles
  constexpr int kBufBytes = kMaskAt + 2 * kMaskWords * 4;
  constexpr int kLdsBytes = kDkdvLds<D>;

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, g = lane >> 5, ln = lane & 31;
  const int kblk = wave;  // 32-key block of the pair owned by this wave
  const DeviceTileMap& tm = p.tm;
  const int group = p.group;

  // the item's range (field by field: a struct chosen as a whole is copied through scratch memory)
  auto of_range = [&](int DkdvRange::* field, int n) {
    int x = p.range[0].*field;
#pragma unroll
    for (int i = 1; i < n; ++i) x = item >= p.range[i].first_item ? p.range[i].*field : x;
    return x;
  };
  auto range_of_item = [&](auto n_tag) {
    constexpr int n = decltype(n_tag)::value;
    using R = DkdvRange;
    return R{of_range(&R::rt_lo, n),     of_range(&R::rt_hi, n),      of_range(&R::s_lo, n),     of_range(&R::s_hi, n),
             of_range(&R::clip_rows, n), of_range(&R::d0_tile_lo, n), of_range(&R::n_d0_tiles, n), of_range(&R::d0_split, n),
             of_range(&R::d0_step, n),   of_range(&R::first_item, n), of_range(&R::set, n)};
  };
  DkdvRange rg = range_of_item(std::integral_constant<int, 1>{});
  if (item >= p.range[1].first_item) rg = range_of_item(std::integral_constant<int, kMaxRanges>{});
  int b = item - rg.first_item;
  int kt0, n_tiles, kvh, h_lo, h_hi;  // first key tile of the pair, tiles present (1 or 2)
  const bool chain = item >= p.n_d0_items;
  if (!chain) {
    // Workgroups are dealt round-robin to the XCDs, so b % Hkv pins a KV head to an XCD's L2;
    // within it the key-tile pairs of one query head are adjacent, so the workgroups that are
    // resident together stream the same head's Q / dO rows and share them in L2.
    // The pairs are dealt in passes over the heads: pass 0 takes the pairs [0, d0_split), each later
    // pass the next d0_step pairs.  The key tiles inside a segment have lists that shrink with the
    // pair index, and starting the long lists of every head before the short ones lets the short
    // ones fill the slots that free up (one pass - d0_split = pair count - when all lists are
    // equally long).
    const int n_pairs = (rg.n_d0_tiles - rg.d0_tile_lo + 1) / 2;
    kvh = b;
    b = split_by(kvh, p.by_kv);
    int first = 0, count = rg.d0_split;
    while (b >= count * group) {  // at most a few passes
      b -= count * group;
      first += count;
      count = n_pairs - first < rg.d0_step ? n_pairs - first : rg.d0_step;
    }
    const int head = b / count;  // (a division: count is the pass's)
    const int pair = first + b - head * count;
    kt0 = rg.d0_tile_lo + 2 * pair;
    h_lo = kvh * group + head;
    h_hi = h_lo + 1;
    n_tiles = kt0 + 1 < rg.n_d0_tiles ? 2 : 1;
  } else {
    rg.rt_lo = p.rt_lo;
    rg.rt_hi = p.rt_hi;
    rg.s_lo = p.s_lo;
    rg.s_hi = p.s_hi;
    rg.clip_rows = p.clip_rows;
    b = item - p.n_d0_items;
    kvh = b;
    b = split_by(kvh, p.by_kv);  // (a row tile has at most two chain tiles: one pair)
    kt0 = tm.n_d0 + (p.rt_lo + b) * tm.n_csub;
    n_tiles = tm.n_csub;
    h_lo = kvh * group;
    h_hi = h_lo + group;
  }
  const int my_tile = kblk >> 1;             // which tile of the pair this wave's keys belong to
  const int kt = kt0 + my_tile;
  const bool tile_present = my_tile < n_tiles;

  // row tiles that see a key tile, clipped to [rt_lo, rt_hi): the map stores where each segment
  // starts inside a key tile's (ascending) list.  A launch that covers only part of its segments
  // (a cropped length, or one chunk of a segment) cuts the range further by position: the row tiles
  // of a list are consecutive in a dense map, and in a listed one that is run in chunks (the
  // builder looks, see peagle_tilemap::rows_follow).
  // (All of it wave-uniform and looked up through the scalar path, both tiles of the pair and the first entries at a time: the
  // start of a workgroup is a chain of memory round trips, see fwd_kernel.)
  auto clip = [&](int t, int& lo_out, int& hi_out) {
    const int32_t* sp = tm.key_seg_ptr + (size_t)t * (tm.S + 1);
    int lo = const_int(sp, rg.s_lo), hi = const_int(sp, rg.s_hi);
    if (rg.clip_rows && lo < hi) {
      const int first = const_entry(tm.key_entries, lo).tile;
      const int nlo = lo + (rg.rt_lo > first ? rg.rt_lo - first : 0);
      const int nhi = lo + (rg.rt_hi > first ? rg.rt_hi - first : 0);
      lo = nlo < hi ? nlo : hi;
      hi = nhi < hi ? nhi : hi;
    }
    lo_out = lo;
    hi_out = hi;
  };
  int e_lo, e_hi;            // list of the pair's first tile: drives the loop
  clip(kt0, e_lo, e_hi);
  int e_lo1 = e_lo, e_hi1 = e_hi;  // ... and of its second
  if (n_tiles == 2) clip(kt0 + 1, e_lo1, e_hi1);
  const int my_keys_end = (kt + 1) * kKeysPerTile - 1;  // (depth-0 tiles: a row tile from this anchor on sees all of the wave's tile)
  const bool second = my_tile == 1 && tile_present;
  const int my_lo = second ? e_lo1 : e_lo, my_hi = second ? e_hi1 : e_hi;
  const int n_row_tiles = e_hi - e_lo;
  const int my_skip = tile_present ? n_row_tiles - (my_hi - my_lo) : n_row_tiles;  // leading row tiles that do not see my tile
  const int n_iter = n_row_tiles * (h_hi - h_lo);

  // stationary K, V of this wave's 32 keys: B operands (lane <-> key, registers <-> d)
  bf16x8 kf[D / 16], vf[D / 16];
  int key_tok = 0;
  const bool key_ok = tile_present && key_token(tm, kt, (kblk & 1) * 32 + ln, p.L, key_tok);
  // first key of the wave (anchor; meaningful for depth-0 tiles only)
  const int key0 = __builtin_amdgcn_readfirstlane(kt * kKeysPerTile + (kblk & 1) * 32);
  f32x16 dk[D / 32], dv[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db) {
    dk[db] = zero16();
    dv[db] = zero16();
  }

  const NatOff<D> no = nat_offsets<D>(lane);
  const TrOff<D> to = tr_offsets<D>(lane);

  // Q / dO row tiles and their per-row terms (-lse/scale, -Delta, prepared by the dQ kernel) go
  // straight from global memory into the LDS buffer that the next iteration reads.
  using Toks = RowTokens<D, 4>;
  RowDmaLane<D, 4> rl;
  RowDmaOffsets<D, 4> ro;
  constexpr bool kWhole = ROWS == kRowsWhole, kNear = kWhole || ROWS == kRowsMost;
  if (kNear) ro = row_dma_offsets<D, 4>(tm, p.L, wave, lane, p.Hq);
  else rl = row_dma_lane<D, 4>(tm, p.L, wave, lane);
  // Everything but the per-lane offset is computed on the scalar unit from values forced wave-uniform (the
  // compiler otherwise carries the row tile and head in vector registers and builds each copy's 64-bit
  // address there): LDS addresses are plain integers from the buffer's base, the source pointers scalar
  // multiplies and adds, and the choice between the forms is made once, not per copy.
  const uint32_t lds_addr0 = lds_scalar_addr(lds);
  const uint32_t wave_s = (uint32_t)__builtin_amdgcn_readfirstlane(wave);
  // (Held behind a statement the compiler cannot look through.  Left to itself it selects which of the two parameters to load,
  // and loads it in the loop, in the middle of a row tile, where the wait for a scalar load waits for every LDS read in flight:
  // 10,816 anchors of D = 128 13,540 / 13,410 us, CU busy cycles 1.8 % fewer; 4,096 anchors 2,189 / 2,175.)
  const float* stat_src = wave_s < 2 ? p.nlse : p.delta;
  auto no_stat = wave_s < 2 ? tm.no_row : tm.zeros;  // of a row that a listed tile lacks
  asm volatile("" : "+s"(stat_src));
  if (LISTED) asm volatile("" : "+s"(no_stat));
  constexpr int kPer = RowDmaLane<D, 4>::kPer;
  const int full_rows = tm.A * tm.K;  // rows of every tile but the sequence's last
  const uint32_t tile_bytes = (uint32_t)(tm.A * p.Hq * D * 2);  // from a row tile's first anchor to the next one's
  const uint32_t copy_step = kWhole ? (uint32_t)(kRowsApart<D> / tm.K * p.Hq * D * 2) : 0u;
  auto next_rows = [&](int hh, int rt, int buf) {
    const int hh_s = __builtin_amdgcn_readfirstlane(hh), rt_s = __builtin_amdgcn_readfirstlane(rt);
    // (near rows: every offset into these tensors fits 32 bits)
    const uint32_t row0 = (uint32_t)rt_s * tile_bytes + (uint32_t)hh_s * (D * 2);
    const uint32_t stat0 = ((uint32_t)hh_s * (uint32_t)p.T + (uint32_t)rt_s * (uint32_t)tm.A) * 4u;
    const uint32_t at = lds_addr0 + (uint32_t)buf * kBufBytes;
    uint32_t step = copy_step;  // (behind a statement: formed before the loop, the copies' offsets fill registers that the loop lacks)
    asm volatile("" : "+s"(step));
    return NextRowTile<D, kWhole>{
        (const __bf16*)((const char*)p.q + row0), (const __bf16*)((const char*)p.d_o + row0), (const float*)((const char*)stat_src + stat0), ro,
        step, at + wave_s * 1024,
        at + 2 * kTileBytes + (wave_s < 2 ? 0 : kRowsPerTile * 4) + (wave_s & 1) * 64 * 4,
        kRowsPerTile - kRowsApart<D> + (int)wave_s * (512 / D) + lane / (D / 8) < full_rows,
        (int)(wave_s & 1) * 64 + lane < full_rows, tm.zeros};
  };
  // rows are ordered anchor by anchor: those that exist are the first rows_of()
  auto rows_of = [&](int rt) {
    const int left = p.L - __builtin_amdgcn_readfirstlane(rt) * tm.A;
    return (left < tm.A ? left : tm.A) * tm.K;
  };
  auto issue_near = [&](int hh, int rt, int buf) {
    const auto n = next_rows(hh, rt, buf);
    const int n_valid = rows_of(rt);
    if (n_valid == full_rows) {
      unrolled<0, n.kCopies>([&](auto c) { n.template issue<decltype(c)::value>(); });
      return;
    }
    // (the last row tile of the sequence: only the copies that hold rows past n_valid need per-lane addresses, which take
    // those rows from the zero page)
    const int row = (int)wave_s * (512 / D) + lane / (D / 8);
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const uint32_t off = kWhole ? ro.off[0] + i * n.step : ro.off[i];
      if ((int)(i * 4 + wave_s + 1) * (512 / D) <= n_valid) {
        dma16_untracked(n.q, off, n.dst + i * 4 * 1024);
        dma16_untracked(n.d_o, off, n.dst + kTileBytes + i * 4 * 1024);
      } else {
        const bool ok = row + i * kRowsApart<D> < n_valid;
        dma16_untracked(ok ? (const void*)((const char*)n.q + off) : tm.zeros, n.dst + i * 4 * 1024);
        dma16_untracked(ok ? (const void*)((const char*)n.d_o + off) : tm.zeros, n.dst + kTileBytes + i * 4 * 1024);
      }
    }
    const bool ok = (int)(wave_s & 1) * 64 + lane < n_valid;
    dma4_untracked(ok ? (const void*)((const char*)n.stat + ro.stat_off) : tm.zeros, n.stat_dst);
  };
  auto next_listed = [&](int hh, const Toks& t, int buf) {
    const int hh_s = __builtin_amdgcn_readfirstlane(hh);
    const uint32_t at = lds_addr0 + (uint32_t)buf * kBufBytes;
    return NextListedRowTile<D, ROWS == kRowsListedFar>{
        p.q + (size_t)hh_s * D, p.d_o + (size_t)hh_s * D, stat_src + (size_t)hh_s * p.T, t, rl,
        (uint32_t)p.Hq * (D * 2), at + wave_s * 1024,
        at + 2 * kTileBytes + (wave_s < 2 ? 0 : kRowsPerTile * 4) + (wave_s & 1) * 64 * 4, no_stat};
  };
  auto issue = [&](int hh, const Toks& t, int buf) {
    if (LISTED) {
      const auto n = next_listed(hh, t, buf);
      unrolled<0, n.kCopies>([&](auto c) { n.template issue<decltype(c)::value>(); });
      return;
    }
    char* base = lds + buf * kBufBytes;
    dma_row_tile<D, 4>(base, p.q, p.Hq, hh, tm, rl, t, wave);
    dma_row_tile<D, 4>(base + kTileBytes, p.d_o, p.Hq, hh, tm, rl, t, wave);
    float* stat = reinterpret_cast<float*>(base + 2 * kTileBytes);
    if (wave < 2) dma_row_stat<D, 4>(stat, p.nlse, p.T, hh, tm, t, wave & 1);
    else if (wave < 4) dma_row_stat<D, 4>(stat + kRowsPerTile, p.delta, p.T, hh, tm, t, wave & 1);
  };
  // Iteration `it` handles row tile ei = it % n_row_tiles of head h_lo + it / n_row_tiles.  The
  // pipeline runs three deep: the list entry of iteration it+3 is fetched now and moved to scalar
  // registers after the barrier; the row tokens of it+2 are fetched now (they need that
  // iteration's row tile); the copy of it+1 is issued now; the mask of it+2 is fetched now.  Key-
  // side mask ids: -1 every element visible, >= 0 a bitmask, INT_MIN nothing to do (a row tile
  // that does not see this wave's key tile; also set by the map for row tiles listed only for the
  // other tile of the pair), other ids <= -2 visible for keys with anchor >= -id - 2 (the row
  // tile's sequence starts inside the key tile).
  // The list is walked from its last row tile down: every key tile of a launch ends at the same
  // row tile, so workgroups of one head that start together then read the same Q / dO rows at the
  // same time (they share them in L2) whether their lists are long or short.
  auto list_pos = [&](int ei) { return n_row_tiles - 1 - ei; };
  auto fetch_row_tile = [&](int ei) { return fetch_entry(tm.key_entries, e_lo + list_pos(ei)); };
  // (The row tiles of a dense map's list follow one another, and their place says whether they carry a bitmask: of the list only
  // the ids of bitmasks are looked up in the loop, 30 to 45 instructions fewer an iteration with the offsets in 32 bits.  us per
  // step, from the list / so: L = 4,096 4,841 / 4,811, first-layer form L = 3,891 4,641 / 4,632, 4 heads L = 1,000 141.2 / 139.6,
  // 32 heads at D = 128 L = 1,000 445 / 440, L = 10,816 31,520 / 31,420; the same: listed maps, which keep their lists, and at D = 128 K = 5 and 7, two of
  // whose registers moved to accumulation registers, dK/dV of 32 heads L = 1,391 220 / 218 and 301 / 300.)
  auto whole_tile = [&](int rt) { return !LISTED && !chain && rt * tm.A >= my_keys_end; };
  auto mask_pos = [&](int ei) {
    const int li = list_pos(ei);
    return li >= my_skip ? my_lo + li - my_skip : e_lo + li;
  };
  auto fetch_mask = [&](int ei) { return fetch_entry(tm.key_entries, mask_pos(ei)); };
  constexpr int kSkip = INT_MIN;
  auto mask_of = [&](int ei, const TileEntry& en) {  // (wave-uniform: through readfirstlane so that it stays scalar)
    return list_pos(ei) >= my_skip ? en.mask_id : kSkip;
  };
  auto step = [&](int& ei, int& hh) {  // advance (ei, hh) by one iteration
    if (++ei == n_row_tiles) {
      ei = 0;
      ++hh;
    }
  };

  // The key-major bitmask of a row tile, if it has one, travels with its copies (see dma_tile_mask): one wave of each key tile
  // copies it.
  auto issue_mask = [&](int mask, int buf) {
    const int id = __builtin_amdgcn_readfirstlane(mask);
    if (id < 0 || (wave_s & 1)) return;
    dma16_untracked(uniform_ptr(tm.masks_by_key + (size_t)id * kMaskWords), lane_id() * 16u,
                    lds_addr0 + (uint32_t)buf * kBufBytes + kMaskAt + (wave_s >> 1) * (kMaskWords * 4));
  };
  auto key_mask = [&](int buf) {  // the lane's key: four words, one per 32-row unit
    return *reinterpret_cast<const u32x4*>(lds + buf * kBufBytes + kMaskAt + (my_tile * kKeysPerTile + (kblk & 1) * 32 + ln) * 16);
  };

  int ei_n = 0, hh_n = h_lo;        // iteration it+1 (its copy is issued now)
  int ei_a = 0, hh_a = h_lo;        // it+2 (its row tokens and mask are fetched now)
  int ei_b = 0, hh_b = h_lo;        // it+3 (its list entry is fetched now)
  int rt_n = 0, rt_a = 0, rt_top = 0, mask_c = kSkip, mask_n = kSkip;
  Toks tok_n{};
  if (n_iter > 0) {
    step(ei_n, hh_n);
    step(ei_a, hh_a);
    step(ei_a, hh_a);
    step(ei_b, hh_b);
    step(ei_b, hh_b);
    step(ei_b, hh_b);
    auto mask_entry = [&](int ei) { return const_entry(tm.key_entries, __builtin_amdgcn_readfirstlane(mask_pos(ei))); };
    const int rt0 = const_entry(tm.key_entries, e_lo + list_pos(0)).tile;
    rt_top = rt0;
    const TileEntry m0 = mask_entry(0), m1 = mask_entry(ei_n);
    rt_n = LISTED ? const_entry(tm.key_entries, e_lo + list_pos(ei_n)).tile : rt0 - ei_n;
    rt_a = LISTED ? const_entry(tm.key_entries, e_lo + list_pos(ei_a)).tile : rt0 - ei_a;
    mask_c = mask_of(0, m0);
    if (n_iter > 1) mask_n = mask_of(ei_n, m1);
    if (kNear) {
      issue_near(h_lo, rt0, 0);
    } else {
      tok_n = row_tokens<D, 4, LISTED>(tm, rl, rt0, p.L);
      Toks tok_1 = tok_n;
      if (LISTED) tok_1 = row_tokens<D, 4, LISTED>(tm, rl, rt_n, p.L);
      issue(h_lo, tok_n, 0);
      tok_n = tok_1;
    }
    issue_mask(mask_c, 0);
  }
  {  // (behind the first row tile's copies; a key that does not exist computes on token 0's: a lane's key meets no other lane's,
     // and what it leaves is not stored, in the first-layer form counts as zero, and among the partials is not summed)
    const size_t off = ((size_t)(key_ok ? key_tok : 0) * p.Hkv + kvh) * D + g * 8;
    const __bf16* vrow = SV && chain ? p.v_shared + (size_t)kvh * D + g * 8 : p.v + off;
#pragma unroll
    for (int st = 0; st < D / 16; ++st) {
      kf[st] = as_frag(ld16(p.k + off + st * 16));
      vf[st] = as_frag(ld16(vrow + st * 16));
    }
  }
  dma_publish();

  auto run = [&](auto chain_tag) {
    constexpr bool CHAIN = decltype(chain_tag)::value;
    for (int it = 0; it < n_iter; ++it) {
      if (D == 128) {
        // K and V of the wave's keys stay in accumulation registers, where the matrix instructions read them directly.
        // (Left to itself the compiler puts them there too, but copies four registers before each use.)
#pragma unroll
        for (int st = 0; st < D / 16; ++st) {
          u32x4 a = __builtin_bit_cast(u32x4, kf[st]), b = __builtin_bit_cast(u32x4, vf[st]);
          asm volatile("" : "+a"(a), "+a"(b));
          kf[st] = __builtin_bit_cast(bf16x8, a);
          vf[st] = __builtin_bit_cast(bf16x8, b);
        }
      }
      const int buf = it & 1;
      const bool have1 = it + 1 < n_iter;
      // Does the routine of this iteration issue the next one's copies itself?  At D = 64 (depth-0 keys; a second body
      // per mode costs spilled registers) its unmasked form always does: the next row tile is never the sequence's
      // last, which a list starts with, and behind the last one it copies a tile that nobody reads (row tile 0 of a dense
      // map, which is whole wherever a row tile is unmasked: row 0 sees one key only).  At D = 128 both forms have a body without.
      const bool rides = D == 64 ? (kNear || LISTED) && !CHAIN && mask_c == -1
                                 : (kNear || LISTED) && have1 && mask_c >= -1 && (LISTED || rows_of(rt_n) == full_rows);
      const bool have2 = it + 2 < n_iter, have3 = it + 3 < n_iter;
      Toks tok_a = tok_n;
      if (have1) issue_mask(mask_n, buf ^ 1);
      if (LISTED) {
        if (have2) tok_a = row_tokens<D, 4, LISTED>(tm, rl, rt_a, p.L);
        if (have1 && !rides) issue(hh_n, tok_n, buf ^ 1);
      } else if (have1 && !rides) {
        if (kNear) issue_near(hh_n, rt_n, buf ^ 1);
        else issue(hh_n, row_tokens<D, 4, LISTED>(tm, rl, rt_n, p.L), buf ^ 1);
      }
      // (fetched after the copies were issued: anything the copy code has to wait for - a reloaded register -
      // then finds no list load in flight)
      u32x2 rt_raw{}, mask_raw{};
      if (LISTED) rt_raw = fetch_row_tile(have3 ? ei_b : 0);
      const bool whole_a = whole_tile(rt_a);
      if (!whole_a) mask_raw = fetch_mask(have2 ? ei_a : 0);
      if (mask_c != kSkip) {
        const char* q_lds = lds + buf * kBufBytes;
        const char* do_lds = q_lds + kTileBytes;
        const float* lse_lds = reinterpret_cast<const float*>(q_lds + 2 * kTileBytes);
        const float* delta_lds = lse_lds + kRowsPerTile;
        if (kSkips && CHAIN) {  // (chain tiles always carry a bitmask)
          const u32x4 cm = key_mask(buf);
          dkdv_rowtile_chain<D>(q_lds, do_lds, lse_lds, delta_lds, no, to, kf, vf, dk, dv, g, p.c_log2, cm);
        } else if (mask_c == -1) {
          if (kNear && rides)
            dkdv_rowtile_pipelined<D, 0>(next_rows(D == 64 ? h_lo : hh_n, have1 ? rt_n : 0, buf ^ 1), q_lds, do_lds, lse_lds,
                                         delta_lds, no, to, kf, vf, dk, dv, g, p.c_log2);
          else if (LISTED && rides)  // (behind the last row tile: tok_n still names its rows)
            dkdv_rowtile_pipelined<D, 0>(next_listed(D == 64 ? h_lo : hh_n, tok_n, buf ^ 1), q_lds, do_lds, lse_lds, delta_lds, no, to, kf, vf, dk, dv,
                                         g, p.c_log2);
          else if (ROWS == kRowsFar || D == 128)
            dkdv_rowtile_pipelined<D, 0>(NoCopies{}, q_lds, do_lds, lse_lds, delta_lds, no, to, kf, vf, dk, dv, g, p.c_log2);
        } else if (mask_c >= 0) {
          u32x4 cm = key_mask(buf);  // which of the tile's 128 rows see this lane's key
          // (Shifted to the lane's half here, behind a statement the compiler cannot look through.  Left to itself it
          // tests the unshifted words against sixteen bits that it shifts up before the loop, keeps those in registers
          // across it, spills them, and reloads them behind the copies just issued.)
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            uint32_t x = cm[w] >> (4 * g);
            asm volatile("" : "+v"(x));
            cm[w] = x;
          }
          if (!kSkips || __builtin_amdgcn_ballot_w64((cm[0] | cm[1] | cm[2] | cm[3]) != 0) != 0)  // (else: every key is in the rows' future)
          {
            if (D == 128 && LISTED && rides)
              dkdv_rowtile_pipelined<D, 1>(next_listed(hh_n, tok_n, buf ^ 1), q_lds, do_lds, lse_lds, delta_lds, no, to, kf, vf, dk,
                                           dv, g, p.c_log2, false, cm);
            else if (D == 128 && kNear && rides)
              dkdv_rowtile_pipelined<D, 1>(next_rows(hh_n, rt_n, buf ^ 1), q_lds, do_lds, lse_lds, delta_lds, no, to, kf, vf, dk, dv,
                                           g, p.c_log2, false, cm);
            else
              dkdv_rowtile_pipelined<D, 1>(NoCopies{}, q_lds, do_lds, lse_lds, delta_lds, no, to, kf, vf, dk, dv, g, p.c_log2, false,
                                           cm);
          }
        } else if (LISTED) {  // only packed maps carry such ids
          // keys in front of the row's sequence are off; as a lane mask in scalar registers (a vector register that held
          // each lane's key across the loop was spilled, and reloading it waited for the copies just issued)
          int n_off = -__builtin_amdgcn_readfirstlane(mask_c) - 2 - key0;
          n_off = n_off < 0 ? 0 : (n_off > 32 ? 32 : n_off);
          const uint64_t off32 = (1ull << n_off) - 1;
          const bool lane_off = __builtin_amdgcn_inverse_ballot_w64(off32 | off32 << 32);
          dkdv_rowtile_pipelined<D, 2>(NoCopies{}, q_lds, do_lds, lse_lds, delta_lds, no, to, kf, vf, dk, dv, g, p.c_log2, lane_off);
        }
      }
      dma_publish();
      if (LISTED) tok_n = tok_a;
      rt_n = rt_a;
      rt_a = LISTED ? take_entry(rt_raw).tile : rt_top - ei_b;
      mask_c = mask_n;
      mask_n = !have2 ? kSkip : whole_a ? mask_of(ei_a, TileEntry{0, -1}) : mask_of(ei_a, take_entry(mask_raw));
      step(ei_n, hh_n);
      step(ei_a, hh_a);
      step(ei_b, hh_b);
    }
  };
  // store from registers: lane <-> key, registers <-> d = db*32 + 8*q4 + 4g + j
  auto store = [&](auto chain_tag) {
    constexpr bool CHAIN = decltype(chain_tag)::value;
    if (SV && CHAIN) {
      // First-layer form: the chain keys' gradients are only ever needed summed over the keys (they all come from
      // one shared vector), so each wave adds up its 32 keys here - dK after it has been turned back to the
      // unrotated frame, key by key - and stores one row of D sums per tensor.  The sum over keys runs across
      // lanes: the wave lays its values out in LDS as [d][key] (33 floats per d: conflict-free both ways) and lane
      // l adds up row d = l (and l + 64).  The row tiles' buffers are free: every wave is past the loop's last
      // barrier.  Keys that do not exist contribute zero.
      float* red = reinterpret_cast<float*>(lds) + (size_t)wave * (D * 33);
      static_assert(4 * D * 33 * 4 <= kLdsBytes, "the four waves' transposition buffers must fit");
      const bool have = tile_present && key_ok;
      const float* rope = p.rope_table && have ? p.rope_table + (size_t)token_position(tm, key_tok, p.L) * D : nullptr;
      int b_chain = item - p.n_d0_items;
      const size_t prow = (size_t)(p.rt_lo + split_by(b_chain, p.by_kv)) * 4 + wave;
  #pragma unroll
      for (int which = 0; which < 2; ++which) {  // 0: dK, 1: dV
        if (which == 0 && rope) {
  #pragma unroll
          for (int db = 0; db < D / 64; ++db)
  #pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
              const int d0 = db * 32 + 8 * q4 + 4 * g;
              f32x4 lo, hi;
  #pragma unroll
              for (int j = 0; j < 4; ++j) {
                lo[j] = dk[db][4 * q4 + j];
                hi[j] = dk[db + D / 64][4 * q4 + j];
              }
              rope_turn4<true>(lo, hi, *reinterpret_cast<const f32x4*>(rope + d0),
                               *reinterpret_cast<const f32x4*>(rope + D / 2 + d0));
  #pragma unroll
              for (int j = 0; j < 4; ++j) {
                dk[db][4 * q4 + j] = lo[j];
                dk[db + D / 64][4 * q4 + j] = hi[j];
              }
            }
        }
  #pragma unroll
        for (int db = 0; db < D / 32; ++db)
  #pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int d = db * 32 + 8 * (i / 4) + 4 * g + (i % 4);
            const float x = which ? dv[db][i] : dk[db][i] * p.scale;
            red[d * 33 + ln] = have ? x : 0.f;
          }
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");  // the wave's own LDS writes have landed
        float* out = (which ? p.shared_dv_part : p.shared_dk_part) + (prow * p.Hkv + kvh) * D;
  #pragma unroll
        for (int d = lane; d < D; d += 64) {
          float sum = 0.f;
  #pragma unroll
          for (int j = 0; j < 32; ++j) sum += red[d * 33 + j];
          out[d] = sum;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");  // ... and its reads, before the buffer is written again
      }
      return;
    }

    if (tile_present) {
      float* dkd;
      float* dvd;
      bool write = true, accumulate = false;
      if (!CHAIN) {
        const size_t row = (size_t)h_lo * p.L64 + (size_t)kt * kKeysPerTile + (kblk & 1) * 32 + ln;
        dkd = part_of(p, rg.set, 0) + row * D;
        dvd = part_of(p, rg.set, 1) + row * D;
      } else {
        write = key_ok;
        accumulate = p.chain_accumulate != 0;
        const size_t row = (size_t)(key_ok ? key_tok : 0) * p.Hkv + kvh;
        dkd = p.dk_acc + row * D;
        dvd = p.dv_acc + row * D;
      }
      if (CHAIN && write && p.rope_table) {
        // k was the rotated copy: turn the chain keys' dK back (lane <-> key, both members of a feature
        // pair in its registers).  Depth-0 keys are turned back where their per-head partials are summed.
        const float* rope = p.rope_table + (size_t)token_position(tm, key_tok, p.L) * D;
  #pragma unroll
        for (int db = 0; db < D / 64; ++db)
  #pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const int d0 = db * 32 + 8 * q4 + 4 * g;
            f32x4 lo, hi;
  #pragma unroll
            for (int j = 0; j < 4; ++j) {
              lo[j] = dk[db][4 * q4 + j];
              hi[j] = dk[db + D / 64][4 * q4 + j];
            }
            rope_turn4<true>(lo, hi, *reinterpret_cast<const f32x4*>(rope + d0),
                             *reinterpret_cast<const f32x4*>(rope + D / 2 + d0));
  #pragma unroll
            for (int j = 0; j < 4; ++j) {
              dk[db][4 * q4 + j] = lo[j];
              dk[db + D / 64][4 * q4 + j] = hi[j];
            }
          }
      }
      if (write) {
  #pragma unroll
        for (int db = 0; db < D / 32; ++db)
  #pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            f32x4 a, c;
  #pragma unroll
            for (int j = 0; j < 4; ++j) {
              a[j] = dk[db][4 * q4 + j] * p.scale;
              c[j] = dv[db][4 * q4 + j];
            }
            const int d0 = db * 32 + 8 * q4 + 4 * g;
            if (accumulate) {
              a += *reinterpret_cast<const f32x4*>(dkd + d0);
              c += *reinterpret_cast<const f32x4*>(dvd + d0);
            }
            *reinterpret_cast<f32x4*>(dkd + d0) = a;
            *reinterpret_cast<f32x4*>(dvd + d0) = c;
          }
      }
    }
  };
  // (D = 64: two loops and two epilogues: accumulators that meet again behind them cost spills)
  if (!kSkips) {
    run(std::false_type{});
    if (chain) store(std::true_type{});
    else store(std::false_type{});
  } else if (chain) {
    run(std::true_type{});
    store(std::true_type{});
  } else {
    run(std::false_type{});
    store(std::false_type{});
  }
}

template <int D, int ROWS, bool SV>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void dkdv_kernel(BwdParams p) {
  __shared__ __attribute__((aligned(16))) char lds[kDkdvLds<D>];
  dkdv_item<D, ROWS, SV>(p, lds, blockIdx.x);
}

// dK/dV and dQ as one grid, where both are short of workgroups: neither reads what the other writes once the
// per-row terms are there (the forward of the same call leaves them, or row_terms_kernel), so dQ's workgroups fill the
// slots that unequal dK/dV lists leave, and a launch of a few workgroups, a chain of memory round trips, is not waited for
// before the next.  dQ's come last, heaviest row tiles first: dealt between the chain tiles of the same rows, whose Q and dO
// they share, they were slower (step of 64 heads, L = 411 127 against 119 us, L = 4,096 4,775 against 4,730; chain tiles 4 or 16 row tiles ahead: L = 411 122 and
// 116 against 115, others the same).
// (p_dq: the same parameters once more.  Read from one block, the two halves' scalar registers are loaded together and held
// together, more than there are.)
template <int D, int ROWS, bool SV>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void bwd_kernel(BwdParams p, BwdParams p_dq) {
  constexpr int kDq = D == 64 ? kDqPipeLds<D> : kDqLds<D>;
  __shared__ __attribute__((aligned(16))) char lds[kDkdvLds<D> > kDq ? kDkdvLds<D> : kDq];
  const int n_dkdv = p.n_d0_items + p.n_chain_items;
  const int b = blockIdx.x;
  if (b < n_dkdv) dkdv_item<D, ROWS, SV>(p, lds, b);
  else if constexpr (D == 64) dq_pipe_item<D, SV, false>(p_dq, lds, b - n_dkdv);
  else dq_item<D, false, false>(p_dq, lds, b - n_dkdv);
}

// The per-row terms of a backward that no forward left them for (D = 64): two lanes per row and head, each with the pieces
// of 8 features that the lanes of dq_pipe_kernel hold, added in the same order.  Bound by reading O and dO once.
__global__ __launch_bounds__(256) void row_terms_kernel(BwdParams p) {
  constexpr int D = 64;
  const int rt = p.rt_lo + (int)blockIdx.x / p.Hq;
  const int u = (int)blockIdx.x % p.Hq * kRowsPerTile + (int)(threadIdx.x >> 1), g = threadIdx.x & 1;
  const int r = u / p.Hq, h = u - r * p.Hq;  // neighbouring lanes: neighbouring heads of a row
  int tq;
  if (!row_token(p.tm, rt, r, p.L, tq)) return;  // (both lanes of the row)
  const size_t off = ((size_t)tq * p.Hq + h) * D + g * 8;
  float dl = 0.f;
#pragma unroll
  for (int st = 0; st < D / 16; ++st) dl = add_delta8(dl, as_frag(ld16(p.d_o + off + st * 16)), as_frag(ld16(p.o + off + st * 16)));
  dl += __shfl_xor(dl, 1);
  if (g == 0) {
    const size_t at = (size_t)h * p.T + tq;
    p.delta[at] = -dl;
    p.nlse[at] = -(p.lse[at] * kLog2e) / p.c_log2;
  }
}

// Sum the per-head partials of the depth-0 keys over each KV group into dk_acc / dv_acc, set by set: keys [key_first,
// key_end) of a set, those with anchor < acc_below added to what is there, the others overwriting it.  Several sets of one
// launch give the bits of a launch and a sum each.  (SETS: at most so many.  Bound by reading the partials, 4.9 TB/s; one set by the
// form for several took 5 % longer.)
struct PartSets {
  int n, key_lo, key_hi;  // sets, and all their keys
  int key_first[kMaxRanges], key_end[kMaxRanges], acc_below[kMaxRanges];
};
template <int D, int SETS, int TOGETHER>  // TOGETHER: heads whose loads are on their way together
__global__ __launch_bounds__(256) void reduce_partials_kernel(BwdParams p, PartSets sets) {
  const int group = p.group;
  const size_t per = (size_t)(sets.key_hi - sets.key_lo) * p.Hkv * (D / 4);
  for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < 2 * per; idx += (size_t)gridDim.x * blockDim.x) {
    const int which = idx >= per;
    const size_t rem = which ? idx - per : idx;
    const int c4 = rem % (D / 4);
    int kvh = (int)(rem / (D / 4));  // (K rows of all keys: fewer than 2^31)
    const int j = sets.key_lo + split_by(kvh, p.by_kv);
    // With rotary embedding the summed dK is turned back to the unrotated keys' frame: the thread of
    // a lower-half piece also sums its partner piece of the upper half and stores both.
    const bool turn = !which && p.rope_table != nullptr;
    if (turn && c4 >= D / 8) continue;
    float* dst = (which ? p.dv_acc : p.dk_acc) + (((size_t)j * p.Hkv + kvh) * D + c4 * 4);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f}, acc_hi = acc;  // once `have`: what the sets so far leave
    bool have = false;
#pragma unroll
    for (int i = 0; i < SETS; ++i) {
      if (SETS > 1 && (i >= sets.n || j < sets.key_first[i] || j >= sets.key_end[i])) continue;
      const float* part = part_of(p, i, which);
      f32x4 sum = {0.f, 0.f, 0.f, 0.f}, sum_hi = {0.f, 0.f, 0.f, 0.f};
      const float* src = part + (((size_t)(kvh * group) * p.L64 + j) * D + c4 * 4);
      const size_t head = (size_t)p.L64 * D;
      int hh = 0;
      for (; hh + TOGETHER <= group; hh += TOGETHER) {
        f32x4 x[TOGETHER], y[TOGETHER];
#pragma unroll
        for (int u = 0; u < TOGETHER; ++u) {
          x[u] = *reinterpret_cast<const f32x4*>(src + (hh + u) * head);
          if (turn) y[u] = *reinterpret_cast<const f32x4*>(src + (hh + u) * head + D / 2);
        }
#pragma unroll
        for (int u = 0; u < TOGETHER; ++u) {
          sum += x[u];
          if (turn) sum_hi += y[u];
        }
      }
      for (; hh < group; ++hh) {
        sum += *reinterpret_cast<const f32x4*>(src + hh * head);
        if (turn) sum_hi += *reinterpret_cast<const f32x4*>(src + hh * head + D / 2);
      }
      if (turn) {
        const float* rope = p.rope_table + (size_t)token_position(p.tm, j, p.L) * D + c4 * 4;  // depth-0 key j is token j
        rope_turn4<true>(sum, sum_hi, *reinterpret_cast<const f32x4*>(rope), *reinterpret_cast<const f32x4*>(rope + D / 2));
      }
      if (j < sets.acc_below[i]) {
        if (!have) {
          acc = *reinterpret_cast<const f32x4*>(dst);
          if (turn) acc_hi = *reinterpret_cast<const f32x4*>(dst + D / 2);
        }
        sum += acc;
        sum_hi += acc_hi;
      }
      acc = sum;
      acc_hi = sum_hi;
      have = true;
    }
    if (!have) continue;
    *reinterpret_cast<f32x4*>(dst) = acc;
    if (turn) *reinterpret_cast<f32x4*>(dst + D / 2) = acc_hi;
  }
}

__global__ __launch_bounds__(256) void cast_bf16_kernel(const float* src, __bf16* dst, size_t n4) {
  for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n4; idx += (size_t)gridDim.x * blockDim.x) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(src + idx * 4);
    u32x2 w;
    w[0] = pack_bf16(x[0], x[1]);
    w[1] = pack_bf16(x[2], x[3]);
    *reinterpret_cast<u32x2*>(dst + idx * 4) = w;
  }
}

// =====================================================================================
// Inference-side drafting step: the K new rows of a request (depth 0 = next-token position, depths
// 1..K-1 = multi-token positions, all of the anchor that follows the cached context) are the last
// anchor's rows of the parallel-prediction mask: every cached key is visible, and the new key of
// depth e is visible to the rows of depth >= e.  One workgroup per (context split, KV head,
// request) loops over the split's 64-token pages with the forward's tile routine and leaves an
// unnormalised partial (reference max, row sum, O) for the combine kernel.
// The work is bound by reading the cache once; the matrix cores only keep the arithmetic off
// the critical path.
//
// A wave owns 32 of the K x (Hq/Hkv) query rows that share the KV head (row = depth * group + head).  Where few
// workgroups share a CU, the chain of one tile (LDS reads, matrix instructions, exponentials) and one tile's copy at a
// time set the pace, not the memory system.  So kGroups groups of waves hold the same rows and take the split's tiles
// in turn (tile i: group i % kGroups), kGroups tiles are copied at a time, and the groups are merged through LDS at
// the end.  Where two groups are worth their LDS: see the launcher.
// =====================================================================================
constexpr int kLongPiece = 16;  // pages; see the launcher

// ONE: one piece per request, whose results are written here; otherwise a partial record per piece, which the combine
// kernel merges.
template <int D, int kGroups, int kThreads, bool ONE>
__global__ __launch_bounds__(kThreads) void draft_decode_kernel(DecodeParams p) {
  constexpr int kTileBytes = kKeysPerTile * D * 2;
  constexpr int kBlocks = kTileBytes / 1024;
  constexpr int LAG = ONE ? kDraftLagOnePiece : kDraftLag;
  constexpr int kRing = 2 * kGroups;  // two rounds of kGroups consecutive tiles: one being read, one on its way
  __shared__ __attribute__((aligned(16))) char lds[kRing][2][kTileBytes];  // [buffer][K|V]
  __shared__ int tile_keys[kRing];  // keys present in the tile of each buffer (0 .. 64), set by the wave that copies K
  __shared__ int table_bad;         // the wave that copies K met a page id outside the pool

  // The last two waves of the workgroup only copy (global -> LDS; one K, one V; with three row blocks at D = 128 the last one
  // both), the others only compute: the wait for a copy is counted per wave, so the computing waves never wait on one.  One
  // workgroup barrier per round hands the buffers over.  (One wave for both takes most of a round to issue its copies, 16 or
  // 32 a tile.  us, one / two: 4 requests of 2,048 - 4,096 tokens 14.0 / 13.1, 32 of 1,000 - 4,096 36.9 / 35.9, 64 of 512 - 8,192
  // 121.4 / 119.4; D = 128 16.3 / 15.4, 42.5 / 41.9, 133.8 / 130.9.  Deeper rings, three rounds of one tile, took LDS from the
  // workgroups that share a CU and were slower: 255 against 206 us on 64 equal contexts of 8,192 tokens.)
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, g = lane >> 5, ln = lane & 31;
  const int n_compute = kGroups * (p.rows_pad / 32);
  const bool producer = wave >= n_compute;
  const bool copies_v = wave > n_compute;  // (a copying wave: V rather than K)
  const bool copies_both = D == 128 && kGroups == 1 && (int)(blockDim.x >> 6) == n_compute + 1;  // (three row blocks: see the launcher)
  const int split = blockIdx.x, kvh = blockIdx.y;
  const int group = p.group;
  const int n_rows = p.K * group;

  // Request of this workgroup: workgroups start in the order of blockIdx.z, and the requests take them by falling
  // context length, so that the short ones fill the slots that the long ones leave (64 requests of 512 to 8,192
  // tokens: see the launcher).  Every wave ranks the lengths for itself, one request per lane - unless no request is as
  // long as the table allows for, where the order earns nothing and ranking is most of a workgroup's time (16 requests of
  // 500 to 1,000 tokens in a table for 20,000, D = 128, ranked / not: 28.2 / 26.9 us; 64 in a table for 8,192, D = 64:
  // 42.3 / 33.3).
  int c = blockIdx.z, n_ctx;
  if (!p.by_length) {
    n_ctx = p.ctx_len[c];
  } else {
    const int len = lane < p.C ? p.ctx_len[lane] : INT_MIN;
    if (__builtin_amdgcn_ballot_w64(len > kLongPiece * kKeysPerTile * p.n_splits) != 0) {
      int rank = 0;
      for (int j = 0; j < p.C; ++j) {
        const int other = __builtin_amdgcn_readlane(len, j);
        rank += (other > len || (other == len && j < lane)) ? 1 : 0;
      }
      c = __builtin_ctzll(__builtin_amdgcn_ballot_w64(lane < p.C && rank == (int)blockIdx.z));
    }
    n_ctx = __builtin_amdgcn_readlane(len, c);
  }

  // context of this request, clamped to what the block table can describe
  bool bad = n_ctx < 0 || n_ctx > p.max_pages * kKeysPerTile;
  n_ctx = n_ctx < 0 ? 0 : (n_ctx > p.max_pages * kKeysPerTile ? p.max_pages * kKeysPerTile : n_ctx);
  const int n_pg = (n_ctx + kKeysPerTile - 1) / kKeysPerTile;
  int up = n_pg + p.n_splits - 1;
  const int per = split_by(up, p.by_splits);
  const int p0 = split * per < n_pg ? split * per : n_pg;
  const int p1 = p0 + per < n_pg ? p0 + per : n_pg;
  const int n_tiles = (p1 - p0) + (split == 0 ? 1 : 0);  // split 0 also takes the new keys
  const int n_rounds = (n_tiles + kGroups - 1) / kGroups;

  // Tile i of this split is a cache page or, last in split 0, the K new keys.  Only the copying waves
  // read the block table - through the scalar (constant) path, because a vector load would be ordered
  // behind their copies and using the result would wait for all of them, and one tile ahead of its use,
  // so that the load's latency is off the path; the one that copies K tells the computing waves how many keys each tile
  // holds through tile_keys[] (a page id outside the pool makes the tile empty and flags the request).
  typedef const int32_t __attribute__((address_space(4))) * ConstTable;
  auto page_of = [&](int i) {
    return i < p1 - p0 ? ((ConstTable)(uintptr_t)p.block_table)[(size_t)c * p.max_pages + p0 + i] : 0;
  };

  if (producer) {
    // Rows of a tile that hold no key (tail of the last page, rows past the K new keys, an empty tile)
    // are filled from the request's first new key, which is always present and finite user data: their
    // probabilities are masked to zero, and zero times a finite value adds nothing.
    const __bf16* fill = uniform_ptr((copies_v ? p.v_new : p.k_new) + ((size_t)c * p.K * p.Hkv + kvh) * D);
    const __bf16* pages = uniform_ptr(copies_v ? p.v_pages : p.k_pages);
    const int row_in_blk = lane / (D / 8), phys = lane % (D / 8);
    // A whole page: 1 KiB pieces of consecutive memory, their addresses on the scalar unit (with per-lane 64-bit
    // addresses this wave needed most of a microsecond to issue one tile's copies).  The chunk a lane fetches from a
    // piece depends on the piece only through the swizzle, whose period is 16 rows.
    constexpr int kPeriod = 16 / (512 / D);
    uint32_t voff[kPeriod];
#pragma unroll
    for (int j = 0; j < kPeriod; ++j)
      voff[j] = (uint32_t)(row_in_blk * D + ((phys ^ swz<D>(j * (512 / D) + row_in_blk)) << 3)) * 2u;
    auto copy_half = [&](int i, int page, bool is_new, int valid, const __bf16* pages, const __bf16* fill, bool v_half) {
      // (untracked copies: a tracked one would make every workgroup barrier below wait for all of them)
      const uint32_t dst = __builtin_amdgcn_readfirstlane(lds_scalar_addr(lds[i % kRing][0]) + (v_half ? kTileBytes : 0));
      if (!is_new && valid == kKeysPerTile) {
        const __bf16* src = uniform_ptr(pages + ((size_t)page * p.Hkv + kvh) * (kKeysPerTile * D));
#pragma unroll
        for (int blk = 0; blk < kBlocks; ++blk) dma16_untracked(src + blk * 512, voff[blk % kPeriod], dst + blk * 1024);
        return;
      }
#pragma unroll 2
      for (int blk = 0; blk < kBlocks; ++blk) {
        const int row = blk * (512 / D) + row_in_blk;
        const int chunk = (phys ^ swz<D>(row)) << 3;
        const __bf16* src;
        if (row >= valid) src = fill + chunk;
        else if (is_new) src = fill + (size_t)row * p.Hkv * D + chunk;
        else src = pages + (((size_t)page * p.Hkv + kvh) * kKeysPerTile + row) * D + chunk;
        dma16_untracked(src, dst + blk * 1024);
      }
    };
    int page_next = page_of(0);
    auto copy_tile = [&](int i) {
      const int page = page_next;
      page_next = page_of(i + 1);
      const bool is_new = i >= p1 - p0;
      int valid = p.K;
      if (!is_new) {
        valid = n_ctx - (p0 + i) * kKeysPerTile;
        valid = valid > kKeysPerTile ? kKeysPerTile : valid;
        if (page < 0 || page >= p.n_pages) {
          bad = true;
          valid = 0;
        }
      }
      if (lane == 0 && !copies_v) tile_keys[i % kRing] = valid;
      copy_half(i, page, is_new, valid, pages, fill, copies_v);
      if (copies_both)
        copy_half(i, page, is_new, valid, uniform_ptr(p.v_pages), uniform_ptr(p.v_new + ((size_t)c * p.K * p.Hkv + kvh) * D), true);
    };
    int issued = 0;  // tiles
    auto copy_round = [&] {
      for (int t = 0; t < kGroups && issued < n_tiles; ++t) copy_tile(issued++);
    };
    copy_round();
    for (int q = 0; q < n_rounds; ++q) {
      wait_outstanding<0>();  // round q has landed
      if (q == n_rounds - 1 && lane == 0 && !copies_v) table_bad = bad ? 1 : 0;  // every tile has been looked up by now
      __syncthreads();  // round q is published; the computing waves are done with round q-1 ...
      copy_round();     // ... whose buffers take round q + 1
    }
    if (n_rounds == 0) {
      if (lane == 0 && !copies_v) table_bad = 0;
      __syncthreads();
    }
    if (kGroups > 1) {  // the two barriers of the merge below
      __syncthreads();
      __syncthreads();
    }
    return;  // barriers executed: the same as the computing waves below
  }

  const int n_row_waves = p.rows_pad / 32;
  const int grp = wave / n_row_waves;                    // which of the kGroups
  const int r = (wave - grp * n_row_waves) * 32 + ln;    // query row of this lane (shared with lane ^ 32)
  const bool row_ok = r < n_rows;
  const int depth = row_ok ? small_quotient(r, p.group_reciprocal) : 0, head = kvh * group + (row_ok ? r - depth * group : 0);
  bf16x8 qf[1][D / 16];
  {
    const __bf16* qrow = p.q_new + (((size_t)c * p.K + depth) * p.Hq + head) * D + g * 8;
#pragma unroll
    for (int st = 0; st < D / 16; ++st) qf[0][st] = as_frag(ld16(qrow + st * 16));
  }
  f32x16 o[1][D / 32];
  float m[1] = {kNegInit}, lsum[1] = {0.f};
#pragma unroll
  for (int db = 0; db < D / 32; ++db) o[0][db] = zero16();
  const NatOff<D> no = nat_offsets<D>(lane);
  const TrOff<D> to = tr_offsets<D>(lane);

  if (n_rounds == 0) __syncthreads();
  for (int q = 0; q < n_rounds; ++q) {
    __syncthreads();  // round q has landed
    const int i = q * kGroups + grp;
    if (i >= n_tiles) continue;
    const int buf = i % kRing;
    const bool is_new = i >= p1 - p0;
    const int valid = __builtin_amdgcn_readfirstlane(tile_keys[buf]);
    if (!is_new && valid == kKeysPerTile) {
      const uint32_t mw[2] = {0xffffffffu, 0xffffffffu};
      fwd_tile<D, 1, false, true, LAG>(lds[buf][0], lds[buf][1], no, to, qf, o, m, lsum, mw, p.c_log2);
    } else {
      // keys [0, n) of the tile are visible: n = the page's valid tokens, or depth + 1 of the new keys
      const int n = is_new ? depth + 1 : valid;
      const uint64_t bits = n >= 64 ? ~0ull : ((1ull << n) - 1);
      const uint32_t mw[2] = {(uint32_t)bits >> (4 * g), (uint32_t)(bits >> 32) >> (4 * g)};
      fwd_tile<D, 1, true, true, LAG>(lds[buf][0], lds[buf][1], no, to, qf, o, m, lsum, mw, p.c_log2);
    }
  }

  if (kGroups > 1) {
    // Merge of the groups: each but the first leaves (max, sum, O) in the buffers, [value][lane] per wave, and the
    // first adds them up in order.  A group that had no tile carries the start values, which add nothing.
    constexpr int kVals = 2 + (D / 32) * 16;
    static_assert((kGroups - 1) * (kThreads / 64 - 2) / kGroups * kVals * 256 <= (int)sizeof(lds), "merge records must fit");
    float* x = reinterpret_cast<float*>(&lds[0][0][0]);
    __syncthreads();  // every wave has left the tiles
    if (grp > 0) {
      float* mine = x + (size_t)(wave - n_row_waves) * (kVals * 64) + lane;
      mine[0] = m[0];
      mine[64] = lsum[0];
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) mine[(2 + db * 16 + i) * 64] = o[0][db][i];
    }
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int og = 1; og < kGroups; ++og) {
      const float* his = x + (size_t)((og - 1) * n_row_waves + wave) * (kVals * 64) + lane;
      const float hm = his[0], hl = his[64];
      const float mm = __builtin_fmaxf(m[0], hm);
      const float a = exp2_fast(m[0] - mm), b = exp2_fast(hm - mm);
      m[0] = mm;
      lsum[0] = lsum[0] * a + hl * b;
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[0][db][i] = o[0][db][i] * a + his[(2 + db * 16 + i) * 64] * b;
    }
  }

  const float l_tot = sum_halves(lsum[0]);
  if (ONE) {
    if (row_ok) {
      const float inv = 1.0f / l_tot;
      __bf16* orow = p.o + (((size_t)c * p.K + depth) * p.Hq + head) * D;
#pragma unroll
      for (int db = 0; db < D / 32; ++db) store_row_bf16(orow + db * 32, o[0][db], inv, g);
      if (g == 0) p.lse[((size_t)c * p.Hq + head) * p.K + depth] = (m[0] + __builtin_log2f(l_tot)) * kLn2;
    }
    if (p.status && kvh == 0 && tid == 0) p.status[c] = bad || table_bad != 0;  // (table_bad: written before the last barrier)
    return;
  }

  // partial record of this split: lane <-> row, registers <-> d = db*32 + 8*q4 + 4g + j
  const size_t rec = ((size_t)c * p.Hkv + kvh) * p.n_splits + split;
  if (r < p.rows_pad) {
    float* po = p.part_o + (rec * p.rows_pad + r) * D;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        f32x4 a;
#pragma unroll
        for (int j = 0; j < 4; ++j) a[j] = o[0][db][4 * q4 + j];
        *reinterpret_cast<f32x4*>(po + db * 32 + 8 * q4 + 4 * g) = a;
      }
    if (g == 0) {
      float* ml = p.part_ml + rec * 3 * p.rows_pad;
      ml[r] = m[0];
      ml[p.rows_pad + r] = l_tot;
      ml[2 * p.rows_pad + r] = (bad || table_bad != 0) ? 1.f : 0.f;  // (table_bad: written before the last barrier)
    }
  }
}

// Merges the splits of a request's rows: M = max m_s, L = sum l_s 2^(m_s - M), O = sum O_s 2^(m_s - M) / L.
// kLanes threads per (request, KV head, row, 4 features), kEach splits per thread, all of a thread's loads issued
// before the first is used: the kernel's time is one memory round trip (two passes over the splits, and all status
// words set by one workgroup, took 6.2 / 8.9 / 13.6 us for 4 x 16, 2 x 32 and 64 x 2 requests x splits; this 4.3 /
// 4.0 / 6.3).  Request and KV head are grid dimensions: taken from a row number, three 64-bit divisions stood before the first
// load.  us per drafting step with them / so: 4 requests of 2,048 - 4,096 tokens 12.6 / 11.8, 2 of 10,800 - 20,000 at D = 128
// 20.9 / 20.1, 16 of 1,000 13.4 / 12.8, 64 of 512 - 8,192 118.5 / 117.2 (the main kernel without divisions included).  The threads of a row sit D/4 lanes apart and are merged by lane exchange.  The wave of a request's
// first row of KV head 0 also sets its status word: every KV head's workgroups look at the same block-table entries,
// so head 0's records tell.
template <int D, int kLanes, int kEach>
__global__ __launch_bounds__(256) void draft_decode_combine_kernel(DecodeParams p) {
  constexpr int kPerRow = (D / 4) * kLanes, kRowsPerWave = 64 / kPerRow;
  static_assert(kPerRow <= 64, "the threads of a row are one wave's");
  const int n_rows = p.K * p.group;
  const int lane = threadIdx.x & 63;
  const int c4 = lane % (D / 4), sl = lane / (D / 4) % kLanes;
  const int kvh = blockIdx.y, c = blockIdx.z;
  const int row = ((int)blockIdx.x * 4 + (int)(threadIdx.x >> 6)) * kRowsPerWave + lane / kPerRow;
  const bool ok = row < n_rows;
  const int r = ok ? row : n_rows - 1;
  const size_t rec0 = ((size_t)c * p.Hkv + kvh) * p.n_splits;
  const float* ml0 = p.part_ml + rec0 * 3 * p.rows_pad + r;
  const float* o0 = p.part_o + (rec0 * p.rows_pad + r) * D + c4 * 4;
  float mv[kEach], lv[kEach];
  f32x4 ov[kEach];
#pragma unroll
  for (int j = 0; j < kEach; ++j) {  // (splits past the last are read as the last and weigh nothing)
    const int s = sl * kEach + j < p.n_splits ? sl * kEach + j : p.n_splits - 1;
    mv[j] = ml0[(size_t)s * 3 * p.rows_pad];
    lv[j] = ml0[(size_t)s * 3 * p.rows_pad + p.rows_pad];
    ov[j] = *reinterpret_cast<const f32x4*>(o0 + (size_t)s * p.rows_pad * D);
  }
  bool any = false;
  const bool flags = p.status && ok && r == 0 && kvh == 0;
  if (flags) {
    for (int s = lane % kPerRow; s < p.n_splits; s += kPerRow) any |= ml0[((size_t)s * 3 + 2) * p.rows_pad] != 0.f;
  }
  float M = mv[0];
#pragma unroll
  for (int j = 1; j < kEach; ++j) M = __builtin_fmaxf(M, mv[j]);
#pragma unroll
  for (int x = D / 4; x < kPerRow; x <<= 1) M = __builtin_fmaxf(M, __shfl_xor(M, x));
  float L = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < kEach; ++j) {
    const float w = sl * kEach + j < p.n_splits ? exp2_fast(mv[j] - M) : 0.f;
    L = __builtin_fmaf(lv[j], w, L);
    acc += ov[j] * w;
  }
#pragma unroll
  for (int x = D / 4; x < kPerRow; x <<= 1) {
    L += __shfl_xor(L, x);
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] += __shfl_xor(acc[j], x);
  }
  const float inv = 1.0f / L;
  const int depth = small_quotient(r, p.group_reciprocal), head = kvh * p.group + (r - depth * p.group);
  if (ok && sl == 0) {
    u32x2 w2;
    w2[0] = pack_bf16(acc[0] * inv, acc[1] * inv);
    w2[1] = pack_bf16(acc[2] * inv, acc[3] * inv);
    *reinterpret_cast<u32x2*>(p.o + (((size_t)c * p.K + depth) * p.Hq + head) * D + c4 * 4) = w2;
    if (c4 == 0) p.lse[((size_t)c * p.Hq + head) * p.K + depth] = (M + __builtin_log2f(L)) * kLn2;
  }
  const uint64_t votes = __builtin_amdgcn_ballot_w64(any);
  if (flags && lane % kPerRow == 0) {
    const uint64_t row_lanes = kPerRow == 64 ? ~0ull : ((1ull << (kPerRow & 63)) - 1) << lane;
    p.status[c] = (votes & row_lanes) != 0 ? 1 : 0;
  }
}

// ------------------------------------------------------------------------------------- launchers

// Pure MFMA issue loop (no memory traffic): four independent accumulator chains per wave,
// 8 workgroups x 4 waves per CU.  Used only to report the measured matrix-core ceiling.
// RANDOM = false: small integer operands that never change (little switching activity in the multipliers);
// RANDOM = true: four sets of operands drawn from a hash, roughly uniform in (-2, 2) with every significand
// bit in use, taken in turn - the activity the matrix cores see on real Q, K, V.  The chip lowers its clock
// under the second kind of load, so the two rates differ.
template <bool RANDOM>
__global__ __launch_bounds__(256) void mfma_ceiling_kernel(float* out, int iters) {
  bf16x8 a[4], b[4];
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (RANDOM) {
        uint32_t x = (blockIdx.x * 256u + threadIdx.x) * 64u + s * 16u + j;
        x ^= x >> 16; x *= 0x7feb352du; x ^= x >> 15; x *= 0x846ca68bu; x ^= x >> 16;
        a[s][j] = (__bf16)(((float)(x & 0xffffu) - 32767.5f) * (2.0f / 32768.0f));
        b[s][j] = (__bf16)(((float)(x >> 16) - 32767.5f) * (2.0f / 32768.0f));
      } else {
        a[s][j] = (__bf16)(float)(threadIdx.x % 3);
        b[s][j] = (__bf16)(float)(threadIdx.x % 5);
      }
    }
  f32x16 acc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i] = zero16();
  for (int it = 0; it < iters; it += 4) {  // (iters is a multiple of four)
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = mfma32(a[RANDOM ? i : 0], b[RANDOM ? (i + u) & 3 : 0], acc[i]);
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) s += acc[i][r];
  out[(size_t)blockIdx.x * 256 + threadIdx.x] = s;
}

namespace {

constexpr int kCus = 256;  // compute units of the device

// The forward's form at D = 64, by the number of workgroups of one query head and the mean length of the row tiles' lists: two
// heads per workgroup (which share K/V tiles) at three per CU where there are at least eight workgroups of one head for each CU
// (lists of up to four tiles: twelve); one head where there are fewer, to fill the chip; two heads at two per CU (registers
// to schedule with) in between with long lists.  A head's results do not depend on the choice.  Forward us, one head / two
// heads at two per CU / at three, by (mean list; workgroups of one head):
//   many: 64 heads, L = 700 (8; 2,816) 57 / 54 / 52, L = 1,391 (13; 5,568) 168 / 158 / 156, L = 4,096 (35; 16,384) 1,213 / 1,156 / 1,128, L =
//     20,480 (165; 81,920) 28,010 / 26,310 / 26,000, eight packed sequences of 203 to 517 anchors (6; 11,072) 186 / 183 / 168, of 64 to 1,728
//     (12; 25,800) 753 / 727 / 690; 16 heads, L = 2,048 (19; 2,048) 88.5 / 83.7 / 84.5, L = 4,096 (35; 4,096) 303 / 290 / 289;
//   very short lists: K = 32, 64 heads L = 128 (4; 2,048) 27.6 / 29.5 / 28.3, but L = 330, 32 heads (5; 2,656) 39.6 / 41.3 / 37.7, sixty
//     packed sequences of 16 anchors, K = 8 (3; 3,840) 40.1 / 43.1 / 38.2;
//   few: 4 heads, L = 1,391 (13; 348) 21.7 / 29.8 / 33.9, L = 2,048 (19; 512) 31.1 / 40.1 / 45.8, L = 4,096 (35; 1,024) 86 / 91 / 96, packed 64 to
//     1,728 (12; 1,612) 56 / 59 / 63; 16 heads, L = 1,391 (13; 1,392) 46.1 / 48.3 / 48.4;
//   in between: 8 heads, L = 3,000 (26; 1,504) 87 / 88 / 93, L = 4,000 (33; 2,000) 145 / 138 / 143; 4 heads, L = 8,000 (65; 2,000) 280 / 270 / 279.
// One head runs three workgroups per CU (148 registers, a third buffer) where that many run at once, and, while lists are long and
// unequal, up to four per CU, and with short lists where four per CU would leave a quarter of a second round; else four (128
// registers, two buffers).  Forward us, three / four, by (mean list; workgroups):
//   4 heads, K = 4 L = 2,048 (19; 256) 27.1 / 30.2, L = 1,391 (13; 348) 21.7 / 23.7, L = 2,048 (19; 512) 30.6 / 32.5, 64 heads L = 128
//     (4; 512) 9.2 / 9.5, 16 heads L = 700 (7; 704) 18.3 / 18.9, 4 heads L = 3,000 (26; 752) 53.3 / 53.1;
//   long: 6 heads L = 2,500 (22; 942) 51.4 / 53.1, 4 heads L = 4,096 (34; 1,024) 83.6 / 86.9;  but 64 heads L = 200 (4; 832) 15.3 / 13.7,
//     16 heads L = 1,000 (10; 1,008) 31.2 / 29.5, 64 heads L = 256 (5; 1,024) 18.9 / 16.3, 12 heads L = 1,391 (13; 1,044) 38.8 / 37.2;
//   a quarter of a round (in a step, under the profiler): K = 7, 32 heads L = 600 (7; 1,088) 29.1 / 30.6, 64 heads L = 330 (5; 1,216) 25.9 /
//     27.1, K = 8 L = 300 (5; 1,216) 24.0 / 24.3, but 64 heads L = 330 (5; 1,344) 26.5 / 26.4, 16 heads L = 1,200 (12; 1,200) 43.7 / 42.5;
//   many: 64 heads L = 411 (6; 1,664) 30.3 / 28.4; 24 heads in groups of three L = 2,500 (22; 3,768) 180 / 176, L = 8,192 (66; 12,288) 1,673 / 1,632.
constexpr int kShortMeanTiles = 4, kFewMeanTiles = 24, kLongMeanTiles = 14, kTailMeanTiles = 8;
enum class FwdForm { kOneHead, kOneHeadThreePerCu, kTwoHeads, kTwoHeadsThreePerCu };
inline FwdForm pick_fwd_form(int group, int mean_tiles, int n_wg) {
  const bool three_per_cu = n_wg <= 3 * kCus || (n_wg <= 4 * kCus ? mean_tiles > kLongMeanTiles : n_wg < 5 * kCus && mean_tiles <= kTailMeanTiles);
  const FwdForm one_head = three_per_cu ? FwdForm::kOneHeadThreePerCu : FwdForm::kOneHead;
  if (group % 2 != 0 || n_wg <= 4 * kCus) return one_head;
  if (n_wg >= (mean_tiles <= kShortMeanTiles ? 12 : 8) * kCus) return FwdForm::kTwoHeadsThreePerCu;
  return mean_tiles <= kFewMeanTiles ? one_head : FwdForm::kTwoHeads;
}

struct TimedSpan {
  KernelTimer* t;
  hipStream_t stream;
  hipError_t err = hipSuccess;
  TimedSpan(KernelTimer* timer, int kind, hipStream_t s) : t(timer), stream(s) {
    if (t) err = t->begin(kind, s);
  }
  hipError_t finish() {
    hipError_t e = hipGetLastError();
    if (t && err == hipSuccess) err = t->end(stream);
    return e != hipSuccess ? e : err;
  }
};

}  // namespace

hipError_t KernelTimer::begin(int kind, hipStream_t stream) {
  Span sp{nullptr, nullptr, kind};
  hipError_t e = hipEventCreate(&sp.start);
  if (e != hipSuccess) return e;
  e = hipEventCreate(&sp.stop);
  if (e != hipSuccess) {
    (void)hipEventDestroy(sp.start);
    return e;
  }
  spans.push_back(sp);
  return hipEventRecord(sp.start, stream);
}

hipError_t KernelTimer::end(hipStream_t stream) { return hipEventRecord(spans.back().stop, stream); }

hipError_t KernelTimer::collect(float* ms, int32_t* launches) {
  hipError_t rc = hipSuccess;
  for (Span& sp : spans) {
    float t = 0.f;
    hipError_t e = hipEventSynchronize(sp.stop);
    if (e == hipSuccess) e = hipEventElapsedTime(&t, sp.start, sp.stop);
    if (e == hipSuccess) {
      ms[sp.kind] += t;
      launches[sp.kind] += 1;
    } else {
      rc = e;
    }
  }
  return rc;
}

KernelTimer::~KernelTimer() {
  for (Span& sp : spans) {
    (void)hipEventDestroy(sp.start);
    (void)hipEventDestroy(sp.stop);
  }
}

hipError_t launch_fwd(const FwdParams& p, int D, hipStream_t stream, KernelTimer* timer) {
  const int n_rt = p.rt_hi - p.rt_lo;
  if (n_rt <= 0) return hipSuccess;
  const bool sv = p.v_shared != nullptr;  // first-layer form: kernels that read chain V rows from the shared vector
  if (D == 128 && sv) return hipErrorInvalidValue;  // (D = 128 has no such instantiation: its callers expand V instead)
  TimedSpan span(timer, kKindFwd, stream);
  auto go = [&](auto kernel, int heads) {
    FwdParams fp = p;
    fp.by_heads = make_divisor(p.group / heads);
    hipLaunchKernelGGL(kernel, dim3((unsigned)(n_rt * (p.Hq / heads))), dim3(256), 0, stream, fp);
  };
  if (D == 128) {
    go(fwd_kernel<128, 1, false, 2>, 1);
  } else {
    switch (pick_fwd_form(p.group, p.mean_tiles, n_rt * p.Hq)) {
      case FwdForm::kOneHeadThreePerCu: go(sv ? fwd_kernel<64, 1, true, 3> : fwd_kernel<64, 1, false, 3>, 1); break;
      case FwdForm::kOneHead: go(sv ? fwd_kernel<64, 1, true, 4> : fwd_kernel<64, 1, false, 4>, 1); break;
      case FwdForm::kTwoHeads: go(sv ? fwd_kernel<64, 2, true, 2> : fwd_kernel<64, 2, false, 2>, 2); break;
      case FwdForm::kTwoHeadsThreePerCu: go(sv ? fwd_kernel<64, 2, true, 3> : fwd_kernel<64, 2, false, 3>, 2); break;
    }
  }
  return span.finish();
}

constexpr int kPlainMeanTiles = 24, kPlainWorkgroups = 2 * 3 * kCus;
hipError_t launch_dq(const BwdParams& p, int D, hipStream_t stream, KernelTimer* timer) {
  const int n_rt = p.rt_hi - p.rt_lo;
  if (n_rt <= 0) return hipSuccess;
  // First-layer form.  The dQ kernel reads chain V rows from the shared vector at D = 64 only: at D = 128 it has
  // no registers to spare (that instantiation spilled three times as much and ran 25 % slower), so there the
  // caller passes an expanded V in `v` for it; the dK/dV kernel takes the shared vector at either size.
  const bool sv = p.v_shared != nullptr && D == 64;
  // D = 64: the plain kernel where the lists are short, the pipelined one elsewhere; a row's dQ has the same bits from both.  What
  // runs as one grid with dK/dV (backward_in_one_grid()) does not come here: a step does with short lists and more than 4,096
  // workgroups - the plain kernel -, a backward called by itself with more than 3,072, and a step timed kernel by kernel, which
  // alone has few (below two full rounds of the plain kernel's three per CU it shows the pipelined one, as the one grid runs).
  // One launch: the row tiles of one split between the two kernels by list length ran one after the other, each leaving the
  // chip to drain (2,048 anchors, K = 4, 4 heads: 66 us).  us, pipelined / plain, by mean list length (workgroups): L = 1,391, 64
  // heads (14; 5,568) 289 / 262; L = 4,096, 16 heads (35; 4,096) 422 / 427, 64 heads (35; 16,384) 1,666 / 1,646, sampled 8,192
  // (67) 3,195 / 3,277.  (The first-layer form comes here with short lists only.)
  const int n_wg = n_rt * p.Hq;  // one query head per workgroup
  const bool plain = sv || (p.mean_tiles <= kPlainMeanTiles && n_wg >= kPlainWorkgroups);
  TimedSpan span(timer, kKindDq, stream);
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((unsigned)n_wg), dim3(256), 0, stream, p); };
  if (D == 128) go(dq_kernel<128, false>);
  else if (plain) go(sv ? dq_kernel<64, true> : dq_kernel<64, false>);
  else go(dq_pipe_kernel<64>);
  return span.finish();
}

// dK/dV and dQ as one grid, or dQ (which then also forms the per-row terms) before dK/dV?  At D = 64 one grid with long
// lists, where dQ's half is the pipelined kernel (it gains at any number of workgroups: dQ's fill the end of dK/dV), and
// with short lists (where the plain one runs three workgroups per CU, and the one grid two) as long as workgroups are few
// enough that unequal lists and the launches' ends cost more.  us per step, dQ first / one grid (mean list; dQ workgroups):
// 4 heads L = 256, K = 4 46.9 / 36.8 (4; 32), L = 1,000 164 / 148 (11; 252), L = 4,096 693 / 634 (35; 1,024), L = 16,000
// 4,990 / 4,740 (128; 4,000), packed 396 / 338 (12; 1,612), 16 heads L = 2,048 458 / 394 (19; 2,048), 64 heads L = 411 148 /
// 120 (6; 1,664), L = 700 258 / 236 (8; 2,816), L = 1,000 412 / 403 (11; 4,032), L = 3,000 2,657 / 2,611 (26; 12,032), L =
// 4,096 4,749 / 4,670 (35; 16,384), L = 8,000 16.82 / 16.73 ms (65; 32,000), L = 16,000 65.04 / 64.80, L = 20,480 104.25 /
// 103.84 (165; 81,920), in one segment 105.97 / 105.47, first-layer form L = 3,891 4,456 / 4,402, sampled 8,192 9,871 /
// 9,821; but L = 1,391 709 / 716 (14; 5,568), eight packed sequences 3,156 / 3,344 (12; 12,896).
// At D = 128 a dK/dV workgroup has a CU to itself, and in one grid dQ's have, too, of which two share one otherwise: where
// there are few.  4 heads L = 256, K = 4 67 / 50.7 (32 dQ workgroups), L = 1,000 252 / 215 (252), L = 4,096 1,109 / 966 (1,024),
// packed 630 / 504 (1,612), L = 8,000 2,770 / 2,719 (2,000), 32 heads L = 128 68.6 / 54.8 (256), L = 500 201 / 176 (1,024),
// L = 800 340 / 329 (1,600); but L = 1,000 442 / 459 (2,016), L = 1,391 727 / 793 (2,784), L = 4,096 4,899 / 5,360.  (The
// first-layer form reads two forms of V there and stays apart.)
// A backward called by itself at D = 64 pays a pass over O and dO for the terms: 4 heads L = 4,096 664 / 607, 16 heads L = 2,048 455 /
// 412, 64 heads L = 700 254 / 247; but L = 3,000 2,740 / 2,784.
bool backward_in_one_grid(int D, int mean_tiles, int n_row_tiles, int Hq, bool terms_left, bool sv) {
  constexpr int kMostWorkgroups = 16 * kCus, kMostWithTermsPass = 12 * kCus, kMostD128 = 13 * kCus / 2;
  const int n_wg = n_row_tiles * Hq;
  if (D != 64) return !sv && terms_left && n_wg <= kMostD128;
  if (!terms_left) return n_wg <= kMostWithTermsPass;
  return mean_tiles > kPlainMeanTiles || n_wg <= kMostWorkgroups;
}

hipError_t launch_row_terms(const BwdParams& p, hipStream_t stream) {
  const int n_rt = p.rt_hi - p.rt_lo;
  if (n_rt <= 0) return hipSuccess;
  hipLaunchKernelGGL(row_terms_kernel, dim3((unsigned)(n_rt * p.Hq)), dim3(256), 0, stream, p);
  return hipGetLastError();
}

// Where a range's key-tile pairs x heads are few, the next ranges' fill the slots, and the launches' ends are fewer: up to
// 768 items in the last range (512 run at once) at D = 64, 512 (256) at D = 128.  us per step, a launch per range / up to
// four together (items of the last): 4 heads L = 256 in segments of 64 86 / 33 (8), of 128 66 / 40, L = 512 of 128 127 / 46
// (16; D = 128 174 / 64), L = 2,500 of 1,024 368 / 206 (80), L = 4,096 631 / 351 (128), by itself 610 / 399, L = 8,000 in
// segments of 2,048 1,490 / 1,140 (252), L = 16,000 4,880 / 4,360 (500), L = 20,480 in segments of 1,024 8,490 / 7,250
// (640), sampled L = 3,000 328 / 281, 16 heads L = 4,096 1,343 / 1,247 (512), 64 heads L = 1,500 834 / 826 (768); but L =
// 2,048 1,404 / 1,417 (1,024), L = 4,096 4,927 / 4,997 (2,048); D = 128 4 heads L = 4,096 968 / 732 (128), 32 heads L =
// 2,048 1,458 / 1,436 (512).  The partials of every set beyond the first are as large as the problem's depth-0 keys x heads
// in fp32.
int dkdv_part_sets(int D, int L64, int Hq, int n_ranges) {
  const int64_t items = (int64_t)((L64 / kKeysPerTile + 1) / 2) * Hq;
  const int most = items > (D == 64 ? 3 : 2) * kCus ? 1 : kMaxRanges;
  return n_ranges < most ? (n_ranges < 1 ? 1 : n_ranges) : most;
}

// A key-tile pair's workgroup walks its row tiles one after the other, 1.9 us each at D = 64, and with few heads the longest
// walk is the whole of dK/dV: the 63 of 4 heads' L = 1,000 are most of a step's 140 us, while most slots are idle.  So a range
// of rows is cut into chunks, up to the four whose partials one launch sums, while
//  - the work items of all chunks run at once (512 slots at D = 64, 256 at D = 128).  16 heads L = 3,000, 384 items: 660 us in
//    two chunks, 665 in three; 8 heads L = 3,000, 192: 344 and 350; D = 128 4 heads L = 4,096, 128: 683 and 702 in four;
//  - with short lists (under 40 row tiles) a quarter of them do: 64 heads L = 400, 256 items, 102 us in one chunk and 106 in
//    two, 32 heads at D = 128, 128 items, 127.5 and 133;
//  - there is one chunk for 16 row tiles (the fourth from 64 on, so that its partials, a quarter of the workspace's, are worth
//    it: 63 row tiles 70 us in three, 63 in four), in sampled and packed maps up to three;
//  - the chunks of a sampled or packed map cut its longest walk, by a sixteenth at least: where a boundary falls between sequences
//    they do not (400, 300 and 90 anchors, 32 heads, 100 us and 104 in two, 16 heads at D = 128 126 and 131; seven sequences of 331 to
//    1,388, K = 4, 4 heads, 125 and 154 in three), where it falls inside the long ones they do (363, 170, 701 and 226, 8 heads at D = 128,
//    walks of 46 and 31 row tiles, 189 and 147 in two; 164 to 1,446, 4 heads at D = 128, 389 and 288).  Where all slots are taken and
//    the walks fill a fifth of the longest one's time, a chunk is also shorter than that one, by an eighth (16 heads, seven sequences
//    of 61 to 785, walks of 48 and 36, chunks of 58, 165 and 176; but 8 heads at D = 128, 56, 578 and 1,288, walks of 90 and 61, chunks of
//    61, 367 and 314); and where the longest walk is short, they fill less than a quarter of its time (16 heads at D = 128, 603, 53
//    and 364, walks of 38 and 33, 179 and 206);
//  - the problem's segments leave sets (4 heads L = 4,096 in four segments 328 us, with each in two chunks 340).
// us per step, uncut / so: 4 heads L = 300 54.6 / 40.5, L = 600 91 / 51, L = 1,000 140 / 70, L = 1,391 187 / 82, L = 2,048 269 /
// 119, L = 4,096 in two segments 377 / 338, K = 4 L = 2,500 185 / 97, K = 5 L = 1,200 117 / 63; 16 heads L = 700 113 / 72, L =
// 2,048 390 / 333; 32 heads L = 700 137 / 118; D = 128 4 heads L = 600 137 / 72, L = 1,391 283 / 124, 8 heads L = 2,048 464 /
// 394; 4 heads, sampled L = 1,500 125 / 70, L = 3,000 239 / 137, packed 200 and 300 anchors 70 / 53, 3,000 and 100
// 416 / 220.  A key's sums then have other last bits than the same heads' in a call of many.  From four query heads on, which is the
// smallest drafter; calls of one to three would be faster in chunks too (three heads L = 2,048 take what four took uncut), and are left
// in one range so that parts of a call, taken up to three heads at a time, keep the bits that they have in the whole.
constexpr int kSplitHeads = 4, kSplitRowTiles = 16, kShortLists = 40;
ChunkSplit dkdv_chunk_split(int D, int L64, int Hq, int n_ranges) {
  const int64_t items = (int64_t)((L64 / kKeysPerTile + 1) / 2) * Hq;
  const int slots = (D == 64 ? 2 : 1) * kCus;
  if (Hq < kSplitHeads || items > slots) return {1, 0, 1};
  return {(int)items, slots, kMaxRanges / n_ranges};
}
int dkdv_chunks(int n_row_tiles, const ChunkSplit& split, bool listed) {
  const int least = listed ? 1 : (n_row_tiles + 127) / 128, by_slots = split.slots / split.items;
  int n = n_row_tiles < kShortLists ? by_slots / 4 : by_slots;
  if (n > split.by_sets) n = split.by_sets;
  int worth = (n_row_tiles + kSplitRowTiles - 1) / kSplitRowTiles;
  const int most = listed || n_row_tiles < kMaxRanges * kSplitRowTiles ? kMaxRanges - 1 : kMaxRanges;
  if (worth > most) worth = most;
  if (n > worth) n = worth;
  return n > least ? n : least;
}
bool dkdv_chunks_pay(int n, int chunk, const ChunkSplit& split, int whole, int cut, int64_t total) {
  if (16 * cut > 15 * whole) return false;
  if (16 * n * split.items > 15 * split.slots && 8 * chunk > 7 * whole && 5 * total > (int64_t)split.slots * whole) return false;
  return whole >= 3 * kSplitRowTiles || 17 * total <= (int64_t)4 * split.slots * whole;
}

// dK/dV of a dense map runs over equal chunks of at most 128 row tiles (few heads: more and shorter ones, see above), each with a set of partials of its
// own, later chunks adding to what the earlier ones wrote.  The key tiles below a chunk's first anchor have equally long
// lists, which balances the workgroups the way the paper's segments do; but a small last chunk leaves most of the
// chip idle, and every chunk writes and sums all partials again.  dK/dV + reduction, us, chunks of 64 / up to 128:
// L = 1,391 361 / 311 (D = 128 482 / 389), L = 2,600 1,006 / 976, ten segments of 2,048 anchors 49,000 / 48,100;
// chunks of 128 and a remainder lose at L = 2,600 (998), whole segments of any length at 3,000 anchors of D = 128
// (1,493 against 1,431).
hipError_t DkdvLauncher::add(const BwdParams& rows, int key_lo, int a_hi, int acc_below) {
  const int n_rt = rows.rt_hi - rows.rt_lo;
  if (n_rt <= 0) return hipSuccess;
  const int A = p_.tm.A;
  const bool listed_map = p_.tm.row_tok != nullptr;
  const int chunk = (n_rt + rows.n_chunks - 1) / rows.n_chunks;
  for (int c0 = rows.rt_lo; c0 < rows.rt_hi; c0 += chunk) {
    const int c1 = c0 + chunk < rows.rt_hi ? c0 + chunk : rows.rt_hi;
    const bool partial = c0 != rows.rt_lo || c1 != rows.rt_hi;
    const int c_a_hi = listed_map || c1 * A > a_hi ? a_hi : c1 * A;
    // (where a listed row tile ends is not known here: its first chunk leaves every key's sum, zero if no row of it sees the key)
    const int c_start = listed_map ? a_hi : c0 * A;
    const int c_acc = c0 == rows.rt_lo || acc_below == INT_MAX ? acc_below : (acc_below > c_start ? acc_below : c_start);
    const hipError_t e = add_range(c0, c1, rows, rows.cropped || partial, key_lo, c_a_hi, c_acc);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t DkdvLauncher::add_range(int rt_lo, int rt_hi, const BwdParams& rows, bool clip, int key_lo, int a_hi, int acc_below) {
  DkdvRange& r = range_[n_];
  r.rt_lo = rt_lo;
  r.rt_hi = rt_hi;
  r.s_lo = rows.s_lo;
  r.s_hi = rows.s_hi;
  r.clip_rows = clip ? 1 : 0;
  r.n_d0_tiles = (a_hi + kKeysPerTile - 1) / kKeysPerTile;  // depth-0 key tiles visible to rows < a_hi ...
  r.d0_tile_lo = key_lo / kKeysPerTile & ~1;                // ... from the (even) tile pair of the first visible key on
  r.set = n_;
  // pairs wholly below the segment's first anchor see every row tile (equal lists); the others shrink
  const int n_pairs = (r.n_d0_tiles - r.d0_tile_lo + 1) / 2;
  const int equal = acc_below == INT_MAX ? 0 : (acc_below / kKeysPerTile - r.d0_tile_lo) / 2;
  const int shrinking = n_pairs - (equal > 0 ? equal : 0);
  constexpr int kPasses = 8;  // (four: dK/dV at 4,096 anchors in two chunks 2,231 instead of 2,178 us)
  r.d0_step = (shrinking + kPasses - 1) / kPasses;
  if (r.d0_step < 1) r.d0_step = 1;
  r.d0_split = n_pairs - shrinking + r.d0_step;
  if (r.d0_split > n_pairs) r.d0_split = n_pairs;
  key_end_[n_] = a_hi;
  acc_below_[n_] = acc_below;
  ++n_;
  return n_ == p_.part_sets ? finish() : hipSuccess;
}

hipError_t DkdvLauncher::finish() {
  if (n_ == 0) return hipSuccess;
  BwdParams& p = p_;
  const int n = n_, D = D_;
  n_ = 0;
  p.rt_lo = range_[0].rt_lo;
  p.rt_hi = range_[n - 1].rt_hi;
  p.s_lo = range_[0].s_lo;
  p.s_hi = range_[n - 1].s_hi;
  p.clip_rows = 0;
  p.n_d0_items = 0;
  PartSets sets{};
  sets.n = n;
  sets.key_lo = INT_MAX;
  for (int i = 0; i < kMaxRanges; ++i) p.range[i].first_item = INT_MAX;
  for (int i = 0; i < n; ++i) {  // the last ranges, which see the most keys, first
    DkdvRange& r = p.range[i] = range_[n - 1 - i];
    r.first_item = p.n_d0_items;
    p.n_d0_items += (r.n_d0_tiles - r.d0_tile_lo + 1) / 2 * p.Hq;  // key-tile pairs x query heads
    p.clip_rows |= r.clip_rows;
    sets.key_first[r.set] = r.d0_tile_lo * kKeysPerTile;
    sets.key_end[r.set] = key_end_[r.set];
    sets.acc_below[r.set] = acc_below_[r.set];
    if (sets.key_first[r.set] < sets.key_lo) sets.key_lo = sets.key_first[r.set];
    if (sets.key_end[r.set] > sets.key_hi) sets.key_hi = sets.key_end[r.set];
  }
  p.n_chain_items = p.tm.n_csub > 0 ? (p.rt_hi - p.rt_lo) * p.Hkv : 0;
  const bool sv_dkdv = p.shared_dk_part != nullptr;  // (first-layer form)
  const bool listed_map = p.tm.row_tok != nullptr;
  {
    const dim3 grid((unsigned)(p.n_d0_items + p.n_chain_items + (with_dq_ ? (p.rt_hi - p.rt_lo) * p.Hq : 0)));
    TimedSpan span(timer_, kKindDkDv, stream_);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream_, p); };
    auto both = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream_, p, p); };
    auto pick = [&](auto rows) {
      constexpr int ROWS = decltype(rows)::value;
      if (with_dq_ && D == 64) sv_dkdv ? both(bwd_kernel<64, ROWS, true>) : both(bwd_kernel<64, ROWS, false>);
      else if (with_dq_) both(bwd_kernel<128, ROWS, false>);
      else if (D == 64) sv_dkdv ? go(dkdv_kernel<64, ROWS, true>) : go(dkdv_kernel<64, ROWS, false>);
      else sv_dkdv ? go(dkdv_kernel<128, ROWS, true>) : go(dkdv_kernel<128, ROWS, false>);
    };
    const int apart = D == 64 ? kRowsApart<64> : kRowsApart<128>;
    if (listed_map && p.near_rows) pick(std::integral_constant<int, kRowsListed>{});
    else if (listed_map) pick(std::integral_constant<int, kRowsListedFar>{});
    else if (p.near_rows && apart % p.tm.K == 0) pick(std::integral_constant<int, kRowsWhole>{});
    else if (p.near_rows && p.tm.A * p.tm.K > kRowsPerTile - apart) pick(std::integral_constant<int, kRowsMost>{});
    else pick(std::integral_constant<int, kRowsFar>{});
    const hipError_t e = span.finish();
    if (e != hipSuccess) return e;
  }
  const size_t n4 = 2 * (size_t)(sets.key_hi - sets.key_lo) * p.Hkv * (D / 4);
  size_t blocks = (n4 + 255) / 256;
  if (blocks > kCus * 16) blocks = kCus * 16;
  const dim3 grid((unsigned)blocks), block(256);
  TimedSpan span(timer_, kKindReduce, stream_);
  auto sum = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, stream_, p, sets); };
  // Four heads' loads together where the sum is short or of several sets (which are those of few heads): a thread's time is then
  // one round trip after the other.  One set of 128 MiB or more is summed at the memory system's rate, and loses.  us per launch, one /
  // four: 64 heads, 128 anchors 4.9 / 4.5, 1,000 9.1 / 8.0, K = 4 2,048 12.6 / 13.1, in segments of 1,024 to 8,192 11.2, 18.7, 26.6,
  // 32.8 / 10.8, 17.4, 25.4, 32.3 (the first 4,096), of 2,048 to 20,480 43.5, 58, 72, 150 / 44.8, 61, 77, 158 (6,144, 8,192, 10,240, 20,480
  // anchors); 32 heads at D = 128, 2,048 anchors 18.0 / 16.7, 4,096 31 / 32.5, 10,240 74 / 82; several sets, one after the other / four: 4 heads
  // 1,000 anchors 5.7 / 4.7, 2,048 7.5 / 4.7, in segments of 1,024 8.6 / 6.1, 16 heads 8.9 / 7.4.
  constexpr size_t kLongSum = (size_t)128 << 20;
  const bool longer = 2 * (size_t)(sets.key_hi - sets.key_lo) * p.Hq * D * sizeof(float) >= kLongSum;
  auto form = [&](auto d) {
    constexpr int DD = decltype(d)::value;
    if (n > 1) sum(reduce_partials_kernel<DD, kMaxRanges, 4>);
    else longer ? sum(reduce_partials_kernel<DD, 1, 1>) : sum(reduce_partials_kernel<DD, 1, 4>);
  };
  if (D == 64) form(std::integral_constant<int, 64>{});
  else form(std::integral_constant<int, 128>{});
  return span.finish();
}

// Pieces that each request's context is cut into, at most `laid_out` (which the workspace is laid out for: a thousand
// workgroups, at least four pages each).  Every piece pays the chain of round trips at a workgroup's start and end again, so
// fewer are taken, in two steps.  One workgroup per CU while pieces stay within kLongPiece pages: at D = 64 at least one, at
// D = 128 at most one, because there two wave groups fill a CU's LDS and a second workgroup costs them (see the launch).
// Otherwise at most two workgroups per CU, all running at once, while pieces stay within 32 pages (D = 64) or 20 (D = 128,
// one wave group).  All others as laid out: requests differ in length, and the longest one's pieces would be waited for.
// us per call (thirty in one graph), pieces a request (workgroups) as laid out / as taken: D = 64, 4 requests of 2,048 -
// 4,096 tokens 14.3 (16; 512) / 12.7 (8; 256), 16 of 1,000 15.9 (4; 512) / 13.6 (2; 256), 8 of 300 - 3,000 16.7 (12; 768) /
// 14.8 (4; 256), 4 of 8,000 - 20,000 28.6 (32; 1,024) / 26.3 (16; 512; 8 pieces 30.5), 64 of 100 - 1,000 27.2 (2; 1,024) /
// 19.8 (1; 512), 12 of 3,000 - 6,000 30.5 (11; 1,056) / 26.7 (5; 480; 6 pieces, 576 workgroups, 28.4); D = 128, 16 of 800 -
// 8,192 43.5 (16; 1,024) / 38.3 (8; 512), 3 of 13,701 - 18,407 26.7 (32; 384) / 25.4 (21; 252; 22 pieces, 264 workgroups,
// 28.5), 35 of 2,137 - 3,838 58.2 (8; 1,120) / 48.0 (3; 420; 4 pieces, 560 workgroups, 57.5). As laid out: D = 64, 16 of
// 2,000 - 20,000 78 (8; 1,024; 4 pieces 88), 55 of 1,691 - 2,469 56 (3; 1,320; 2 pieces, 880 workgroups, 59); D = 128, 27 of
// 3,914 - 6,578 81 (10; 1,080; 4 pieces of 26 pages 62), but 46 of 511 and one of 3,558 34 (6; 1,104; 2 pieces of 28 pages
// 49). 260 batches drawn over numbers and lengths, against all pieces as laid out (and one copying wave): evenly spread
// lengths, D = 64 / 128, -9 / -8 % in the mean, +5 / +2 % at worst; one to three long requests among short ones -11 / -4 %,
// +3 / +16 %.
// One piece leaves its rows' results itself, without the launch that merges pieces (4 of 64 - 256 tokens 9.4 / 6.6). Up to
// kOnePiece pages that is worth a longer chain in fewer workgroups, pieces 2 or 3 / 1: D = 64, one request of 512 tokens 9.1
// / 8.3, 4 of 768 10.4 / 10.3, 2 of 1,000 (16 pages) 9.8 / 12.4; D = 128, 4 of 512 11.8 / 11.2, 4 of 768 12.5 / 13.7.
constexpr int kOnePiece64 = 12, kOnePiece128 = 8, kLongestPiece64 = 32, kLongestPiece128 = 20;  // pages
int draft_pieces(int64_t wgs_per_piece, int max_pages, int laid_out, int D) {
  auto within = [&](int64_t n) { return (int)(n < 1 ? 1 : n < laid_out ? n : laid_out); };
  auto pages = [&](int n) { return (max_pages + n - 1) / n; };
  if (max_pages <= (D == 64 ? kOnePiece64 : kOnePiece128)) return 1;
  const int one_per_cu = within((D == 64 ? kCus + wgs_per_piece - 1 : kCus) / wgs_per_piece);
  if (pages(one_per_cu) <= kLongPiece) return one_per_cu;
  const int two_per_cu = within(2 * kCus / wgs_per_piece);
  return pages(two_per_cu) <= (D == 64 ? kLongestPiece64 : kLongestPiece128) ? two_per_cu : laid_out;
}

hipError_t launch_draft_decode(const DecodeParams& pin, int D, hipStream_t stream) {
  DecodeParams p = pin;
  p.n_splits = draft_pieces((int64_t)p.C * p.Hkv, p.max_pages, p.n_splits, D);
  p.group = p.Hq / p.Hkv;
  p.group_reciprocal = small_reciprocal(p.group);
  p.by_splits = make_divisor(p.n_splits);
  const int row_waves = p.rows_pad / 32;  // 1 .. 4
  const dim3 grid((unsigned)p.n_splits, (unsigned)p.Hkv, (unsigned)p.C);
  const int64_t n_wg = (int64_t)p.C * p.Hkv * p.n_splits;
  const bool long_pieces = (p.max_pages + p.n_splits - 1) / p.n_splits > kLongPiece;  // pages of the longest request's pieces
  // Two groups of waves per workgroup cost twice the LDS. At D = 64 two such workgroups still share a CU (of one group, four
  // do), which is enough while there are no more, or where pieces are long and few; at D = 128 one does (of one group, two),
  // which pays while there is at most one per CU anyway. us per call, one / two groups (pages of the longest pieces;
  // workgroups): D = 64, 4 requests of 2,048 - 4,096 tokens (8; 256) 15.1 / 13.1, 64 of 100 - 1,000 (16; 512) 25.5 / 19.8, 64
  // of 512 - 8,192 (64; 1,024) 133 / 119, 16 of 2,000 - 20,000 (40; 1,024) 85 / 77, 55 of 1,691 - 2,469 (13; 1,320) 56.6 /
  // 56.6, 65 of 300 (5; 520) 14.3 / 16.8, 128 of 300 (5; 1,024) 20.9 / 25.1; D = 128, 2 of 10,800 - 20,000 (10; 256) 25.0 /
  // 21.8, 16 of 800 - 4,096 (16; 256) 33.0 / 25.7, 70 of 500 (8; 280) 23.3 / 27.0, 64 of 3,000 - 4,000 (16; 1,024) 110 / 115,
  // 64 of 512 - 8,192 (32; 1,024) 131 / 141, but 35 of 2,137 - 3,838 (20; 420) 48.9 / 48.1. More than 64 query rows make
  // eight waves or ten, too many for two per CU.
  const bool two = row_waves <= 2 && (D == 64 ? n_wg <= 2 * kCus || long_pieces : n_wg <= kCus);
  // Long pieces of requests of different lengths: with more workgroups than two per CU, those of the longest requests start
  // first. us per call in order of the request / by length: the 64 requests of 512 to 8,192 tokens above 141 / 119, at D =
  // 128 149 / 131, 16 of 2,000 - 20,000 84 / 77. Ranking costs most of a page's time: with pieces of 8 pages, 35 of 2,137 -
  // 3,838 at D = 128 took 70.8 / 74.7. Up to 64 requests, which one wave can rank; with more, a CU sees many anyway.
  p.by_length = p.C > 1 && p.C <= 64 && n_wg > 2 * kCus && long_pieces;
  // Copying waves: two, but with three row blocks at D = 128 one, because two workgroups of five waves share a CU's four
  // SIMDs badly (us, one / two copying waves, 96 query rows: 64 requests of 512 - 8,192 tokens 142 / 160, 32 of 1,000 - 4,096
  // 47 / 63, 128 of 300 23.5 / 26.6; but D = 64 64 of 512 - 8,192 144 / 134, and D = 128 with one, two and four row blocks
  // 123 / 119, 134 / 131 and 168 / 164 on that batch).
  const int copying = D == 128 && row_waves == 3 ? 1 : 2;
  const dim3 block((unsigned)(((two ? 2 : 1) * row_waves + copying) * 64));
  // (The bound of 576 threads, of which 384 are launched, has the compiler schedule for four waves per SIMD: 120
  // against 136 us on the 64 requests of 512 to 8,192 tokens.  The other forms run the same with either bound.)
  auto go = [&](auto one_tag) {
    constexpr bool ONE = decltype(one_tag)::value;
    auto run = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, stream, p); };
    if (D == 64) two ? run(draft_decode_kernel<64, 2, 576, ONE>) : run(draft_decode_kernel<64, 1, 384, ONE>);
    else two ? run(draft_decode_kernel<128, 2, 384, ONE>) : run(draft_decode_kernel<128, 1, 384, ONE>);
  };
  p.n_splits == 1 ? go(std::true_type{}) : go(std::false_type{});
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || p.n_splits == 1) return e;
  // threads per row and splits per thread: n_splits is at most 32
  auto merge = [&](auto kernel, int rows_per_wave) {
    const int per_block = 4 * rows_per_wave;
    hipLaunchKernelGGL(kernel, dim3((unsigned)((p.K * p.group + per_block - 1) / per_block), (unsigned)p.Hkv, (unsigned)p.C), dim3(256),
                       0, stream, p);
  };
  if (D == 64) {
    if (p.n_splits <= 2) merge(draft_decode_combine_kernel<64, 1, 2>, 4);
    else if (p.n_splits <= 8) merge(draft_decode_combine_kernel<64, 2, 4>, 2);
    else merge(draft_decode_combine_kernel<64, 4, 8>, 1);
  } else {
    if (p.n_splits <= 2) merge(draft_decode_combine_kernel<128, 1, 2>, 2);
    else if (p.n_splits <= 8) merge(draft_decode_combine_kernel<128, 2, 4>, 1);
    else merge(draft_decode_combine_kernel<128, 2, 16>, 1);
  }
  return hipGetLastError();
}

hipError_t launch_cast_bf16(const float* src, void* dst, size_t n, hipStream_t stream) {
  const size_t n4 = n / 4;
  if (n4 == 0) return hipSuccess;
  size_t blocks = (n4 + 255) / 256;
  if (blocks > kCus * 16) blocks = kCus * 16;
  hipLaunchKernelGGL(cast_bf16_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, src, (__bf16*)dst, n4);
  return hipGetLastError();
}

hipError_t measure_mfma_ceiling(hipStream_t stream, bool random_operands, float* tflops) {
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  const int blocks = cus * 8, iters = 4000;
  float* out = nullptr;
  e = hipMalloc(&out, (size_t)blocks * 256 * sizeof(float));
  if (e != hipSuccess) return e;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  e = hipEventCreate(&e0);
  if (e == hipSuccess) e = hipEventCreate(&e1);
  if (e == hipSuccess) {
    auto launch = [&] {
      if (random_operands) hipLaunchKernelGGL(mfma_ceiling_kernel<true>, dim3(blocks), dim3(256), 0, stream, out, iters);
      else hipLaunchKernelGGL(mfma_ceiling_kernel<false>, dim3(blocks), dim3(256), 0, stream, out, iters);
    };
    // warm-up: the clock settles over a few milliseconds of load
    for (int w = 0; w < 3; ++w) launch();
    (void)hipEventRecord(e0, stream);
    for (int w = 0; w < 3; ++w) launch();
    (void)hipEventRecord(e1, stream);
    e = hipEventSynchronize(e1);
    float ms = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    if (e == hipSuccess) *tflops = (float)(3.0 * (double)blocks * 4 * iters * 4 * 32768.0 / ((double)ms * 1e9));
  }
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  (void)hipFree(out);
  return e;
}

}  // namespace peagle
