// Kernel parameter blocks and host launchers of the attention path.
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

#include "tilemap.h"

namespace peagle {

struct FwdParams {
  const __bf16* q;
  const __bf16* k;
  const __bf16* v;
  __bf16* o;
  float* lse;          // [Hq, T]
  DeviceTileMap tm;
  int L, T, Hq, Hkv;
  int rt_lo, rt_hi;    // row tiles of the segment
  int group;           // query heads per KV head
  Divisor by_kv, by_heads;  // by Hkv; by the workgroups that share a KV head and a row tile (filled by the launcher)
  float c_log2;        // softmax scale * log2(e)
  int mean_tiles;      // mean length of the row tiles' lists over the whole length-L problem
  const __bf16* v_shared;  // null, or [Hkv, D]: the value row of every chain key (first-layer form; v then holds
                           // the depth-0 rows only)
  const __bf16* d_o;       // null, or the backward's dO (a whole step): the forward then leaves the backward's per-row terms
  float* delta;            // [Hq, T], as in BwdParams
  float* nlse;
};

// Row tiles whose sums over the depth-0 keys make one set of partials (a segment, or a chunk of a long one), and the work on
// those keys; filled by the launcher.
struct DkdvRange {
  int rt_lo, rt_hi, s_lo, s_hi;
  int clip_rows;              // [rt_lo, rt_hi) covers only part of the segments s_lo..s_hi
  int d0_tile_lo, n_d0_tiles; // depth-0 key tiles visible to the rows are [d0_tile_lo, n_d0_tiles)
  int d0_split, d0_step;      // their pairs are dealt in passes, [0, d0_split) then d0_step at a time
  int first_item;             // of the launch's work items, INT_MAX: no such range
  int set;                    // of partials
};
constexpr int kMaxRanges = 4;  // of one launch

// How many chunks at most a range of rows may be cut into to fill the chip: by the slots that its work items leave, and by
// the sets of partials that a launch sums.
struct ChunkSplit {
  int items, slots, by_sets;
};

struct BwdParams {
  const __bf16* q;
  const __bf16* k;
  const __bf16* v;
  const __bf16* o;
  const __bf16* d_o;
  const float* lse;    // [Hq, T]
  __bf16* dq;
  float* dk_acc;       // [T, Hkv, D]
  float* dv_acc;
  float* delta;        // workspace [Hq, T]: -rowsum(dO * O), written by the dQ kernel or, for one grid, before it
  float* nlse;         // workspace [Hq, T]: -lse / scale, likewise
  float* dk_part;      // workspace [Hq, L64, D]: per-query-head dK of the depth-0 keys, of the first range of rows of a launch
  float* dv_part;
  float* part_more;    // workspace [part_sets - 1][dK, dV][part_stride]: of the others
  size_t part_stride;
  int part_sets;       // as many ranges of rows as one launch may take
  int n_chunks;        // that dK/dV of the row range is run over, see dkdv_chunks()
  DeviceTileMap tm;
  int L, T, Hq, Hkv, L64;
  int group;            // query heads per KV head
  Divisor by_kv, by_group;
  int rt_lo, rt_hi;
  int s_lo, s_hi, cropped;  // segment boundary indices of the row range; cropped: rt_hi cuts the last segment short
  int n_d0_items;       // filled by the launcher: depth-0 work items (key-tile pairs x query heads) of all ranges
  int n_chain_items;    // filled by the launcher: chain work items; dQ's, where it shares the grid, come behind
  int clip_rows;        // filled by the launcher, as in DkdvRange: of all rows, for the chain items
  int near_rows;        // Q-shaped tensors and the [Hq, T] statistics span less than 4 GiB: row copies may use 32-bit offsets
  int mean_tiles;       // as in FwdParams
  int chain_accumulate; // chain keys: add to dk_acc/dv_acc instead of overwriting
  float c_log2, scale;
  const float* rope_table;  // null, or [positions][2][D/2] cosines and sines: q and k are rotated copies, and dQ / dK
                            // are turned back to the unrotated inputs' frame before they are stored
  // First-layer form (every chain key carries the same K and V vector, rotated by its position): v_shared [Hkv, D]
  // is the value row of every chain key (v then holds the depth-0 rows only), and the chain keys' dK / dV are not
  // stored per key but summed over the 32 keys of a wave into shared_dk_part / shared_dv_part
  // [(row tile * chain-tile pairs + pair) * 4 + wave][Hkv][D], which a reduction then adds up.  All null otherwise.
  const __bf16* v_shared;
  float* shared_dk_part;
  float* shared_dv_part;
  DkdvRange range[kMaxRanges];  // filled by the launcher, in the order of their items
};

// Inference-side drafting step (Sec. 2 of the paper: all K draft positions in one forward pass): the K
// rows of each request against its paged KV cache plus the K new keys.
struct DecodeParams {
  const __bf16* q_new;         // [C, K, Hq, D]
  const __bf16* k_new;         // [C, K, Hkv, D]
  const __bf16* v_new;
  const __bf16* k_pages;       // [n_pages, Hkv, 64, D]
  const __bf16* v_pages;
  const int32_t* block_table;  // [C, max_pages] page of each 64-token block of a request's context
  const int32_t* ctx_len;      // [C] cached tokens per request
  __bf16* o;                   // [C, K, Hq, D]
  float* lse;                  // [C, Hq, K]
  int32_t* status;             // [C] or null: 1 if the request's block table or length was out of range
  float* part_o;               // workspace [C, Hkv, n_splits, rows_pad, D]: unnormalised partial outputs
  float* part_ml;              // workspace [C, Hkv, n_splits, 3, rows_pad]: reference max (log2), row sum, flag
  int C, K, Hq, Hkv, n_pages, max_pages, rows_pad;
  int n_splits;                // pieces the workspace is laid out for; the launcher replaces it by draft_pieces()
  int group;                   // filled by the launcher, like what follows: query heads per KV head,
  uint32_t group_reciprocal;   // its small_reciprocal()
  Divisor by_splits;
  int by_length;               // requests take the workgroups by falling context length (C <= 64)
  float c_log2;
};
hipError_t launch_draft_decode(const DecodeParams& p, int D, hipStream_t stream);
// Pieces per request that the launch takes (host only): workgroups per piece are requests x KV heads, `laid_out` is the
// number of pieces that the workspace has records for.
int draft_pieces(int64_t wgs_per_piece, int max_pages, int laid_out, int D);

// Optional per-kernel timing: an event pair is recorded around every launch on the launch stream.
enum KernelKind { kKindFwd = 0, kKindDq = 1, kKindDkDv = 2, kKindReduce = 3, kKindRope = 4, kNumKinds = 5 };
struct KernelTimer {
  struct Span { hipEvent_t start, stop; int kind; };
  std::vector<Span> spans;
  hipError_t begin(int kind, hipStream_t stream);
  hipError_t end(hipStream_t stream);
  // Waits for the recorded work, adds the elapsed ms per kind into ms[] / launches[], frees the events.
  hipError_t collect(float* ms, int32_t* launches);
  ~KernelTimer();
};

hipError_t launch_fwd(const FwdParams& p, int D, hipStream_t stream, KernelTimer* timer = nullptr);
// Do dK/dV and dQ of a backward over n_row_tiles row tiles run as one grid?  terms_left: the forward of the same call leaves
// the per-row terms; otherwise launch_row_terms() has to.  sv: first-layer form.
bool backward_in_one_grid(int D, int mean_tiles, int n_row_tiles, int Hq, bool terms_left, bool sv);
// The per-row terms of the row range (D = 64).
hipError_t launch_row_terms(const BwdParams& p, hipStream_t stream);
// dQ of the row range, and the per-row terms that dK/dV consumes.
hipError_t launch_dq(const BwdParams& p, int D, hipStream_t stream, KernelTimer* timer = nullptr);
// dK/dV of segments, in order.  Up to part_sets ranges of rows - segments, or chunks of a long one - share a launch, and the
// sum of their partials is taken range by range, as if each had been launched by itself.  with_dq (backward_in_one_grid()): dQ
// of the same rows too.
class DkdvLauncher {
 public:
  // p: everything but the rows
  DkdvLauncher(const BwdParams& p, int D, bool with_dq, hipStream_t stream, KernelTimer* timer = nullptr)
      : p_(p), D_(D), with_dq_(with_dq), stream_(stream), timer_(timer) {}
  // Segment of the row tiles and segment boundaries in `rows`; key_lo: first depth-0 key it sees; a_hi: its end anchor
  // (depth-0 keys [key_lo, a_hi) are visible); depth-0 keys with anchor below acc_below are added to dk_acc/dv_acc, the
  // others overwritten.
  hipError_t add(const BwdParams& rows, int key_lo, int a_hi, int acc_below);
  hipError_t finish();  // launches what is left

 private:
  hipError_t add_range(int rt_lo, int rt_hi, const BwdParams& rows, bool clip, int key_lo, int a_hi, int acc_below);
  BwdParams p_;
  const int D_;
  const bool with_dq_;
  const hipStream_t stream_;
  KernelTimer* const timer_;
  int n_ = 0;                      // ranges waiting
  DkdvRange range_[kMaxRanges];    // ... by set
  int key_end_[kMaxRanges], acc_below_[kMaxRanges];
};
// Chunks that dK/dV of a range of row tiles is run over (listed: of a sampled or packed map, if dkdv_chunks_pay()), split:
// dkdv_chunk_split() of the problem and of the number of ranges that it has of itself.
int dkdv_chunks(int n_row_tiles, const ChunkSplit& split, bool listed);
ChunkSplit dkdv_chunk_split(int D, int L64, int Hq, int n_ranges);
// Whether n chunks of `chunk` row tiles pay that leave `cut` row tiles of the longest walk of a key-tile pair, which is `whole`;
// total: row tiles that all walks of the range take together.
bool dkdv_chunks_pay(int n, int chunk, const ChunkSplit& split, int whole, int cut, int64_t total);
// Sets of partials worth having for a problem of n_ranges ranges of rows in all: several where a range's work items leave
// slots idle.
int dkdv_part_sets(int D, int L64, int Hq, int n_ranges);
// Dense bf16 MFMA issue loop on every CU: the measured matrix-core ceiling of the device, in TFLOP/s, on
// constant small-integer operands or on changing pseudo-random ones (the chip clocks lower under the latter).
hipError_t measure_mfma_ceiling(hipStream_t stream, bool random_operands, float* tflops);
hipError_t launch_cast_bf16(const float* src, void* dst_bf16, size_t n, hipStream_t stream);
// Rotary embedding: table [n_pos][2][D/2] of cosines and sines; rotation of a bf16 [T, H, D] tensor
// by each token's position (inverse: the transpose).
hipError_t launch_rope_table(double base, int D, int n_pos, float* table, hipStream_t stream);
// First-layer form: expansion of (own depth-0 rows, one shared vector for every later token) into a full
// [T, H, D] tensor, rotated when a table is given.
hipError_t launch_expand_shared(const void* x0, const void* x_shared, void* out, int H, int T, int L0, int D,
                                const DeviceTileMap& tm, int L, const float* table_or_null, hipStream_t stream);
// Column sums of part_k / part_v [rows][cols] (the per-wave sums of the chain keys' gradients) into
// dk_shared / dv_shared [cols], in a fixed order.
hipError_t launch_shared_grads(const float* part_k, const float* part_v, int rows, float* dk_shared, float* dv_shared,
                               int cols, hipStream_t stream);
hipError_t launch_rope_rotate(const void* x, void* out, int H, int T, int D, const DeviceTileMap& tm, int L,
                              const float* table, bool inverse, hipStream_t stream, KernelTimer* timer = nullptr);

}  // namespace peagle
