// Internal layouts shared by the host API and the HIP kernels of libxsv (not part of the ABI).
//
// Packed cache of one layer (per head), private to the library:
//   keys    kc  [Tcap][64*bits/8 B]     one row per token, channel c at bit c*bits (little endian)
//           ks, kz [Tcap/G][64] fp32    scale / zero point per (group of G tokens, channel)
//   values  vc  [Tcap/64][64][64*bits/8 B]  blocks of 64 tokens, TRANSPOSED: one row per channel,
//                                       token j of the block at bit j*bits — so that 8 (16) tokens
//                                       of one channel are one dword, the unit the PV MFMA consumes
//           vs, vz [Tcap][64/G] fp32    scale / zero point per (token, group of G channels)
//   bits == 16: kc rows are 64 bf16, vc rows are 64 bf16 (still transposed in 64-token blocks).
//   token ids   tok_frame, tok_index [sets][Tcap] per layer; sets = 1 (one retained index set per layer, shared by
//               the heads) or H (one per head, see xsv_config.score_mode)
// Every layer has two such buffers; a step reads one and writes the other.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace xsv {

constexpr int kD = 64;         // head_dim
constexpr int kTile = 64;      // tokens per value block and per attention key tile
constexpr int kMaxBatch = 32;  // layers per batched launch
constexpr int kPoolParts = 4;    // partial sums per head of the pooled-query pass

struct CachePool {
  uint8_t* kc;
  float* ks;
  float* kz;
  uint8_t* vc;
  float* vs;
  float* vz;
  int32_t* tok_frame;
  int32_t* tok_index;
  int L, H, Tcap, bits, G;
  int sets;  // retained index sets per layer: 1, or H when every head selects for itself
  int buffers;  // 2: a step reads one buffer and writes the other; 1 (a cache that is never pruned: rows never move):
                // a step rewrites the blocks it touches in place

  // slab = one (buffer, layer); sizes in elements of the respective array
  __host__ __device__ size_t code_row_bytes() const { return (size_t)kD * bits / 8; }
  __host__ __device__ size_t code_slab() const { return (size_t)H * Tcap * code_row_bytes(); }
  __host__ __device__ size_t kparam_slab() const { return (size_t)H * (Tcap / G) * kD; }
  __host__ __device__ size_t vparam_slab() const { return (size_t)H * Tcap * (kD / G); }
  __host__ __device__ size_t tok_slab() const { return (size_t)(sets > 1 ? sets : 1) * Tcap; }
  __host__ __device__ size_t slab_index(int buf, int layer) const { return (size_t)buf * L + layer; }
};

// index of the score vector / keep list / token-id row that head h of `layer` uses
__host__ __device__ inline size_t list_index(int sets, int layer, int h) {
  return sets > 1 ? (size_t)layer * sets + h : (size_t)layer;
}

// One layer's view of the pool (device pointers of one buffer), head 0.
struct LayerCache {
  uint8_t* kc;
  float* ks;
  float* kz;
  uint8_t* vc;
  float* vs;
  float* vz;
  int32_t* tok_frame;
  int32_t* tok_index;
};

// (A 16-bit cache has no parameters: those four pointers are then meaningless, and nobody reads them.  No test for it here -
// a kernel's first loads wait behind this.)
__host__ __device__ inline LayerCache layer_cache(const CachePool& p, int buf, int layer) {
  const size_t i = p.slab_index(buf, layer);
  LayerCache c;
  c.kc = p.kc + i * p.code_slab();
  c.vc = p.vc + i * p.code_slab();
  c.ks = p.ks + i * p.kparam_slab();
  c.kz = p.kz + i * p.kparam_slab();
  c.vs = p.vs + i * p.vparam_slab();
  c.vz = p.vz + i * p.vparam_slab();
  c.tok_frame = p.tok_frame + i * p.tok_slab();
  c.tok_index = p.tok_index + i * p.tok_slab();
  return c;
}

// The layers one launch works on, and their frame tensors.
struct Batch {
  int n_layers;     // layers in this launch
  int layer0;       // pool index of the first
  uint32_t bufsel;  // bit i: buffer that currently holds layer (layer0+i)'s cache
  const uint16_t* q[kMaxBatch];
  const uint16_t* k[kMaxBatch];
  const uint16_t* v[kMaxBatch];
  uint16_t* out[kMaxBatch];
  int64_t q_sh, q_st, k_sh, k_st, v_sh, v_st;  // strides in elements

  __host__ __device__ int src_buf(int i) const { return (bufsel >> i) & 1; }
};

// Per-layer workspaces (device), indexed by pool layer.
struct Workspace {
  float* scores;      // [L][sets][Tcap + n]  importance of the middle tokens
  int32_t* keep;      // [L][sets][Tcap + n]  keep list
  float* qpart;       // [L][H][kPoolParts][64] partial weighted query sums
  uint64_t* sync;     // [L][sets] counters of front_kernel, zero between launches
  uint16_t* attn_o;   // [pieces][batch layers][H][ceil(n/32)] blocks of 32 rows x 64 fp16 mantissas of the unnormalized
                      // partial outputs, each block stored [16-byte piece 0..3][lane half][row] (4 KB)
  float* attn_ml;     // [pieces][batch layers][H][n][4]  softmax reference (log2 domain), row sum, row scale, -
  uint32_t* unit_done;  // [units of an attention launch] where the workgroups of a cut unit meet (attend.hip), zero between launches
  int scores_stride;  // Tcap + n
  int sets;           // lists per layer (CachePool::sets)
};

// ---- launchers (defined in the .hip files; every one only enqueues on `stream`) -----------------

constexpr int kMaxPieces = 16;  // workgroups that may share one unit
// Words between the counters of two units: many workgroups look at them at the same time, and side by side in a few lines they
// held up each other and the partials' stores (24 layers with deferred joins: 1406 us, 1214 apart).
constexpr int kMeetStride = 64;
// LDS of a compute unit, and what attention launches that want none of front_kernel's workgroups beside them leave of it (launch_attend_t):
// too little for one (a static_assert there), enough for three of requant_kernel.
constexpr int kLdsOfComputeUnit = 160 * 1024, kLdsBesideAttention = 16 * 1024;
constexpr int kMergeInside = 5;  // see AttendArgs::merge_inside
constexpr int kMergeLooks = 32;  // see AttendArgs::merge_looks
// One layer of an attention launch: device pointers at head 0 of the buffer that holds the layer's cache, and of the
// frame's tensors.  (Resolved on the host: a workgroup's first tile waits behind whatever address arithmetic the
// kernel has to do, and the argument block stays small.)
struct AttendLayer {
  const uint32_t* kc;
  const float* ks;
  const float* kz;
  const uint32_t* vc;
  const float* vs;
  const float* vz;
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  uint16_t* out;
};
struct AttendArgs {
  AttendLayer layer[kMaxBatch];
  int n_layers, H, bits, G;
  uint32_t code_head, kparam_head, vparam_head;  // elements (dwords / floats) between two heads of kc|vc, ks|kz, vs|vz
  int64_t q_sh, q_st, k_sh, k_st, v_sh, v_st;    // strides of the frame tensors in elements
  uint16_t* attn_o;  // partial outputs of cut units, see Workspace
  float* attn_ml;
  uint32_t* unit_done;  // see Workspace
  int Tc, n;
  int variant;   // waves x query rows per wave of a workgroup: 0: 4 x 64, 1: 4 x 32, 2: 8 x 32, 3: 8 x 64
  int n_wgs;     // workgroups the (unit, tile) line is cut into (from plan_attend)
  int rows_wg;   // query rows per workgroup of this variant
  int cut;       // some unit is shared by several workgroups: partials are written and merged
  // The workgroups of a cut unit merge it, each a share of its rows (see meet in attend.hip), instead of a second launch: where the
  // library cuts one layer's units into three and more equal pieces, whatever runs beside it, and with other cuts of up to kMergeInside pieces
  // beside a chain with scores, where a second launch waits for places among the chain's workgroups.  us per pass, second launch
  // and inside: frame-wise attention of 16 x 1374 (5 pieces) 23.4 and 19.3, a bf16 cache grown by 16 frames, four layers, 5700
  // and 5440, one layer of 16 x 1374 without scores 50.5 and 46.6, one of 5 x 539 in 11 pieces 41 and 33, six 2-bit layers of 12 x 777 in
  // 8 282 and 272 (within what that case's runs differ by); two pieces of 9 x 501 17.8 and 18.4.  (With the last workgroup merging all by itself, 6 us for five
  // pieces of 512 rows where four that share it take 2, 24 layers with deferred joins took 1305 and not 1212.)
  int merge_inside;
  int equal_ranges;  // > 0: every unit is cut into exactly this many key ranges, at the same tiles:
  // range p of a unit is its tiles [range_begin[p], range_begin[p + 1]); chosen on the host so that the ranges
  // COST the same (a tile of the frame's own bf16 rows takes longer to stage than a tile of packed codes), or
  // so that the last one is deliberately short (see xsv_set_short_range)
  int32_t range_begin[17];
  int xcd_ranges;  // > 0: every unit is cut into this many key ranges and the grid is permuted for L2 sharing
  int xcd_heads;   // with xcd_ranges: (layer, head) pairs rather than (layer, head, range) triples are dealt to the XCDs
  int short_last;   // the last of a unit's equal_ranges was made short (see range_begin)
  // Workgroups that merge inside wait for the others of their unit: only where all units are cut alike, so that its workgroups end
  // together - a 2-bit stack on a line partition is 1 % slower with it - and no more of them than have a place at once.  (Another
  // stream's work, or a chain that deferred joins left running, may hold places all the same: then the number of looks bounds the wait.
  // Frame-wise attention behind deferred steps of 16 x 1374 / 16 x 700: 315 and 301, 222 and 206 us with the second launch and inside.)
  int merge_waits;
  // How often such a workgroup looks for the others before it leaves them its share (a look takes about 0.7 us).  Long enough for
  // those that started late because a chain still held their compute units.  us at 0 / 4 / 8 / 16 / 32 / 64 looks: 24 layers with
  // deferred joins 1283 / 1238 / 1224 / 1212 / 1214 / 1215, six 2-bit layers of 12 x 777, deferred, 310 / 310 / 308 / 296 / 258 / 253.
  // Two streams of 16 x 1374 at a time, whose grids do not fit the chip together, would rather not wait: 340 / 350 / 360 / - / 361.
  int merge_looks;
  float qscale;  // softmax scale * log2(e)
};
struct AttendPlan {
  int n_wgs, rows_wg, max_pieces;
};
// Chooses the grid: at most want_wgs workgroups, pieces of at least 4 tiles, and no unit shared by
// more workgroups than the partial workspace (part_rows rows) and the merge can hold.
AttendPlan plan_attend(int variant, int n_layers, int H, int n, int Tc, int want_wgs, size_t part_rows);
void partition_query(long long n_units, int n_tiles, int n_wgs, int wg, long long* begin, long long* end);
void partition_unit_query(long long n_units, int n_tiles, int n_wgs, int unit, int* first_wg, int* last_wg);
// `between` (optional): an event recorded after the attention kernel, before the merge kernel.
hipError_t launch_attend(const AttendArgs& a, hipStream_t stream, hipEvent_t between = nullptr);
int attend_rows_per_workgroup(int variant);
int attend_places_per_cu(int variant, int G);  // workgroups that a compute unit holds at once
bool attend_merges_inside(int variant, int n_layers);  // the shape has kernels that can (see AttendArgs::merge_inside)

// Pool, score and select (score_select.hip).  One layer: device pointers, resolved on the host.
struct FrontLayer {
  const uint16_t* q;   // head 0
  const uint8_t* kc;   // packed keys, scales and zero points of head 0 (plain keys: a bf16 tensor [H][P][64], T_first = 0)
  const float* ks;
  const float* kz;
  float* qpart;        // [H][kPoolParts][64]
  float* scores;       // first list of the layer
  int32_t* keep;
  uint64_t* sync;      // see Workspace
};
struct FrontCommon {
  int64_t q_sh, q_st;  // strides in elements
  int n_layers, H, n, n_special, pool_size;
  int T_first, P, k, T_cur;  // middle = cache positions [T_first, T_first + P), k of them are kept
  int head_rows;       // key rows between two heads
  int stride;          // between two lists
  int per_head;        // 1: no averages over heads, head h has list h of the layer
  int polls;           // how often front_kernel looks for the pool before it pools by itself (a matter of time only)
  int blocks;          // score workgroups per list (filled by the launchers)
};
template <int LAYERS>
struct FrontArgsT {
  FrontCommon c;
  FrontLayer layer[LAYERS];
};
using FrontArgs = FrontArgsT<kMaxBatch>;
// Scores and keep lists of the layers' middle tokens, 0 < k < P.
hipError_t launch_front(FrontArgs& a, int bits, int G, hipStream_t stream);
// Scores of plain bf16 keys: two launches, no counters.
hipError_t launch_score(const FrontArgs& a, hipStream_t stream);

struct SelectArgs {
  const float* scores;  // [lists][scores_stride]
  int32_t* keep;        // [lists][keep_stride]
  int scores_stride, keep_stride;
  int P, k, T_first, T_cur;
};
hipError_t launch_select(const SelectArgs& a, int n_lists, hipStream_t stream);
// keep = 0..T-1 (keep_middle) or first ∪ current
hipError_t launch_fill_keep(int32_t* keep, int T_first, int P, int T_cur, bool keep_middle, hipStream_t stream);

struct RequantArgs {
  CachePool pool;
  Batch b;
  Workspace ws;
  int Tc, n, Tn;  // old cache length, frame tokens, new cache length (= keep length)
  int frame_id;
  // new positions [0, identity_end) keep their cache row (first frame, or everything cached when nothing is pruned),
  // positions [Tn - n, Tn) are the frame's rows; only the positions in between are looked up in the keep list
  int identity_end;
  // the leading stable_blocks blocks of 64 positions hold the same cached rows as before the step (whole blocks inside
  // [0, identity_end)): such a block is re-quantized from what it already holds, and once that reproduces it bit for
  // bit - flagged per (layer, head, block) by the step that saw it happen - it never changes again and is skipped
  int stable_blocks;
  uint8_t* stable_flag;  // [L][H][Tcap / 64]
  int first_block;       // blocks in front of it are flagged, as the host knows (16 bits without a budget; else 0)
  int carry_values;      // xsv_config.value_mode == 1: value rows that come from the cache keep their codes and parameters
};
hipError_t launch_requant(const RequantArgs& a, hipStream_t stream);
hipError_t launch_zero_bytes(uint8_t* p, size_t n, hipStream_t stream);  // a fill kernel (no memset node)

// A plain tensor [H][T][64] quantized to canonical codes, scales and zero points (keys: groups of G tokens per channel;
// values: groups of G channels per token).  H <= 65536 (grid.y), x 16-byte aligned.
struct QuantizeArgs {
  const uint16_t* x;
  uint8_t* codes;  // [H][T][64]
  float* scale;    // keys [H][ceil(T/G)][64], values [H][T][64/G]
  float* zero;
  int H, T;
  bool wide;  // codes is 16-byte aligned
};
hipError_t launch_quantize_plain(const QuantizeArgs& a, int bits, int G, bool keys, hipStream_t stream);

// Canonical (one code per byte, untransposed) copies of one layer buffer → device arrays.
struct UnpackArgs {
  CachePool pool;
  int buf, layer, T;
  uint8_t* k_codes;  // [H][T][64] or null
  float* k_scale;    // [H][ceil(T/G)][64]
  float* k_zero;
  uint8_t* v_codes;
  float* v_scale;  // [H][T][64/G]
  float* v_zero;
  uint16_t* k_bf16;  // [H][T][64] dequantized view / stored rows
  uint16_t* v_bf16;
};
hipError_t launch_unpack(const UnpackArgs& a, hipStream_t stream);

}  // namespace xsv
