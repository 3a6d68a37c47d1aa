// Fused dequantize + flash-style attention of one frame's queries over [packed cache ; frame]
// (paper Sec. 3.1 temporal attention, Sec. 3.3 dequantization at attention time) for gfx950.
//
// Work decomposition
//   workgroup = NW waves; each wave owns QB blocks of 32 query rows of one head and keeps, per
//   lane, the transposed tiles  S^T = K Q^T  (32 tokens x 32 queries per block)  and
//   O^T = V^T P^T  (64 channels x 32 queries per block) in MFMA 32x32x16 bf16 accumulators.  In
//   this orientation one lane holds the logits of ONE query, so the online-softmax row reductions
//   are in-lane plus one exchange with lane^32, and the exponentiated tile is already laid out as
//   the B operand of the PV product — provided the key rows of the first product are read in a
//   permuted order (tau below), which costs nothing.  Every K / V fragment read from LDS feeds QB
//   MFMAs.
//   The workgroup walks the key axis in tiles of 64 tokens (two half-steps of 32).  All waves
//   cooperatively dequantize a tile ONCE into LDS as bf16 (K row-major [token][channel], V
//   transposed [channel][token], the layout the packed cache already has), so the unpack/convert
//   cost is shared by NW*QB*32 queries (half of the threads stage K, the other half V, with the
//   same code on mirrored layouts).  LDS is double buffered; the next tile's packed codes are fetched into
//   registers before the current tile's MFMAs are issued, the group parameters of the tile after that on their way
//   to LDS (one float per thread).
//   Partition.  A unit is one (layer, head, block of NW*QB*32 query rows); its work is its key tiles.
//   Two forms, chosen by the host.  (a) Every unit is cut into the same number R of key ranges
//   (gridDim.x = units * R): the host passes where each range begins, placed so that the ranges cost
//   the same (a tile of the frame's own rows costs a little less than a cache tile, and the last
//   range may be made short on purpose so that its compute units are free early for the kernels
//   that run beside this one); the grid is permuted so that a head's workgroups run on one XCD
//   and share its L2: the query blocks of a range read the same tiles, the ranges of a query block the same
//   queries, and the merge, permuted alike, finds the partials there.  (b) Otherwise all units'
//   tiles form one line of n_units * n_tiles items cut into gridDim.x equal pieces, so that any
//   number of workgroups gets the same amount of work; a piece may end one unit and begin the
//   next, and the workgroup handles them one after the other.  In both forms a unit covered by one
//   workgroup is normalized and written directly; otherwise each workgroup writes an unnormalized
//   partial, and the unit's workgroups merge them together, or combine_kernel does (AttendArgs::merge_inside).
//   Softmax.  No row maximum and no rescaling on the common path: the reference of the exponent is the row maximum
//   of a range's first 32 tokens plus 8 powers of two, and probabilities may grow above 1 - they are as exact there, in bf16 as
//   in fp32.  Only when a tile's row sum passes 2^24 - looked at once per tile - are the references moved, which rescales sums and
//   accumulators (recenter).  The loop over full tiles is straight-line code: a ragged last tile (cache or frame) has its own,
//   simpler, code behind it.  NaN, infinite logits and overflowing accumulators send the workgroup through its tiles once more,
//   each row on its own (the careful pass).
//   The headroom is small on purpose.  Products of probability and value are accumulated at the probabilities' scale: at 2^-60
//   values below 2^-66 lose bits and below 2^-89 vanish.  At 2^-8 they keep what bf16 holds down to its smallest numbers.
//   What the loop's time goes to: vector issue first.  Per wave and tile 64 multiply-adds, 64 exponentials, 32 conversions, some 70 plain
//   instructions of dequantizing and of looking at the sums, and 40 MFMAs.  At the rates measured on this part (a plain instruction
//   4.9 cycles of a wave's issue, an exponential 8.6, an MFMA 7 beside the other wave's arithmetic) the two waves of a SIMD need
//   some 3290 cycles for that, against 2340 of the matrix pipe.  A 4-bit tile takes 3900 (a bf16 one 3400, where the same count
//   gives some 2750): 600 more, which no count here explains - the barrier of a tile, reads and writes of LDS, the prefetch.
//   v_dot2c_f32_bf16 must stay out of it: it executes on the matrix pipe (beside a wave that issues MFMAs back to back it makes no
//   progress at all), so row sums taken with it serialize MFMAs and softmax; they are MFMAs of their own here (sum_step).  At 16
//   heads, 1374 rows, 5470 keys, one key range per 512 rows: 1.88 -> 1.66 us per tile of a workgroup on the 4-bit cache (at 2.4 GHz; the
//   part grants 2.15 beside a chain and 2.0 with 24 layers per launch); a bf16 cache grown by 16 frames of 1374 tokens, four layers: 7220
//   -> 5780 us.
#include <cstddef>
#include <type_traits>

#include "xsv_internal.h"

namespace xsv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kLdsStride = 72;  // bf16 elements per LDS row: 64 + 8 pad (144 B, keeps 16 B alignment)
constexpr int kLdsTile = 64 * kLdsStride;  // elements of one K (or V) tile in LDS
// the kernel's local functions are called from several places and are large: without this some of them become calls whose
// captured registers go through memory
#define XSV_INLINE __attribute__((always_inline))
constexpr float kNegBig = -1.0e30f;
// References end here.  Logits (times the softmax scale, log2 domain) above this count as +infinity: fp32 does not resolve the
// difference of two such numbers anywhere near 1.
constexpr float kFar = 3.0e38f;
// A row's reference is put this many powers of two above its largest logit so far, so that sums over a whole range of like
// logits stay of the order of 1 (values up to the largest bf16 numbers do not overflow) ...
constexpr float kHeadroom = 8.0f;
// ... and moves when a row's sum passes this: 96 powers of two are left for what a single tile can add.  On a 2-bit cache of 24
// frames' selection the first tokens of a range lie 36 powers of two below the largest (89 at most).
constexpr float kSumLimit = 0x1p24f;

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  const f32x2 v = {a, b};  // one v_cvt_pk_bf16_f32: round to nearest even, a in the low half
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
__device__ __forceinline__ uint32_t pack_f16(float a, float b) {
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
}

// Row of the K tile that MFMA row i of S^T reads, so that accumulator register r of the lane
// half hh holds token 16*(r/8) + 8*hh + r%8 — the order in which the PV product consumes tokens.
__device__ __forceinline__ int tau(int i) {
  const int a = i >> 3;
  return 16 * (a >> 1) + 8 * ((i >> 2) & 1) + 4 * (a & 1) + (i & 3);
}

// code e (0 .. 32/BITS-1) of a packed dword as float; the masks are shared between neighbours
template <int BITS>
__device__ __forceinline__ void unpack_codes(uint32_t w, float* out) {
  if constexpr (BITS == 4) {
    uint32_t t0 = w & 0x0f0f0f0fu, t1 = (w >> 4) & 0x0f0f0f0fu;
    // (opaque to the optimizer, which would otherwise fold the masks into one bit-field extract
    // PER code in front of each conversion instead of the byte-select conversions below)
    asm volatile("" : "+v"(t0), "+v"(t1));
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      out[2 * b] = (float)((t0 >> (8 * b)) & 0xffu);  // v_cvt_f32_ubyte<b>
      out[2 * b + 1] = (float)((t1 >> (8 * b)) & 0xffu);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t t = (w >> (2 * i)) & 0x03030303u;
      asm volatile("" : "+v"(t));
#pragma unroll
      for (int b = 0; b < 4; ++b) out[4 * b + i] = (float)((t >> (8 * b)) & 0xffu);
    }
  }
}

// ---- staging of one key tile -------------------------------------------------------------------
// A tile is 64 tokens x 64 channels of K and of V.  It is cut into "items" of one dword of codes
// (8 or 16 elements; bf16 tiles: 16 bytes = 8 elements).  The first half of the workgroup's threads
// stages K, the second half V; both run the SAME code on different pointers, because the packed
// layouts mirror each other:  K item i = (token i / RI, channel run i % RI) with per-channel
// parameters,  V item i = (channel i / RI, token run i % RI) with per-token parameters, and the
// LDS tile of either is [row = i / RI][column run].  A thread stages items u, u + NH, .. (u = its
// index within its half, NH threads per half); NH is a multiple of RI, so all its items share the
// column run and (within a group) the parameters.
template <int BITS, int G, int NH>
struct Stage {
  static constexpr bool kQuant = BITS != 16;
  static constexpr int kPer = kQuant ? 32 / BITS : 8;  // elements per item
  static constexpr int kRI = kD / kPer;                 // items per row
  static constexpr int kItems = kTile * kRI;            // per tile and role
  static constexpr int kIter = kItems / NH;             // items per thread
  static constexpr int kRowStep = NH / kRI;             // rows between a thread's consecutive items
  // parameter sets per thread: with G = 32 the rows < 32 and >= 32 of a tile are different groups
  static constexpr int kSets = (G >= 64 || kIter == 1) ? 1 : 2;
  static_assert(kItems % NH == 0 && NH % kRI == 0, "thread count must tile the items");
  static_assert(kSets == 1 || (kIter % 2 == 0 && kRowStep * (kIter / 2) == 32), "two groups need an even split");
  // A tile has kPrm scales and kPrm zero points per role, consecutive in memory (K: [group][channel], V: [token][channel
  // group]).  Only the first tile of a range takes them from there; for the others they come through LDS, where they are
  // put a tile ahead (see PrmStage): held in registers across a tile's MFMAs, as the codes are, they would cost a
  // thread up to 64 registers.
  static constexpr int kPrm = kTile * kD / G;
};

// A tile on its way to LDS: packed codes or bf16 rows of the cache, or rows of the frame.  (Two types, held by two
// loops: one array for both costs register copies right behind the loads, which then wait for them.)
template <int BITS, int G, int NH>
struct CacheRegs {
  uint32_t w[Stage<BITS, G, NH>::kIter * (BITS == 16 ? 4 : 1)];
};
template <int NH>
struct FrameRegs {
  uint32_t w[512 / NH * 4];
};

// The parameters of one tile and role on their way to LDS: scales, then zero points, one float per thread and step.
template <int BITS, int G, int NH>
struct PrmStage {
  static constexpr int kFloats = 2 * Stage<BITS, G, NH>::kPrm;
  static constexpr int kIter = (kFloats + NH - 1) / NH;
  float x[kIter];
};

struct RolePtrs {      // what distinguishes the K half from the V half
  const uint32_t* codes;  // packed tile base of (layer, head): row-major [Tcap rows][row dwords]
  const float* ps;        // parameter arrays of (layer, head)
  const float* pz;
  uint16_t* lds;          // first of the two LDS tiles of this role (the second follows it)
  float* prm;             // first of the two LDS parameter blocks of this role (the second follows it)
  bool is_v;
};

template <int BITS, int G, int NH>
__device__ __forceinline__ void fetch_cache_tile(CacheRegs<BITS, G, NH>& st, const RolePtrs& rp, int tile, int u) {
  using S = Stage<BITS, G, NH>;
  constexpr int kRowDw = kD * BITS / 32;  // dwords per K row == dwords per V block row
  const uint32_t* base = rp.codes + (size_t)tile * kTile * kRowDw;
  if constexpr (!S::kQuant) {
#pragma unroll
    for (int it = 0; it < S::kIter; ++it) {
      const u32x4 v = reinterpret_cast<const u32x4*>(base)[u + it * NH];
      st.w[4 * it] = v[0]; st.w[4 * it + 1] = v[1]; st.w[4 * it + 2] = v[2]; st.w[4 * it + 3] = v[3];
    }
  } else {
#pragma unroll
    for (int it = 0; it < S::kIter; ++it) st.w[it] = base[u + it * NH];
  }
}

template <int BITS, int G, int NH>
__device__ __forceinline__ void fetch_params(PrmStage<BITS, G, NH>& st, const RolePtrs& rp, int tile, int u) {
  using P = PrmStage<BITS, G, NH>;
  constexpr int kPrm = Stage<BITS, G, NH>::kPrm;
#pragma unroll
  for (int it = 0; it < P::kIter; ++it) {
    const int i = u + it * NH;
    if (P::kFloats % NH == 0 || i < P::kFloats) st.x[it] = (i < kPrm ? rp.ps : rp.pz - kPrm)[(size_t)tile * kPrm + i];
  }
}

template <int BITS, int G, int NH>
__device__ __forceinline__ void store_params(const PrmStage<BITS, G, NH>& st, float* prm, int u) {
  using P = PrmStage<BITS, G, NH>;
#pragma unroll
  for (int it = 0; it < P::kIter; ++it) {
    const int i = u + it * NH;
    if (P::kFloats % NH == 0 || i < P::kFloats) prm[i] = st.x[it];
  }
}

// ps, pz: the tile's kPrm scales and zero points of this role, in LDS or in global memory
template <int BITS, int G, int NH>
__device__ __forceinline__ void store_cache_tile(const CacheRegs<BITS, G, NH>& st, uint16_t* lds, const float* ps, const float* pz, bool is_v,
                                                 int u) {
  using S = Stage<BITS, G, NH>;
  const int r0 = u / S::kRI, o = u % S::kRI;
  if constexpr (!S::kQuant) {
#pragma unroll
    for (int it = 0; it < S::kIter; ++it)
      *reinterpret_cast<u32x4*>(lds + (r0 + it * S::kRowStep) * kLdsStride + o * S::kPer) =
          u32x4{st.w[4 * it], st.w[4 * it + 1], st.w[4 * it + 2], st.w[4 * it + 3]};
  } else {
    // The cache's canonical view: (code - zero) exactly, ONE fp32 multiply by the scale, then bf16.
    // (A fused code * scale + (-zero * scale) would save an instruction per element, but it rounds
    // zero * scale first and so breaks ties differently: products of a small integer with
    // scale = range / levels land on bf16 midpoints often enough to move a dominant key's logit.)
#pragma unroll
    for (int set0 = 0; set0 < S::kSets; ++set0) {
      // 32-row half of the tile this set belongs to (a thread with a single item has a single row)
      const int set = (G >= 64) ? 0 : (S::kIter == 1 ? r0 / 32 : set0);
      float s[S::kPer], z[S::kPer];
      if (!is_v || kD / G == 1) {  // K: group `set`, channels o*kPer..;  V with one channel group: tokens o*kPer..
        const int off = (is_v ? 0 : set * kD) + o * S::kPer;
#pragma unroll
        for (int e = 0; e < S::kPer; e += 4) {
          const float4 a4 = *reinterpret_cast<const float4*>(ps + off + e), b4 = *reinterpret_cast<const float4*>(pz + off + e);
          s[e] = a4.x; s[e + 1] = a4.y; s[e + 2] = a4.z; s[e + 3] = a4.w;
          z[e] = b4.x; z[e + 1] = b4.y; z[e + 2] = b4.z; z[e + 3] = b4.w;
        }
      } else {  // V: tokens o*kPer.., channel group `set`
#pragma unroll
        for (int e = 0; e < S::kPer; ++e) {
          s[e] = ps[(o * S::kPer + e) * (kD / G) + set];
          z[e] = pz[(o * S::kPer + e) * (kD / G) + set];
        }
      }
#pragma unroll
      for (int it = set0 * (S::kIter / S::kSets); it < (set0 + 1) * (S::kIter / S::kSets); ++it) {
        float f[S::kPer];
        unpack_codes<BITS>(st.w[it], f);
        uint32_t pk[S::kPer / 2];
#pragma unroll
        for (int e = 0; e < S::kPer; e += 2) pk[e / 2] = pack_bf16((f[e] - z[e]) * s[e], (f[e + 1] - z[e + 1]) * s[e + 1]);
        uint16_t* dst = lds + (r0 + it * S::kRowStep) * kLdsStride + o * S::kPer;
#pragma unroll
        for (int w = 0; w < S::kPer / 8; ++w)
          *reinterpret_cast<u32x4*>(dst + w * 8) = u32x4{pk[4 * w], pk[4 * w + 1], pk[4 * w + 2], pk[4 * w + 3]};
      }
    }
  }
}

// Frame tiles (bf16 rows as given).  K half: 512 items of 16 bytes, item = (token i/8, channel run
// i%8), copied as they are.  V half: the tile must land transposed ([channel][token]); an item is
// (token octet, channel pair): eight 4-byte loads down the token axis (a wave's loads cover whole
// 128-byte rows), two byte-permutes per register pair, and two 16-byte LDS writes.
template <int NH>
struct FrameStage {
  static constexpr int kIterK = 512 / NH;  // 16-byte items per K thread
  static constexpr int kIterV = 256 / NH;  // 8-dword items per V thread
  static_assert(kIterK * 4 == kIterV * 8, "both roles stage the same number of registers");
};

// Frame tile, V half: which (channel pair c2 = 0..31, token octet tq) thread u of the V half stages first (its
// further items are NH / 32 octets further down).  Eight consecutive lanes take four channel pairs of two
// octets, so that their 16-byte LDS writes - rows 2 * c2 (+1) of 144 bytes, column 16 * tq - fall into eight
// different bank groups; with consecutive channel pairs on consecutive lanes they would share four.
__device__ __forceinline__ void frame_v_item(int u, int& c2, int& tq) {
  const int l = u & 63, w = u >> 6;
  c2 = 4 * (l >> 3) + (l & 3);
  tq = 2 * w + ((l >> 2) & 1);
}

// The frame's rows are read through a buffer resource that covers exactly the n rows of the (layer, head): the
// loads take one 32-bit offset register that never changes plus a scalar offset per tile (no 64-bit address per
// load), and rows past the frame read as zeros by the resource's range check (their logits are masked, their
// values must be finite).
struct FrameRows {
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t row_bytes;  // stride between rows
  uint32_t voff;       // this thread's byte offset inside a tile
};

__device__ __forceinline__ FrameRows frame_rows(const uint16_t* xh, int64_t x_st, int n, bool is_v, int u) {
  FrameRows f;
  f.row_bytes = (uint32_t)x_st * 2u;
  const uint32_t bytes = ((uint32_t)(n - 1) * (uint32_t)x_st + (uint32_t)kD) * 2u;
  f.rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(xh), 0, (int)bytes, 0x00020000);
  // K: item (token u/8, channels 8*(u%8)..);  V: item (token octet u/32, channel pair u%32)
  int c2, tq;
  frame_v_item(u, c2, tq);
  f.voff = is_v ? (uint32_t)(8 * tq) * f.row_bytes + 4u * c2 : (uint32_t)(u >> 3) * f.row_bytes + 16u * (u & 7);
  return f;
}

template <int NH>
__device__ __forceinline__ void fetch_frame_tile(FrameRegs<NH>& st, const FrameRows& f, bool is_v, int tile) {
  using F = FrameStage<NH>;
  const uint32_t tile_off = (uint32_t)tile * kTile * f.row_bytes;  // scalar
  if (!is_v) {
#pragma unroll
    for (int it = 0; it < F::kIterK; ++it) {  // items u + it * NH: NH / 8 rows further down
      const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(f.rsrc, f.voff, tile_off + it * (NH / 8) * f.row_bytes, 0);
      st.w[4 * it] = v[0]; st.w[4 * it + 1] = v[1]; st.w[4 * it + 2] = v[2]; st.w[4 * it + 3] = v[3];
    }
  } else {
#pragma unroll
    for (int it = 0; it < F::kIterV; ++it) {  // items u + it * NH: NH / 32 token octets further down
#pragma unroll
      for (int e = 0; e < 8; ++e)
        st.w[8 * it + e] = __builtin_amdgcn_raw_buffer_load_b32(f.rsrc, f.voff, tile_off + (it * (NH / 32) * 8 + e) * f.row_bytes, 0);
    }
  }
}

template <int NH>
__device__ __forceinline__ void store_frame_tile(const FrameRegs<NH>& st, uint16_t* lds, bool is_v, int u) {
  using F = FrameStage<NH>;
  if (!is_v) {
#pragma unroll
    for (int it = 0; it < F::kIterK; ++it) {
      const int i = u + it * NH;
      *reinterpret_cast<uint4*>(lds + (i >> 3) * kLdsStride + (i & 7) * 8) =
          make_uint4(st.w[4 * it], st.w[4 * it + 1], st.w[4 * it + 2], st.w[4 * it + 3]);
    }
  } else {
#pragma unroll
    for (int it = 0; it < F::kIterV; ++it) {
      int c2, tq;
      frame_v_item(u, c2, tq);
      tq += it * (NH / 32);
      uint32_t lo[4], hi[4];  // tokens 8tq.. of channel 2*c2 and of channel 2*c2+1
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        lo[k] = __builtin_amdgcn_perm(st.w[8 * it + 2 * k + 1], st.w[8 * it + 2 * k], 0x05040100u);
        hi[k] = __builtin_amdgcn_perm(st.w[8 * it + 2 * k + 1], st.w[8 * it + 2 * k], 0x07060302u);
      }
      *reinterpret_cast<uint4*>(lds + (2 * c2) * kLdsStride + 8 * tq) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
      *reinterpret_cast<uint4*>(lds + (2 * c2 + 1) * kLdsStride + 8 * tq) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    }
  }
}

// Partials of cut units pass between workgroups on different dies, whose caches do not see each other: agent-scope accesses go
// past them.  (With plain stores a workgroup would have to write its die's whole L2 back before it could say that it is done.)
constexpr int kAgentScope = 16;  // the sc1 bit of a buffer instruction
// The partial rows from a (piece, layer, head)'s on, see Workspace.  Another piece's are a scalar offset away (the host sees to
// it that all pieces of a launch lie within 2 GiB).
struct PartialRows {
  __amdgpu_buffer_rsrc_t o, ml;
};
__device__ __forceinline__ PartialRows partial_rows(const AttendArgs& a, size_t piece_head) {
  const uint32_t blocks = ((uint32_t)a.n + 31u) / 32u;
  return PartialRows{__builtin_amdgcn_make_buffer_rsrc(a.attn_o + piece_head * blocks * 2048, 0, 0x7fffffff, 0x00020000),
                     __builtin_amdgcn_make_buffer_rsrc(a.attn_ml + piece_head * (uint32_t)a.n * 4, 0, 0x7fffffff, 0x00020000)};
}
// This wave's partials have reached memory (its count of outstanding accesses is zero).
__device__ __forceinline__ void partials_written() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The workgroups of a cut unit meet at its counter (Workspace::unit_done), when their partials have reached memory, to share
// the merge.  Who is not last waits for the others, but not for long: after `looks` looks at the counter it leaves, and the
// others do its share.  One word says everything, so that everybody agrees on who is there: pieces that are done (bits 0..4, the
// number before gives each its place), who of the others has seen that all are (bits 8..12), places that were left before all were
// done (bits 16..31; none can be left after that).  Nobody depends on anybody's being resident: the last one to be done
// never waits.  Where nobody waits at all (`waiting` false, the same for the whole launch) the last one is alone with the merge,
// and the others need not say that they leave.
// What bounds it: round trips to memory - the partials' way there, an atomic, a look or two, one trip for a sharer's part of all
// pieces.  16 heads x 1374 rows in four long pieces and a short one: 1.7 us (median) from a partial's being written to the meeting's end, 2.0 us
// of merging, where the last workgroup by itself took 0.8 and 6.1.
constexpr uint32_t kMeetDone = 31u, kMeetAck = 1u << 8;
struct Meeting {
  int rank, sharers;  // this workgroup's number among those that share the merge (sharers = 0: it does not take part)
};
__device__ __forceinline__ Meeting meet(uint32_t* counter, int pieces, bool waiting, int looks) {
  uint32_t v = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u;
  const uint32_t place = (v & kMeetDone) - 1u, all = (uint32_t)pieces;
  if (!waiting) return Meeting{0, (v & kMeetDone) == all ? 1 : 0};
  for (int i = 0; i < looks && (v & kMeetDone) != all; ++i) {
    __builtin_amdgcn_s_sleep(8);
    v = __hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  while ((v & kMeetDone) != all)  // (fails, and goes on with the new value, only when somebody else has come or left)
    if (__hip_atomic_compare_exchange_strong(counter, &v, v | (0x10000u << place), __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      return Meeting{0, 0};
  const uint32_t left = v >> 16;
  return Meeting{(int)(place - (uint32_t)__popc(left & ((1u << place) - 1u))), pieces - (int)__popc(left)};
}

// "No vector-memory load is outstanding here" as an instruction (s_waitcnt vmcnt(0)).  A tile loop fetches the next
// tile under a condition and consumes it under the same condition further down; the compiler does not connect the
// two, assumes that fetched registers may still be in flight on the path that skips the consumer, and would then
// wait for ALL loads - the prefetch just issued included - in front of whatever reuses one of those registers in the
// next iteration or the next loop.  Stated at the end of an iteration, where it is true anyway, it costs nothing.
__device__ __forceinline__ void no_loads_in_flight() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// max of a value with the one held by the lane 32 apart (the other half of the same query's
// tokens): one v_permlane32_swap instead of a round trip through the LDS crossbar
__device__ __forceinline__ float xhalf_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// A callable that issues `N` MFMAs per call (the softmax block uses N to lay out its issue order).
template <int N, bool SUMS, typename F>
struct MfmaHook {
  static constexpr int kMfma = N;
  static constexpr bool kSums = SUMS;
  F f;
  __device__ __forceinline__ void operator()(int i) const { f(i); }
};
template <int N, bool SUMS, typename F>
__device__ __forceinline__ MfmaHook<N, SUMS, F> with_mfma(F f) { return MfmaHook<N, SUMS, F>{f}; }

// ---- partition of the (unit, tile) line over the workgroups -----------------------------------------
struct Partition {
  long long total;  // n_units * n_tiles
  int n_tiles, n_wgs;
  // 64-bit division is a long instruction sequence on this target; launches of realistic size fit 32 bits
  __host__ __device__ bool small() const { return total * (n_wgs + 1) < (1ll << 31); }
  __host__ __device__ long long begin(int w) const {
    return small() ? (long long)((unsigned)total * (unsigned)w / (unsigned)n_wgs) : total * w / n_wgs;
  }
  // workgroup whose piece holds item x
  __host__ __device__ int owner(long long x) const {
    return small() ? (int)((((unsigned)x + 1u) * (unsigned)n_wgs + (unsigned)total - 1u) / (unsigned)total) - 1
                   : (int)(((x + 1) * n_wgs + total - 1) / total) - 1;
  }
  __host__ __device__ int unit_of(long long x) const {
    return small() ? (int)((unsigned)x / (unsigned)n_tiles) : (int)(x / n_tiles);
  }
  __host__ __device__ int first_wg(int unit) const { return owner((long long)unit * n_tiles); }
  __host__ __device__ int last_wg(int unit) const { return owner((long long)(unit + 1) * n_tiles - 1); }
};

// ---- the kernel ----------------------------------------------------------------------------------
// ONE_LAYER: the launch works on a single layer (the per-layer calls).  The layer index is then a constant, so every
// pointer of the launch can be fetched from the kernel arguments right at the start, in one round trip, instead of
// after the workgroup has worked out which layer its piece belongs to.
// INSIDE: AttendArgs::merge_inside.  (A kernel of its own: as a branch it cost the other form 1.4 % of a frame-wise attention.)
template <int BITS, int G, int NW, int QB, bool ONE_LAYER, bool INSIDE>
__global__ __launch_bounds__(NW * 64) void attend_kernel(const AttendArgs a) {
  constexpr int NT = NW * 64, NH = NT / 2;
  constexpr int kRowsWG = 32 * QB * NW;  // query rows per workgroup
  {
    // The argument block is read field by field further down, each read a scalar load the next instructions wait
    // for, and at the start of a launch every one of them misses the scalar cache: several memory round trips in a
    // row before a workgroup can ask for its first tile.  One load from every 64-byte line the kernel will touch
    // (the fields behind the layer table, and the first layer's pointers), all issued here and waited for once,
    // brings those lines in together.
#if defined(__HIP_DEVICE_COMPILE__)  // (the builtin exists in the device pass only)
    const uint32_t* args = static_cast<const uint32_t*>(__builtin_amdgcn_kernarg_segment_ptr());
    constexpr unsigned kFirst = offsetof(AttendArgs, n_layers) / 4, kLast = (sizeof(AttendArgs) - 4) / 4;
    const uint32_t w0 = args[0], w1 = args[16], w2 = args[kFirst], w3 = args[kFirst + 16], w4 = args[kFirst + 32],
                   w5 = args[kLast];
    asm volatile("" ::"s"(w0), "s"(w1), "s"(w2), "s"(w3), "s"(w4), "s"(w5));
#endif
  }
  __shared__ __attribute__((aligned(16))) uint16_t lds_k[2][kLdsTile];
  __shared__ __attribute__((aligned(16))) uint16_t lds_v[2][kLdsTile];
  constexpr int kPrmBlock = BITS == 16 ? 1 : 2 * Stage<BITS, G, NH>::kPrm;  // one tile's scales and zero points of one role
  __shared__ __attribute__((aligned(16))) float lds_prm[2][2][kPrmBlock];    // [role][buffer]
  __shared__ int careful_pass[2];  // some wave asks for it (by the parity of the unit's number in this workgroup)
  __shared__ int meeting[2];       // what thread 0 learned at a unit's meeting

  const int H = a.H, n = a.n, Tc = a.Tc;
  const int nqb = (n + kRowsWG - 1) / kRowsWG;
  // the wave index as a scalar the compiler knows to be the same for all lanes: what depends on it - the staging
  // role and every pointer chosen by it - lives in scalar registers, and the role's branches are scalar branches
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int j = lane & 31, hh = lane >> 5;
  const int krow = tau(j);
  const float c2 = a.qscale;  // softmax scale * log2(e): p = 2^(c2 * (logit - max))
  // staging role of this wave: first half of the workgroup's waves K, second half V
  const bool is_v = wave >= NW / 2;
  const int u = (is_v ? wave - NW / 2 : wave) * 64 + lane;

  // tiles of a unit: cache blocks, then the frame's own tokens (each range padded to 64 on its own)
  const int n_ct = (Tc + kTile - 1) / kTile, n_ft = (n + kTile - 1) / kTile;
  const Partition part{(long long)a.n_layers * H * nqb * (n_ct + n_ft), n_ct + n_ft, (int)gridDim.x};
  // Logical workgroup.  Workgroups whose blockIdx agree modulo 8 run on the same XCD and share its L2;
  // when every unit is cut into the same number of key ranges, the query blocks of one (layer, head,
  // key range) - which read the same K/V tiles - are placed on one XCD.
  // (Every integer division by a launch parameter is some thirty instructions here, and a workgroup's first tile
  // waits behind all of them: where the quotients are already at hand they are kept - `fast` below - instead of
  // being derived again from the logical index.)
  int wg = blockIdx.x;
  bool fast = false;      // this workgroup's (unit, range, query block, head) are known without further divisions
  int f_unit = 0, f_range = 0, f_qb = 0, f_head = 0;
  if (a.xcd_ranges > 0) {
    const int xcd = wg & 7, slot = wg >> 3;
    int gq, gr, sr;  // (layer, head), key range, query block
    if (a.xcd_heads) {  // all workgroups of a head on one XCD
      const int per_head = a.xcd_ranges * nqb;
      const int sq = slot / per_head, rest = slot - sq * per_head;
      gq = sq * 8 + xcd;
      gr = rest / nqb;
      sr = rest - gr * nqb;
    } else {
      const int sq = slot / nqb;
      sr = slot - sq * nqb;
      const int g = sq * 8 + xcd;  // (layer, head, key range) triple
      gq = g / a.xcd_ranges;
      gr = g - gq * a.xcd_ranges;
    }
    wg = (gq * nqb + sr) * a.xcd_ranges + gr;
    if (a.equal_ranges == a.xcd_ranges) {  // unit = wg / ranges, range = wg % ranges
      fast = true;
      f_unit = gq * nqb + sr;
      f_range = gr;
      f_qb = sr;      // unit % nqb
      f_head = gq;    // unit / nqb: (layer, head); the head itself when the launch has one layer
    }
  }
  // this workgroup's piece [piece_first, piece_end) of the (unit, tile) line: an equal share of the line, or - when
  // every unit is cut into the same ranges - range wg % R of unit wg / R from the host's table of range starts
  // (read with constant indices: a dynamically indexed kernel argument would be copied to scratch memory)
  long long piece_first, piece_end;
  int my_range = 0;  // which of its unit's key ranges this workgroup holds (equal ranges only)
  if (a.equal_ranges <= 0) {
    piece_first = part.begin(wg);
    piece_end = part.begin(wg + 1);
  } else {
    const int un = fast ? f_unit : wg / a.equal_ranges;
    my_range = fast ? f_range : wg - un * a.equal_ranges;
    int b0 = 0, b1 = 0;
#pragma unroll
    for (int i = 0; i < kMaxPieces; ++i) {
      if (i == my_range) { b0 = a.range_begin[i]; b1 = a.range_begin[i + 1]; }
    }
    piece_first = (long long)un * part.n_tiles + b0;
    piece_end = (long long)un * part.n_tiles + b1;
    if (!fast) f_unit = un;
  }

  int parity = 0;
  for (long long pos = piece_first; pos < piece_end;) {
  // with equal ranges a piece lies inside one unit
  const int unit = a.equal_ranges > 0 ? f_unit : part.unit_of(pos);
  const int t_begin = (int)(pos - (long long)unit * part.n_tiles);
  const int t_end = (int)min((long long)part.n_tiles, t_begin + (piece_end - pos));
  pos += t_end - t_begin;
  int qb, h, lb;
  if (fast && ONE_LAYER) {
    qb = f_qb; h = f_head; lb = 0;
  } else {
    qb = unit % nqb;
    const int lh = unit / nqb;
    lb = ONE_LAYER ? 0 : lh / H;
    h = lh - lb * H;
  }
  const bool whole = t_begin == 0 && t_end == part.n_tiles;
  const int c_begin = min(t_begin, n_ct), c_end = min(t_end, n_ct);
  const int f_begin = max(t_begin, n_ct) - n_ct, f_end = max(t_end, n_ct) - n_ct;

  const AttendLayer& ly = a.layer[lb];
  const uint16_t* qh = ly.q + (size_t)h * a.q_sh;
  RolePtrs rp;
  rp.is_v = is_v;
  rp.codes = (is_v ? ly.vc : ly.kc) + (size_t)h * a.code_head;
  rp.ps = is_v ? ly.vs + (size_t)h * a.vparam_head : ly.ks + (size_t)h * a.kparam_head;
  rp.pz = is_v ? ly.vz + (size_t)h * a.vparam_head : ly.kz + (size_t)h * a.kparam_head;
  rp.lds = is_v ? lds_v[0] : lds_k[0];
  rp.prm = lds_prm[is_v][0];
  const uint16_t* xh = is_v ? ly.v + (size_t)h * a.v_sh : ly.k + (size_t)h * a.k_sh;
  const int64_t x_st = is_v ? a.v_st : a.k_st;

  // query fragments (B operand): lane holds channels 16*ks + 8*hh .. +8 of its query row, as given
  // (the softmax scale is applied to the fp32 logits, so no extra bf16 rounding enters)
  const int q_row0 = qb * kRowsWG + wave * 32 * QB;  // first row of this wave
  bf16x8 qf[QB][4];
#pragma unroll
  for (int cb = 0; cb < QB; ++cb) {
    const int q_row = q_row0 + 32 * cb + j;
    const uint16_t* qp = qh + (size_t)min(q_row, n - 1) * a.q_st;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
      qf[cb][ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(qp + 16 * ks + 8 * hh));
  }
  // query blocks of this wave that hold at least one real row (wave-uniform)
  const int n_cb = q_row0 >= n ? 0 : min(QB, (n - q_row0 + 31) / 32);

  f32x16 o0[QB], o1[QB];
  // softmax state per query block: mc = -(reference of the exponent, log2 domain) so that a probability is
  // 2^(c2 * logit + mc), the sum of this lane's row up to the tile at hand, and the sums of that tile (layout: see tile_sum)
  float mc[QB], l[QB];
  f32x4 lt[QB];
  // Rows with a logit that is NaN or +infinity (bit = lane; the careful pass finds them): their probabilities are kept finite
  // and their output becomes NaN at the end.
  unsigned long long nan_rows[QB];
  auto clear = [&]() XSV_INLINE {
#pragma unroll
    for (int cb = 0; cb < QB; ++cb) {
#pragma unroll
      for (int r = 0; r < 16; ++r) { o0[cb][r] = 0.f; o1[cb][r] = 0.f; }
      l[cb] = 0.f;
      nan_rows[cb] = 0;
      mc[cb] = -kNegBig;
    }
  };
  clear();
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // Row sums on the matrix pipe: MFMA 16x16x32 of a 0/1 matrix with the packed probabilities - the ROUNDED ones, which
  // the PV product sees.  Read as the B operand of that shape, lane group g = lane / 16 holds query 16 * (g & 1) + lane % 16;
  // row i of the 0/1 matrix takes the groups of i's parity, so result rows of even (odd) index - registers 0, 2 (1, 3) of
  // every lane - are the sums of query lane % 16 (16 + lane % 16) over both halves' tokens.
  const uint32_t ones = (((lane & 15) ^ (lane >> 4)) & 1) ? 0u : 0x3f803f80u;
  const u32x4 sum_rows = {ones, ones, ones, ones};
  // (A probability that is not finite makes the sum of the row 16 away NaN.  That is one reason to take a tile's sums by
  // themselves and to look at them before they are added to the rows': what was summed up before is not lost.)
  const uint32_t odd_rows = (lane & 16) ? ~0u : 0u;  // (a mask: chosen by a condition, the register would be indexed dynamically)
  auto tile_sum = [&](int cb) XSV_INLINE {
    return __uint_as_float((__float_as_uint(lt[cb][1]) & odd_rows) | (__float_as_uint(lt[cb][0]) & ~odd_rows));
  };
  auto sum_step = [&](int cb, const u32x4& p, bool fresh) XSV_INLINE {
    lt[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, sum_rows), __builtin_bit_cast(bf16x8, p),
                                                     fresh ? f32x4{0.f, 0.f, 0.f, 0.f} : lt[cb], 0, 0, 0);
  };
  // step i (0..3) of O^T += V^T P^T for one query block: token step i/2, channel half i%2; `fresh`: the tile's sums begin here
  auto pv_step = [&](int cb, const bf16x8 (&vf)[2][2], const u32x4 (&pb)[2], int i, bool fresh) XSV_INLINE {
    const int k2 = i >> 1;
    const bf16x8 p = __builtin_bit_cast(bf16x8, pb[k2]);
    if (!(i & 1)) sum_step(cb, pb[k2], fresh && i == 0);
    if (i & 1) o1[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[k2][1], p, o1[cb], 0, 0, 0);
    else o0[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[k2][0], p, o0[cb], 0, 0, 0);
  };
  // logits of tokens past the end of the cache / of the frame
  auto mask_tail = [&](f32x16& sv, int tok0, int valid) XSV_INLINE {
    // (the limit passes through an opaque move so that the 16 compares stay where they are)
    int lim = __builtin_amdgcn_readfirstlane(valid - tok0);
    asm volatile("" : "+s"(lim));
    lim -= 8 * hh;
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (16 * (r >> 3) + (r & 7) >= lim) sv[r] = -INFINITY;
  };
  auto load_k = [&](bf16x8 (&kf)[4], int buf, int half) XSV_INLINE {
    const uint16_t* lk = lds_k[buf] + krow * kLdsStride + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) kf[ks] = *reinterpret_cast<const bf16x8*>(lk + 32 * half * kLdsStride + 16 * ks);
  };
  auto load_v = [&](bf16x8 (&vf)[2][2], int buf, int half) XSV_INLINE {
    const uint16_t* lv = lds_v[buf] + j * kLdsStride + 8 * hh;
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      vf[k2][0] = *reinterpret_cast<const bf16x8*>(lv + 32 * half + 16 * k2);
      vf[k2][1] = *reinterpret_cast<const bf16x8*>(lv + 32 * kLdsStride + 32 * half + 16 * k2);
    }
  };
  // step i (0..3) of S^T = K Q^T for one query block (contraction over 16 channels per step)
  auto qk_step = [&](f32x16& sv, const bf16x8 (&kf)[4], int cb, int i) XSV_INLINE {
    sv = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i], qf[cb][i], i == 0 ? zero : sv, 0, 0, 0);
  };
  auto row_max = [&](const f32x16& sv) XSV_INLINE {
    float mx = fmaxf(fmaxf(sv[0], sv[1]), sv[2]);  // v_max3 chain
#pragma unroll
    for (int r = 3; r < 15; r += 2) mx = fmaxf(fmaxf(mx, sv[r]), sv[r + 1]);
    return xhalf_max(fmaxf(mx, sv[15]));  // both lane halves of a row agree on it
  };
  // Probabilities of one query block over the 32 tokens of a half-step: registers r = 8*k2 .. 8*k2+7 of the logits become
  // the packed B operand of token step k2.  `hook(i)`, i = 0..3, is called before each quarter: the caller issues MFMAs
  // there, so that the matrix pipe works underneath this arithmetic.  `clamp`: to 1 (an output modifier of the exponential).
  auto softmax_half = [&](f32x16& sv, u32x4 (&pb)[2], float mcr, auto clamp, auto&& hook) XSV_INLINE {
    auto prob = [&](float x) XSV_INLINE {
      const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(x, c2, mcr));
      if constexpr (clamp) return __builtin_amdgcn_fmed3f(p, 0.f, 1.f);
      else return p;
    };
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      hook(q4);
#pragma unroll
      for (int r = 4 * q4; r < 4 * q4 + 4; r += 2) {
        pb[r >> 3][(r >> 1) & 3] = pack_bf16(prob(sv[r]), prob(sv[r + 1]));
      }
    }
    // prescribed issue order of this block, per quarter: its MFMAs spread between its 10 vector instructions (4 fma,
    // 4 exp, 2 convert) - the MFMAs execute while the VALU works
    using Hook = std::remove_reference_t<decltype(hook)>;
    if constexpr (Hook::kMfma > 0) {
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        // masks: 0x008 MFMA, 0x002 VALU (without transcendentals), 0x400 transcendental
        const int m = Hook::kMfma + (Hook::kSums && q4 % 2 == 0 ? 1 : 0);
        if (m == 3) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
        } else if (m == 2) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
          __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
        } else {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
          __builtin_amdgcn_sched_group_barrier(0x400, 4, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
        }
      }
    }
    // keep this block's probabilities in this block (the compiler would otherwise sink the
    // exponentials down to their consumer, next to the MFMAs they are meant to overlap with)
    asm volatile("" : "+v"(pb[0]), "+v"(pb[1]));
  };

  // The references: row maxima over the first half-step of the range, which is in LDS buffer `buf`.
  auto first_reference = [&](int buf, int valid) XSV_INLINE {
    bf16x8 kf[4];
    load_k(kf, buf, 0);
#pragma unroll
    for (int cb = 0; cb < QB; ++cb) {
      f32x16 sv;
#pragma unroll
      for (int i = 0; i < 4; ++i) qk_step(sv, kf, cb, i);
      if (valid < 32) mask_tail(sv, 0, valid);
      // (a row of which every logit here is -inf gets a reference below all others: the first one that is not raises it)
      mc[cb] = -fminf(fmaxf(__builtin_fmaf(row_max(sv), c2, kHeadroom), kNegBig), kFar);
    }
  };

  // One whole tile of 64 tokens held in LDS buffer `buf`, the references standing: straight-line code.
  auto compute_tile = [&](int buf) XSV_INLINE {
    bf16x8 kf[4], vf[2][2];
    if constexpr (QB == 2) {
      // Software pipeline over the two half-steps and the two query blocks A, B of the wave: every
      // block of softmax arithmetic has independent MFMAs issued inside it —
      //   SM(A,h):  S(B,h) [and O(B,h-1)]      SM(B,h):  O(A,h) [and S(A,h+1)]
      // Blocks past the end of the frame are computed on clamped rows and never stored.
      f32x16 sA, sB;
      u32x4 pA[2], pB[2];
      load_k(kf, buf, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) qk_step(sA, kf, 0, i);
      load_v(vf, buf, 0);
      // ---- half 0 ----
      // (wave priority falls as a wave advances through a tile: of the two waves that share a SIMD the one that is
      // behind is served first, so they stay within a block of each other and each one's MFMAs run under the
      // other's softmax arithmetic, instead of the older wave finishing its tile first and the younger one
      // then working through its own alone; measured 2.7 % on the kernel)
      __builtin_amdgcn_s_setprio(3);
      softmax_half(sA, pA, mc[0], std::false_type{}, with_mfma<1, false>([&](int i) XSV_INLINE { qk_step(sB, kf, 1, i); }));
      load_k(kf, buf, 1);
      __builtin_amdgcn_s_setprio(2);
      softmax_half(sB, pB, mc[1], std::false_type{}, with_mfma<2, true>([&](int i) XSV_INLINE {
        pv_step(0, vf, pA, i, true);
        qk_step(sA, kf, 0, i);
      }));
      // ---- half 1 ----
      __builtin_amdgcn_s_setprio(1);
      softmax_half(sA, pA, mc[0], std::false_type{}, with_mfma<2, true>([&](int i) XSV_INLINE {
        pv_step(1, vf, pB, i, true);
        qk_step(sB, kf, 1, i);
      }));
      load_v(vf, buf, 1);
      __builtin_amdgcn_s_setprio(0);
      softmax_half(sB, pB, mc[1], std::false_type{}, with_mfma<1, true>([&](int i) XSV_INLINE { pv_step(0, vf, pA, i, false); }));
#pragma unroll
      for (int i = 0; i < 4; ++i) pv_step(1, vf, pB, i, false);
    } else {
      load_k(kf, buf, 0);
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        f32x16 sv;
#pragma unroll
        for (int i = 0; i < 4; ++i) qk_step(sv, kf, 0, i);
        load_v(vf, buf, half);
        if (half == 0) load_k(kf, buf, 1);
        u32x4 pw[2];
        softmax_half(sv, pw, mc[0], std::false_type{}, with_mfma<0, false>([](int) XSV_INLINE {}));
#pragma unroll
        for (int i = 0; i < 4; ++i) pv_step(0, vf, pw, i, half == 0);
      }
    }
  };

  // references of one block raised from -mc[cb] to `ref`: its accumulators and sums rescaled
  auto rescale = [&](int cb, float ref) XSV_INLINE {
    const float alpha = __builtin_amdgcn_exp2f(-mc[cb] - ref);
#pragma unroll
    for (int r = 0; r < 16; ++r) { o0[cb][r] *= alpha; o1[cb][r] *= alpha; }
    l[cb] *= alpha;
    mc[cb] = -ref;
  };
  // Lanes that hold a NaN among these logits.  (Floats of this file are compiled as if none was NaN, so they go through an
  // opaque step first.  Its wait covers the time an MFMA's results take: the compiler does not see a reader of theirs here.)
  auto nan_lanes = [&](f32x16& sv) XSV_INLINE {
    asm volatile("s_nop 15" : "+v"(sv));
    uint32_t top = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) top = max(top, __float_as_uint(sv[r]) & 0x7fffffffu);
    return __ballot(top > 0x7f800000u);
  };
  // A tile of which the first `valid` tokens are real, one block after the other, with references that follow the running
  // row maxima: a ragged last tile, and every tile of the careful pass.  There the rows of NaN logits are marked, the logits
  // taken out and probabilities clamped (to 1, for logits so large that the headroom is lost to rounding), so that whatever is
  // not finite ends in its own row.
  auto compute_tile_slowly = [&](int buf, int valid, auto careful) XSV_INLINE {
    for (int half = 0; half < 2 && 32 * half < valid; ++half) {
      bf16x8 kf[4], vf[2][2];
      load_k(kf, buf, half);
      load_v(vf, buf, half);
#pragma unroll
      for (int cb = 0; cb < QB; ++cb) {
        f32x16 sv;
#pragma unroll
        for (int i = 0; i < 4; ++i) qk_step(sv, kf, cb, i);
        mask_tail(sv, 32 * half, valid);
        if constexpr (careful) {
          const unsigned long long lanes = nan_lanes(sv), rows = lanes | (lanes >> 32) | (lanes << 32);
          nan_rows[cb] |= rows;
#pragma unroll
          for (int r = 0; r < 16; ++r) sv[r] = (rows >> lane) & 1 ? -INFINITY : sv[r];
        }
        const float top = __builtin_fmaf(row_max(sv), c2, kHeadroom);
        if constexpr (careful) nan_rows[cb] |= __ballot(top > kFar);
        rescale(cb, fminf(fmaxf(-mc[cb], top), kFar));
        u32x4 pw[2];
        softmax_half(sv, pw, mc[cb], careful, with_mfma<0, false>([](int) XSV_INLINE {}));
#pragma unroll
        for (int i = 0; i < 4; ++i) pv_step(cb, vf, pw, i, true);
        l[cb] += tile_sum(cb);
      }
    }
  };
  // Largest of the tile's row sums that this lane holds (numbers that are not negative, and NaN: by their bits, NaN is largest).
  auto largest_sum = [&]() XSV_INLINE {
    uint32_t top = 0;
#pragma unroll
    for (int cb = 0; cb < QB; ++cb) top = max(top, max(__float_as_uint(lt[cb][0]), __float_as_uint(lt[cb][1])));
    return top;
  };
  constexpr uint32_t kInfBits = 0x7f800000u;
  // After a full tile with a row sum above kSumLimit: every row whose sum has grown above 1 gets a reference that puts it below
  // 2^-8 again (all of them, so that rows which grow alike are not moved one tile after the other); that is a factor for its
  // sum and accumulators.  Where probabilities come near an overflow, the row's accumulators may be lost, and so is the tile's
  // sum of the row 16 away.  What such a row had before weighs less than 2^-58 beside this tile (its sum was below 2^24 a
  // tile): it begins anew with it.  NaN, infinite logits and accumulators that are not finite even so - infinite values, or
  // products of values beyond 2^27 - ask for the careful pass.
  bool ask = false;
  auto recenter = [&](int buf) XSV_INLINE {
#pragma unroll
    for (int cb = 0; cb < QB; ++cb) {
      if (__any(__float_as_uint(tile_sum(cb)) >= __float_as_uint(0x1p100f))) {
        f32x16 s0, s1;
        {
          bf16x8 kf[4];
          load_k(kf, buf, 0);
#pragma unroll
          for (int i = 0; i < 4; ++i) qk_step(s0, kf, cb, i);
          load_k(kf, buf, 1);
#pragma unroll
          for (int i = 0; i < 4; ++i) qk_step(s1, kf, cb, i);
        }
        const float top = fmaxf(row_max(s0), row_max(s1)) * c2;  // log2 domain
        if ((nan_lanes(s0) | nan_lanes(s1) | __ballot(top > kFar)) != 0) {
          ask = true;
          return;
        }
        const bool far = top + mc[cb] > 90.0f;  // (64 probabilities below that stay below the test above)
        mc[cb] = far ? -fminf(top + kHeadroom, kFar) : mc[cb];
        l[cb] = far ? 0.f : l[cb];
#pragma unroll
        for (int r = 0; r < 16; ++r) { o0[cb][r] = far ? 0.f : o0[cb][r]; o1[cb][r] = far ? 0.f : o1[cb][r]; }
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          bf16x8 vf[2][2];
          load_v(vf, buf, half);
          u32x4 pw[2];
          softmax_half(half == 0 ? s0 : s1, pw, mc[cb], std::false_type{}, with_mfma<0, false>([](int) XSV_INLINE {}));
#pragma unroll
          for (int k2 = 0; k2 < 2; ++k2) {
            sum_step(cb, pw[k2], half == 0 && k2 == 0);  // every row's (of rows that stay, as before)
            u32x4 w = pw[k2];
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = far ? w[i] : 0u;
            o0[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[k2][0], __builtin_bit_cast(bf16x8, w), o0[cb], 0, 0, 0);
            o1[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[k2][1], __builtin_bit_cast(bf16x8, w), o1[cb], 0, 0, 0);
          }
        }
      }
      asm volatile("s_nop 15" : "+v"(o0[cb]), "+v"(o1[cb]), "+v"(lt[cb]));  // (see nan_lanes)
      uint32_t top = 0;
#pragma unroll
      for (int r = 0; r < 16; ++r) top = max(top, max(__float_as_uint(o0[cb][r]) & 0x7fffffffu, __float_as_uint(o1[cb][r]) & 0x7fffffffu));
      ask = ask || __any(top >= kInfBits);
      // (a factor of 2^-96 at most, so that it is a normal number; the next tile's end takes the rest)
      l[cb] += tile_sum(cb);
      lt[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
      const int up = l[cb] > 1.0f ? min(__builtin_amdgcn_frexp_expf(l[cb]) + (int)kHeadroom, 96) : 0;
      rescale(cb, (float)up - mc[cb]);
    }
  };

  // A full tile's sums looked at and added to the rows'.  A wave of one query block does that behind the conversion of the next
  // tile, so that it need not wait for them (2-bit stack of 24 layers 2479 -> 2445 us); with two blocks that costs registers
  // and gains nothing (one 4-bit layer alone 39.6 -> 40.7 us).
  constexpr bool kSettleLate = QB == 1;
  auto settle = [&](int buf) XSV_INLINE {
    if (__builtin_expect(__any(largest_sum() > __float_as_uint(kSumLimit)) && !ask, 0)) recenter(buf);
#pragma unroll
    for (int cb = 0; cb < QB; ++cb) l[cb] += tile_sum(cb);
  };

  // This range's tiles: first its tiles of the packed cache, then its tiles of the frame.  In either phase a tile is
  // fetched into registers while the one before it is computed, then converted into the free one of the two LDS buffers:
  // one barrier per tile.  A ragged last tile (cache or frame) is computed outside of the loop over the full ones, which
  // is straight-line code.  `first(buf, valid)`: before the first tile; `full(buf)`, `ragged(buf, valid)`: the tiles;
  // `late(buf)`: after a full tile, behind the conversion of the next one.
  auto walk = [&](auto&& first, auto&& full, auto&& late, auto&& ragged) XSV_INLINE {
    int cur = 0;
    if (c_begin < c_end) {
      constexpr bool kQuant = BITS != 16;
      constexpr int kPrm = Stage<BITS, G, NH>::kPrm;
      CacheRegs<BITS, G, NH> st;
      PrmStage<BITS, G, NH> pst;
      fetch_cache_tile<BITS, G, NH>(st, rp, c_begin, u);
      if (kQuant && c_begin + 1 < c_end) fetch_params<BITS, G, NH>(pst, rp, c_begin + 1, u);
      store_cache_tile<BITS, G, NH>(st, rp.lds, rp.ps + (size_t)c_begin * kPrm, rp.pz + (size_t)c_begin * kPrm, is_v, u);
      if (kQuant && c_begin + 1 < c_end) store_params<BITS, G, NH>(pst, rp.prm + kPrmBlock, u);
      no_loads_in_flight();
      __syncthreads();
      first(0, Tc - c_begin * kTile);
      const int full_end = min(c_end, Tc / kTile);
      for (int t = c_begin; t < full_end; ++t) {
        // tile t is in lds[cur], the parameters of tile t + 1 in prm[cur^1]; everybody is done reading lds[cur^1] and prm[cur]
        __syncthreads();
        if (t + 1 < c_end) fetch_cache_tile<BITS, G, NH>(st, rp, t + 1, u);
        if (kQuant && t + 2 < c_end) fetch_params<BITS, G, NH>(pst, rp, t + 2, u);
        full(cur);
        if (t + 1 < c_end) {
          const float* prm = rp.prm + (cur ^ 1) * kPrmBlock;
          store_cache_tile<BITS, G, NH>(st, rp.lds + (cur ^ 1) * kLdsTile, prm, prm + kPrm, is_v, u);
        }
        late(cur);
        if (kQuant && t + 2 < c_end) store_params<BITS, G, NH>(pst, rp.prm + cur * kPrmBlock, u);
        no_loads_in_flight();
        cur ^= 1;
      }
      if (full_end < c_end) {
        __syncthreads();
        ragged(cur, Tc - full_end * kTile);
        cur ^= 1;
      }
    }
    if (f_begin < f_end) {
      FrameRegs<NH> st;
      const FrameRows fr = frame_rows(xh, x_st, n, is_v, u);
      fetch_frame_tile<NH>(st, fr, is_v, f_begin);
      store_frame_tile<NH>(st, rp.lds + cur * kLdsTile, is_v, u);  // lds[cur] was last read two barriers ago
      no_loads_in_flight();
      if (c_begin >= c_end) {
        __syncthreads();
        first(cur, n - f_begin * kTile);
      }
      const int full_end = min(f_end, n / kTile);
      for (int t = f_begin; t < full_end; ++t) {
        __syncthreads();
        if (t + 1 < f_end) fetch_frame_tile<NH>(st, fr, is_v, t + 1);
        full(cur);
        if (t + 1 < f_end) store_frame_tile<NH>(st, rp.lds + (cur ^ 1) * kLdsTile, is_v, u);
        late(cur);
        no_loads_in_flight();
        cur ^= 1;
      }
      if (full_end < f_end) {
        __syncthreads();
        ragged(cur, n - full_end * kTile);
      }
    }
  };
  auto write_rows = [&]() XSV_INLINE {
    // accumulator register r of o0 (o1) is channel 8*(r/4) + 4*hh + r%4 (+32) of the lane's query row
#pragma unroll
    for (int cb = 0; cb < QB; ++cb) {
      const int q_row = q_row0 + 32 * cb + j;
      const float lsum = __uint_as_float(__float_as_uint(l[cb]) | ((nan_rows[cb] >> lane) & 1 ? 0x7fc00000u : 0u));
      if (q_row >= n) continue;  // (both lanes of a row leave together, so the lane exchange below stays paired)
      if (whole) {
        const float inv = 1.0f / lsum;
        uint16_t* op = ly.out + ((size_t)h * n + q_row) * kD;
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int c = 8 * q4 + 4 * hh;
          *reinterpret_cast<uint2*>(op + c) = make_uint2(pack_bf16(o0[cb][4 * q4] * inv, o0[cb][4 * q4 + 1] * inv),
                                                         pack_bf16(o0[cb][4 * q4 + 2] * inv, o0[cb][4 * q4 + 3] * inv));
          *reinterpret_cast<uint2*>(op + 32 + c) = make_uint2(pack_bf16(o1[cb][4 * q4] * inv, o1[cb][4 * q4 + 1] * inv),
                                                              pack_bf16(o1[cb][4 * q4 + 2] * inv, o1[cb][4 * q4 + 3] * inv));
        }
      } else {
        // Partial of a cut unit, as fp16 mantissas under one power-of-two scale per query row (the
        // row's largest magnitude maps into [0.5, 1): 11 bits below the row maximum, half the bytes of
        // fp32).  Lane (j, hh) owns 32 channels of row j, in register order o0[0..15], o1[0..15], as
        // four 16-byte pieces i; a block of 32 rows is stored [i][hh][j], so that every store
        // instruction of the wave covers 1 KB of consecutive memory.
        const int piece = a.equal_ranges > 0 ? my_range : wg - part.first_wg(unit);
        const int nblk = (n + 31) / 32;
        const size_t row = (((size_t)piece * a.n_layers + lb) * H + h) * n + q_row;
        const size_t blk = (((size_t)piece * a.n_layers + lb) * H + h) * nblk + (q_row >> 5);
        float amax = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) amax = fmaxf(amax, fmaxf(fabsf(o0[cb][r]), fabsf(o1[cb][r])));
        amax = xhalf_max(amax);
        const int e = __builtin_amdgcn_frexp_expf(amax);  // amax = f * 2^e, f in [0.5, 1)  (0 for amax == 0)
        uint32_t hw[16];
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          hw[r >> 1] = pack_f16(__builtin_amdgcn_ldexpf(o0[cb][r], -e), __builtin_amdgcn_ldexpf(o0[cb][r + 1], -e));
          hw[8 + (r >> 1)] = pack_f16(__builtin_amdgcn_ldexpf(o1[cb][r], -e), __builtin_amdgcn_ldexpf(o1[cb][r + 1], -e));
        }
        if constexpr (INSIDE) {
          const PartialRows to = partial_rows(a, ((size_t)piece * a.n_layers + lb) * H + h);
          const uint32_t at = (uint32_t)(q_row >> 5) * 4096u + (uint32_t)(hh * 32 + j) * 16u;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            __builtin_amdgcn_raw_buffer_store_b128(u32x4{hw[4 * i], hw[4 * i + 1], hw[4 * i + 2], hw[4 * i + 3]}, to.o, at + i * 1024u, 0, kAgentScope);
          if (hh == 0) {
            const u32x4 ml = {__float_as_uint(-mc[cb]), __float_as_uint(lsum), __float_as_uint(__builtin_amdgcn_ldexpf(1.0f, e)), 0u};
            __builtin_amdgcn_raw_buffer_store_b128(ml, to.ml, (uint32_t)q_row * 16u, 0, kAgentScope);
          }
        } else {
          uint4* op = reinterpret_cast<uint4*>(a.attn_o) + blk * 256 + hh * 32 + j;
#pragma unroll
          for (int i = 0; i < 4; ++i) op[i * 64] = make_uint4(hw[4 * i], hw[4 * i + 1], hw[4 * i + 2], hw[4 * i + 3]);
          if (hh == 0)
            *reinterpret_cast<float4*>(a.attn_ml + row * 4) = make_float4(-mc[cb], lsum, __builtin_amdgcn_ldexpf(1.0f, e), 0.f);
        }
      }
    }
  };

  // Merge of a unit's S <= MOST pieces in the order of the pieces, whoever does it; the arithmetic is combine_kernel's.
  // The unit's rows are dealt to `sharers` workgroups, this one is number `rank`: an item is a block of 32 rows and one of PARTS
  // parts of the channels, a wave takes one after the other, and a lane the values it would have held of an uncut row, of all pieces
  // at once.
  auto merge = [&](auto parts, auto most, int S, int rank, int sharers) XSV_INLINE {
    constexpr int PARTS = decltype(parts)::value, MOST = decltype(most)::value;
    constexpr int kQuads = 4 / PARTS;  // 16-byte runs of a lane's 32 values
    __builtin_amdgcn_s_setprio(3);
    const int row_first = qb * kRowsWG, items = PARTS * ((min(n - row_first, kRowsWG) + 31) / 32);
    const int end = items * (rank + 1) / sharers;
    const PartialRows from = partial_rows(a, (size_t)lb * H + h);
    const uint32_t pieces_heads = (uint32_t)(a.n_layers * H);
    const uint32_t o_piece = pieces_heads * (((uint32_t)n + 31u) / 32u) * 4096u, ml_piece = pieces_heads * (uint32_t)n * 16u;  // bytes
#pragma unroll 1
    for (int item = items * rank / sharers + wave; item < end; item += NW) {
      const int row0 = row_first + 32 * (item / PARTS), part = item % PARTS;
      const uint32_t at = (uint32_t)(row0 >> 5) * 4096u + (uint32_t)(part * kQuads) * 1024u + (uint32_t)(hh * 32 + j) * 16u;
      const uint32_t at_ml = (uint32_t)min(row0 + j, n - 1) * 16u;
      u32x4 ml[MOST], o[MOST][kQuads];
#pragma unroll
      for (int s = 0; s < MOST; ++s)
        if (s < S) {
          ml[s] = __builtin_amdgcn_raw_buffer_load_b128(from.ml, at_ml, s * ml_piece, kAgentScope);
#pragma unroll
          for (int q = 0; q < kQuads; ++q) o[s][q] = __builtin_amdgcn_raw_buffer_load_b128(from.o, at + q * 1024u, s * o_piece, kAgentScope);
        }
      float M = kNegBig, L = 0.f, acc[8 * kQuads];
#pragma unroll
      for (int r = 0; r < 8 * kQuads; ++r) acc[r] = 0.f;
#pragma unroll
      for (int s = 0; s < MOST; ++s)
        if (s < S) M = fmaxf(M, __uint_as_float(ml[s][0]));
#pragma unroll
      for (int s = 0; s < MOST; ++s) {
        if (s < S) {
          const float wgt = __builtin_amdgcn_exp2f(__uint_as_float(ml[s][0]) - M);
          L += wgt * __uint_as_float(ml[s][1]);
          const float ws = wgt * __uint_as_float(ml[s][2]);
#pragma unroll
          for (int r = 0; r < 8 * kQuads; r += 2) {
            const f16x2 v = __builtin_bit_cast(f16x2, (uint32_t)o[s][r >> 3][(r >> 1) & 3]);
            acc[r] += ws * (float)v[0];
            acc[r + 1] += ws * (float)v[1];
          }
        }
      }
      const int q_row = row0 + j;
      const float inv = 1.0f / L;
      if (q_row < n) {
        uint16_t* op = ly.out + ((size_t)h * n + q_row) * kD + 16 * kQuads * part + 4 * hh;
#pragma unroll
        for (int r = 0; r < 8 * kQuads; r += 4)  // (channels as in write_rows)
          *reinterpret_cast<uint2*>(op + 2 * r) = make_uint2(pack_bf16(acc[r] * inv, acc[r + 1] * inv), pack_bf16(acc[r + 2] * inv, acc[r + 3] * inv));
      }
    }
    __builtin_amdgcn_s_setprio(0);
  };

  if (tid == 0) careful_pass[parity] = 0;  // (barriers of the walk lie between this and anybody's setting it)
  walk([&](int buf, int valid) XSV_INLINE { if (n_cb > 0) first_reference(buf, valid); },
       [&](int buf) XSV_INLINE {
         if (n_cb == 0) return;
         compute_tile(buf);
         if constexpr (!kSettleLate) settle(buf);
       },
       [&](int buf) XSV_INLINE {
         if constexpr (kSettleLate) { if (n_cb > 0) settle(buf); }
       },
       [&](int buf, int valid) XSV_INLINE { if (n_cb > 0) compute_tile_slowly(buf, valid, std::false_type{}); });
  // A row sum that is not finite (row_max and the clamp of the ragged tile pass over a NaN, its sum shows it), and what recenter
  // could not settle: the tiles are walked once more, one at a time and every row on its own, and the rows are written again.
  // A wave cannot do that alone; the rows are written first so that this barrier is the last thing a workgroup does (it also
  // says that everybody has read the unit's last tile).
  bool lost = ask;
#pragma unroll
  for (int cb = 0; cb < QB; ++cb) {
    lost = lost || __any(__float_as_uint(l[cb]) >= kInfBits);
    // An accumulator can overflow without any sum being large: values near 2^128, probabilities that add up to 1/2 or more.
    // (One sum over all of them is not finite if one of them is not; a false alarm costs time only.)
    if (__any(l[cb] >= 0.5f)) {
      f32x4 all = {0.f, 0.f, 0.f, 0.f};  // (four chains: this stands at the end of every launch)
#pragma unroll
      for (int r = 0; r < 16; ++r) all[r & 3] += o0[cb][r] + o1[cb][r];
      uint32_t bits = __float_as_uint((all[0] + all[1]) + (all[2] + all[3]));
      asm volatile("" : "+v"(bits));  // (see nan_lanes; an integer here, or the test becomes one for infinity alone)
      lost = lost || __any((bits & kInfBits) == kInfBits);
    }
  }
  if (n_cb > 0 && lost && lane == 0) careful_pass[parity] = 1;
  write_rows();
  const bool finish = INSIDE && !whole;
  if (finish) partials_written();
  __syncthreads();
  if (__builtin_expect(__builtin_amdgcn_readfirstlane(careful_pass[parity]) != 0, 0)) {
    clear();
    for (int t = t_begin; t < t_end; ++t) {
      if (t < n_ct) {
        constexpr int kPrm = Stage<BITS, G, NH>::kPrm;
        CacheRegs<BITS, G, NH> st;
        fetch_cache_tile<BITS, G, NH>(st, rp, t, u);
        store_cache_tile<BITS, G, NH>(st, rp.lds, rp.ps + (size_t)t * kPrm, rp.pz + (size_t)t * kPrm, is_v, u);
      } else {
        FrameRegs<NH> st;
        fetch_frame_tile<NH>(st, frame_rows(xh, x_st, n, is_v, u), is_v, t - n_ct);
        store_frame_tile<NH>(st, rp.lds, is_v, u);
      }
      __syncthreads();
      if (n_cb > 0) compute_tile_slowly(0, min(kTile, t < n_ct ? Tc - t * kTile : n - (t - n_ct) * kTile), std::true_type{});
      __syncthreads();
    }
    write_rows();
    if (finish) {
      partials_written();
      __syncthreads();
    }
  }
  if (finish) {
    const int w0 = a.equal_ranges > 0 ? 0 : part.first_wg(unit);
    const int pieces = a.equal_ranges > 0 ? a.equal_ranges : part.last_wg(unit) - w0 + 1;
    // (who still has a unit to work on, and a range that was made short so that its compute unit is free early, does not wait)
    const bool waits = pos >= piece_end && !(a.short_last && my_range == pieces - 1);
    uint32_t* const unit_done = a.unit_done + (size_t)unit * kMeetStride;
    uint32_t acks = 0;
    if (tid == 0) {
      const Meeting m = meet(unit_done, pieces, a.merge_waits, waits ? a.merge_looks : 0);
      meeting[0] = m.rank;
      meeting[1] = m.sharers;
      // (alone, it need not say that it has looked)
      if (m.sharers > 1) acks = __hip_atomic_fetch_add(unit_done, kMeetAck, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    const int rank = __builtin_amdgcn_readfirstlane(meeting[0]), sharers = __builtin_amdgcn_readfirstlane(meeting[1]);
    if (sharers > 0) {
      // (parts so small that most waves of a sharer have an item, and no smaller; several layers never have more than kMergeInside
      // pieces here)
      using std::integral_constant;
      if (pieces <= (sharers == 1 ? kMergeInside : 3)) {
        merge(integral_constant<int, 1>{}, integral_constant<int, kMergeInside>{}, pieces, rank, sharers);
      } else if constexpr (ONE_LAYER) {
        if (pieces <= 8) merge(integral_constant<int, 2>{}, integral_constant<int, 8>{}, pieces, rank, sharers);
        else merge(integral_constant<int, 4>{}, integral_constant<int, kMaxPieces>{}, pieces, rank, sharers);
      } else {
        merge(integral_constant<int, 2>{}, integral_constant<int, kMergeInside>{}, pieces, rank, sharers);
      }
      // everybody who will look at the counter has looked: as the next launch wants it
      if (tid == 0 && (acks / kMeetAck) % 32u == (uint32_t)sharers - 1u) __hip_atomic_store(unit_done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  parity ^= 1;
  }  // units of this workgroup's piece

}

// Merge of the pieces of every unit that was cut:  out = sum_p 2^(m_p - M) O_p / sum_p 2^(m_p - M) l_p.
// (A launch of its own for cuts that were asked for and line partitions with nothing beside them, for units in two pieces, and for
// shapes and numbers of pieces that have no kernel that merges inside; see AttendArgs::merge_inside.)
// Grid: y = chunk of 32 query rows of a unit; x = the unit when all units are cut alike, else a boundary
// between workgroups w-1 | w of the attention grid (w = blockIdx.x + 1), standing for the unit it falls
// into: a unit with several boundaries is handled at its first one, and a boundary that coincides with
// a unit's edge has nothing to merge.
// Thread = (row, lane half hh, quarter of the lane's 32 values): 8 fp16 values of every piece.
__global__ __launch_bounds__(256) void combine_kernel(const AttendArgs a) {
  // the merge shares its compute units with the chain's kernels of the same layer, which nothing waits for: its
  // waves are served first
  __builtin_amdgcn_s_setprio(3);
  const int H = a.H, n = a.n;
  const int nqb = (n + a.rows_wg - 1) / a.rows_wg;
  const int n_tiles = (a.Tc + kTile - 1) / kTile + (n + kTile - 1) / kTile;
  const Partition part{(long long)a.n_layers * H * nqb * n_tiles, n_tiles, a.n_wgs};
  int unit, S;
  if (a.equal_ranges > 0) {  // every unit is cut into the same number of ranges: x = unit
    unit = blockIdx.x;
    if (a.xcd_heads) {  // the chunks of a head on the XCD that its partials were written on
      const int slot = unit >> 3, sq = slot / nqb;
      unit = (sq * 8 + (unit & 7)) * nqb + slot - sq * nqb;
    }
    S = a.equal_ranges;
  } else {
    const int w = blockIdx.x + 1;
    const long long pos = part.begin(w);
    unit = part.unit_of(pos);
    if (pos == (long long)unit * n_tiles) return;
    const int w0 = part.first_wg(unit);
    if (w0 + 1 != w) return;
    S = part.last_wg(unit) - w0 + 1;
  }
  const int qb = unit % nqb, h = (unit / nqb) % H, lb = unit / (nqb * H);
  const int tid = threadIdx.x;
  const int jrow = tid & 31, hh = (tid >> 5) & 1, qd = tid >> 6;  // consecutive threads read consecutive 16-byte pieces
  const int q_row = qb * a.rows_wg + 32 * blockIdx.y + jrow;
  if (q_row >= n) return;
  const int nblk = (n + 31) / 32;
  const size_t rows = (size_t)a.n_layers * H * n, blks = (size_t)a.n_layers * H * nblk;
  const size_t row = ((size_t)lb * H + h) * n + q_row;
  const size_t blk = ((size_t)lb * H + h) * nblk + (q_row >> 5);
  float ms[kMaxPieces], ls[kMaxPieces], sc[kMaxPieces];
  float M = kNegBig;
#pragma unroll 4
  for (int s = 0; s < S; ++s) {
    const float4 ml = *reinterpret_cast<const float4*>(a.attn_ml + (s * rows + row) * 4);
    ms[s] = ml.x;
    ls[s] = ml.y;
    sc[s] = ml.z;
    M = fmaxf(M, ml.x);
  }
  float L = 0.f, acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int s = 0; s < S; ++s) {
    const float wgt = __builtin_amdgcn_exp2f(ms[s] - M);
    const uint4 o = reinterpret_cast<const uint4*>(a.attn_o)[(s * blks + blk) * 256 + qd * 64 + hh * 32 + jrow];
    L += wgt * ls[s];
    const float ws = wgt * sc[s];
    const uint32_t ow[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f16x2 v = __builtin_bit_cast(f16x2, ow[i]);
      acc[2 * i] += ws * (float)v[0];
      acc[2 * i + 1] += ws * (float)v[1];
    }
  }
  const float inv = 1.0f / L;
  // values 8*qd + t of the lane: accumulator registers r = 8*(qd%2) + t of o0 (qd < 2) or o1, i.e.
  // channels 32*(qd/2) + 16*(qd%2) + {0, 8} + 4*hh + 0..3
  uint16_t* op = a.layer[lb].out + ((size_t)h * n + q_row) * kD + 32 * (qd >> 1) + 16 * (qd & 1) + 4 * hh;
  *reinterpret_cast<uint2*>(op) = make_uint2(pack_bf16(acc[0] * inv, acc[1] * inv), pack_bf16(acc[2] * inv, acc[3] * inv));
  *reinterpret_cast<uint2*>(op + 8) = make_uint2(pack_bf16(acc[4] * inv, acc[5] * inv), pack_bf16(acc[6] * inv, acc[7] * inv));
}

template <int BITS, int G, int NW, int QB>
static hipError_t launch_attend_t(const AttendArgs& a, hipStream_t stream, hipEvent_t between) {
  // A wave with one block of query rows leaves registers for front_kernel's (62, where it has 172 to 191 itself), and a compute unit
  // that works on both ends last: the launch keeps the LDS that front_kernel would need.  us per step with and without front_kernel
  // on its compute units, 4 bits, 8 x 32: one layer of 16 x 1041 over 4096 tokens 60.4 and 55.1, 10 x 1188 / 4956 57.3 and 52.7, six
  // layers of 16 x 600 / 3000 joined by every step 280 and 248, two such streams at a time 382 and 335.
  // Not with a short range, whose grid leaves so few compute units at first that the chain needs these too (deferred joins, 8 x 600 over
  // 16000 tokens 92 and 102, 16 x 200 / 24000 137 and 158), and not for 16 bits: front_kernel has 115 registers there and finds no
  // place anyway, move_kernel has 9 KB of LDS and should find more than one (10 x 1200 / 8000 56 and 60).
  // (Launches of several layers have the chain's parts beside them one by one, which share as they always did.)
  constexpr int kStatic = 4 * kLdsTile * (int)sizeof(uint16_t) + 8 * Stage<BITS, G, NW * 32>::kPrm * (int)sizeof(float);
  constexpr int kKeep = QB == 1 && BITS != 16 ? (kLdsOfComputeUnit - kLdsBesideAttention) / (NW == 8 ? 1 : 2) - kStatic : 0;
  const int keep = a.n_layers == 1 && !a.short_last ? kKeep : 0;
  auto launch = [&](auto one_layer, auto inside) {
    hipLaunchKernelGGL((attend_kernel<BITS, G, NW, QB, decltype(one_layer)::value, decltype(inside)::value>), dim3(a.n_wgs), dim3(NW * 64), keep, stream, a);
  };
  using std::true_type;
  using std::false_type;
  if (a.merge_inside) {  // (attend_merges_inside)
    if (a.n_layers == 1) {
      if constexpr (NW == 8 || QB == 2) launch(true_type{}, true_type{});
    } else {
      if constexpr (NW == 8) launch(false_type{}, true_type{});
    }
  }
  if (!a.merge_inside) a.n_layers == 1 ? launch(true_type{}, false_type{}) : launch(false_type{}, false_type{});
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (between && (e = hipEventRecord(between, stream)) != hipSuccess) return e;
  if (a.cut && !a.merge_inside) {
    const int n_units = a.n_layers * a.H * ((a.n + a.rows_wg - 1) / a.rows_wg);
    hipLaunchKernelGGL(combine_kernel, dim3(a.equal_ranges > 0 ? n_units : a.n_wgs - 1, (a.rows_wg + 31) / 32), dim3(256), 0,
                       stream, a);
    e = hipGetLastError();
  }
  return e;
}

template <int BITS, int G>
static hipError_t launch_attend_v(const AttendArgs& a, hipStream_t stream, hipEvent_t between) {
  switch (a.variant) {
    case 1: return launch_attend_t<BITS, G, 4, 1>(a, stream, between);
    case 2: return launch_attend_t<BITS, G, 8, 1>(a, stream, between);
    case 3: return launch_attend_t<BITS, G, 8, 2>(a, stream, between);
    default: return launch_attend_t<BITS, G, 4, 2>(a, stream, between);
  }
}

// Host-side queries of the partition the kernel uses when the units are not all cut alike (for tests).
void partition_query(long long n_units, int n_tiles, int n_wgs, int wg, long long* begin, long long* end) {
  const Partition part{n_units * n_tiles, n_tiles, n_wgs};
  *begin = part.begin(wg);
  *end = part.begin(wg + 1);
}
void partition_unit_query(long long n_units, int n_tiles, int n_wgs, int unit, int* first_wg, int* last_wg) {
  const Partition part{n_units * n_tiles, n_tiles, n_wgs};
  *first_wg = part.first_wg(unit);
  *last_wg = part.last_wg(unit);
}

int attend_rows_per_workgroup(int variant) {
  return variant == 1 ? 128 : (variant == 3 ? 512 : 256);
}

// (4 waves x 64 rows with groups of 32 take more than 256 registers: one wave to a SIMD)
int attend_places_per_cu(int variant, int G) { return variant >= 2 || (variant == 0 && G == 32) ? 1 : 2; }

bool attend_merges_inside(int variant, int n_layers) { return variant >= 2 || (variant == 0 && n_layers == 1); }

AttendPlan plan_attend(int variant, int n_layers, int H, int n, int Tc, int want_wgs, size_t part_rows) {
  const int rows_wg = attend_rows_per_workgroup(variant);
  const int nqb = (n + rows_wg - 1) / rows_wg;
  const int n_units = n_layers * H * nqb;
  const int n_tiles = (Tc + kTile - 1) / kTile + (n + kTile - 1) / kTile;
  const long long total = (long long)n_units * n_tiles;
  // a piece never shorter than 4 tiles (unless a whole unit is), never more workgroups than items
  long long w = std::max<long long>(1, std::min<long long>(want_wgs, std::max<long long>(n_units, total / 4)));
  // the partial workspace holds `fit` pieces of every row, the merge at most kMaxPieces
  const int fit = (int)std::min<size_t>(kMaxPieces, part_rows / ((size_t)n_layers * H * ((n + 31) / 32 * 32)));
  AttendPlan p{};
  for (;; --w) {
    const Partition part{total, n_tiles, (int)w};
    int worst = 1;
    for (int unit = 0; unit < n_units; ++unit) worst = std::max(worst, part.last_wg(unit) - part.first_wg(unit) + 1);
    if (worst <= fit || w == 1) {
      p.n_wgs = (int)w;
      p.rows_wg = rows_wg;
      p.max_pieces = worst;
      return p;
    }
    if (w > n_units) w = std::max<long long>(n_units + 1, w - w / 8);  // then --w
  }
}

hipError_t launch_attend(const AttendArgs& a, hipStream_t stream, hipEvent_t between) {
  const int bits = a.bits, G = a.G;
  if (bits == 16) return launch_attend_v<16, 64>(a, stream, between);
  if (bits == 4 && G == 64) return launch_attend_v<4, 64>(a, stream, between);
  if (bits == 4 && G == 32) return launch_attend_v<4, 32>(a, stream, between);
  if (bits == 2 && G == 64) return launch_attend_v<2, 64>(a, stream, between);
  if (bits == 2 && G == 32) return launch_attend_v<2, 32>(a, stream, between);
  return hipErrorInvalidValue;
}

}  // namespace xsv
