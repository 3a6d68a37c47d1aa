// Gather by the keep list + dimension-adaptive quantization of the whole retained cache
// (paper Sec. 3.3: keys per channel over groups of G kept tokens, values per token over groups of G
// channels), the stateless quantizers, and the canonical unpack used by export.  gfx950.
//
// requant_kernel: one workgroup per (block of 64 new cache positions, head, layer), four waves of 16 positions each.
//   source row of a new position = keep[pos]: a cached token (read through its dequantized bf16
//   view (code - zero) * scale) or a row of the current frame (bf16 as given).
//   Keys: a lane holds ONE channel of the wave's 16 tokens.  The source row is then the same for the whole wave (scalar
//   addresses, whole rows per load), the min / max over a group's tokens and its parameters are the lane's own, and only
//   the packed codes change hands at the end: a transposition of 4-bit (2-bit) codes between 8 (16) lanes, three or four
//   exchanges of a dword, turns "8 tokens of my channel" into "8 channels of my token", the dword the cache stores.
//   Values: a lane holds one token and every fourth channel of it (lane = 16 * quarter + token), so that a gathering load
//   touches four neighbouring channel rows of a source block; min / max in the lane plus two lane exchanges, and the same
//   transposition turns "8 channels of my token" into "8 tokens of my channel", the transposed block the attention
//   kernel's PV product consumes, collected in 2 KB of LDS so that it leaves in whole lines.
//   Writes go to the layer's OTHER buffer, so nothing is updated in place - except in a cache that is never pruned
//   (one buffer): there no row ever moves, a block is read and rewritten by its one workgroup, reads first.
//   Blocks whose rows stay where they are (the first frame's, or every block of old rows while nothing is pruned) are
//   re-quantized from their own dequantized values like everything else, but that reaches a fixed point after a
//   round or two; the step that sees a block come out bit-identical flags it, and from then on it is skipped: both
//   buffers hold it and re-quantizing it can only reproduce it.
// Bound: vector arithmetic (every retained element is read once and written once, packed, but dequantized, compared,
// divided, rounded and packed in between); hence the forms of the quotient and of the rounding below, which are exact.
// One thread per (token, 16 channels) of both tensors, with the keys' extremes through a tile in LDS, two more fused
// multiply-adds per quotient and a conversion per code, took 174 us for the 24 layers of a frame in one launch (16 heads, 4096
// tokens, 4 bits) where this takes 150; with the attention kernel running beside it such a frame went from 941 to 907 us.  One
// layer alone is bound by its dependency chain and gained nothing: 12.5 us before, 13.1 now.
// move_kernel: the same gather for a 16-bit cache, rows copied as they are.
// Compiled with -ffp-contract=off; division is IEEE, rounding is nearest-even.
#include <cstddef>

#include "xsv_internal.h"

#define XSV_QUOTIENT __device__ __forceinline__
namespace xsv {
#include "quotient.h"

__device__ __forceinline__ float round_bf16(float x) { return (float)(__bf16)x; }
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ uint16_t bf16_bits(float x) { return __builtin_bit_cast(unsigned short, (__bf16)x); }
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  const f32x2 v = {a, b};  // one v_cvt_pk_bf16_f32
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

struct QParam {
  float s, z;
  float y;    // 1 / s, correctly rounded; 0 where the group needs the division
};

// Adding kRound to a number below 2^22 in magnitude rounds it to an integer, to nearest even, and leaves that integer in the
// low bits of the sum.
constexpr float kRound = 0x1.8p23f;

// Scale and zero point of a group with these extremes.  y != 0: magnitudes for which no intermediate of exact_quotient
// over- or underflows in a way that could change rint(x / s), and quotients small enough for kRound; anything else (also
// NaN) takes the divisions.
template <int BITS>
__device__ __forceinline__ QParam group_param(float lo, float hi) {
  constexpr float levels = (float)((1 << BITS) - 1), inv = 1.0f / levels;
  constexpr float kBig = 0x1p60f, kSmall = 0x1p-60f, kFar = 0x1p21f;
  const float d = hi - lo;
  QParam p;
  p.s = exact_scale(d, levels, inv);
  if (d == 0.0f) p.s = 1.0f;
  const float mag = fmaxf(fabsf(lo), fabsf(hi));
  const bool safe = p.s >= kSmall && p.s <= kBig && mag <= kBig && mag <= kFar * p.s;
  p.y = safe ? 1.0f / p.s : 0.0f;
  p.z = rintf(exact_quotient(-lo, p.s, p.y));
  if (lo == 0.0f) p.z = -lo;  // (the zero's sign, as the division gives it)
  if (!safe) {
    p.s = d / levels;
    if (p.s == 0.0f) p.s = 1.0f;
    p.z = rintf(-lo / p.s);
  }
  return p;
}

template <int BITS>
__device__ __forceinline__ uint32_t quant_code(float x, float s, float z) {
  constexpr float hi = (float)((1 << BITS) - 1);
  float q = rintf(x / s) + z;
  q = fminf(fmaxf(q, 0.0f), hi);
  return (uint32_t)q;
}

// clamp(rint(x / s) + zero, 0, levels) as the float kRound + (that - zero): `lo` = kRound - zero, `hi` = lo + levels.
// (A NaN comes out as code 0, as it does through the division.)
__device__ __forceinline__ float quant_biased(float x, float s, float y, float lo, float hi) {
  return __builtin_amdgcn_fmed3f(exact_quotient(x, s, y) + kRound, lo, hi);
}

// The codes of 8 elements of one group, packed little endian (4 bits: a dword, 2 bits: the low half of one).
// `fast`: the same for the whole wave, every group of it has y != 0.
template <int BITS>
__device__ __forceinline__ uint32_t quant8(const float* x, const QParam& p, bool fast) {
  uint32_t w = 0;
  if (fast) {
    const float lo = kRound - p.z, hi = lo + (float)((1 << BITS) - 1);
#pragma unroll
    for (int e = 0; e < 8; ++e) w += __float_as_uint(quant_biased(x[e], p.s, p.y, lo, hi)) << (BITS * e);
    w -= __float_as_uint(lo) * (BITS == 4 ? 0x11111111u : 0x5555u);  // the bias of all eight
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) w |= quant_code<BITS>(x[e], p.s, p.z) << (BITS * e);
  }
  return w;
}

// one code (y != 0)
template <int BITS>
__device__ __forceinline__ uint32_t quant_code_fast(float x, float s, float y, float z) {
  const float lo = kRound - z;
  return __float_as_uint(quant_biased(x, s, y, lo, lo + (float)((1 << BITS) - 1))) - __float_as_uint(lo);
}

// ---- transposition of packed codes between lanes ----------------------------------------------------
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t w) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)w, CTRL, 0xf, 0xf, true);
}
// the dword of lane ^ K (K = 1, 2, 4, 8), by lane shifts of the ALU
template <int K>
__device__ __forceinline__ uint32_t lane_xor(uint32_t w) {
  if constexpr (K == 1) return dpp<0xB1>(w);           // quad_perm [1,0,3,2]
  else if constexpr (K == 2) return dpp<0x4E>(w);      // quad_perm [2,3,0,1]
  else if constexpr (K == 4) return dpp<0x1B>(dpp<0x141>(w));  // half-row mirror (^ 7), then quad_perm [3,2,1,0] (^ 3)
  else return dpp<0x128>(w);                           // row rotate by 8
}
template <int BITS, int K>
__device__ __forceinline__ uint32_t transpose_step(uint32_t w, int lane) {
  constexpr int sh = BITS * K;
  // elements whose index has bit K clear
  constexpr uint32_t lo_mask = BITS == 4 ? (K == 1 ? 0x0f0f0f0fu : K == 2 ? 0x00ff00ffu : 0x0000ffffu)
                                         : (K == 1 ? 0x33333333u : K == 2 ? 0x0f0f0f0fu : K == 4 ? 0x00ff00ffu : 0x0000ffffu);
  const bool upper = lane & K;
  const uint32_t p = lane_xor<K>(w);
  const uint32_t keep = upper ? ~lo_mask : lo_mask;
  const uint32_t rot = __builtin_amdgcn_alignbit(p, p, upper ? sh : 32 - sh);  // rotate right by the amount
  return (w & keep) | (rot & ~keep);
}
// Element e of lane l (of 32 / BITS lanes) becomes element l of lane e.
template <int BITS>
__device__ __forceinline__ uint32_t transpose_codes(uint32_t w, int lane) {
  w = transpose_step<BITS, 1>(w, lane);
  w = transpose_step<BITS, 2>(w, lane);
  w = transpose_step<BITS, 4>(w, lane);
  if constexpr (BITS == 2) w = transpose_step<BITS, 8>(w, lane);
  return w;
}

typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
// a: rows 1, 3 (16 lanes each) exchanged with rows 0, 2 of b;  a: upper 32 lanes exchanged with the lower ones of b
__device__ __forceinline__ void swap16(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = r[0]; b = r[1];
}
__device__ __forceinline__ void swap32(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0]; b = r[1];
}
// min / max over the four lanes 16 apart that hold a token's channels
__device__ __forceinline__ float min_quarters(float x) {
  uint32_t a = __float_as_uint(x), b = a;
  swap16(a, b);
  x = fminf(__uint_as_float(a), __uint_as_float(b));
  a = b = __float_as_uint(x);
  swap32(a, b);
  return fminf(__uint_as_float(a), __uint_as_float(b));
}
__device__ __forceinline__ float max_quarters(float x) { return -min_quarters(-x); }

// A token's 64 bf16 channels, 16 consecutive ones per quarter (dwords r[0..7]) -> channel 4 * e + quarter in element e:
// element pairs (e, e + 1) of out[e / 2].  A 4 x 4 transposition between the quarters and the channel index modulo 4.
__device__ __forceinline__ void deal_channels(uint32_t* r, uint32_t* out) {
#pragma unroll
  for (int b = 0; b < 4; ++b) swap32(r[2 * b], r[2 * b + 1]);  // now r[2b + i]: channels from quarters 2i, 2i + 1
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int b = 0; b < 4; b += 2) {
      uint32_t p = __builtin_amdgcn_perm(r[2 * (b + 1) + i], r[2 * b + i], 0x05040100u);  // low halves of both
      uint32_t q = __builtin_amdgcn_perm(r[2 * (b + 1) + i], r[2 * b + i], 0x07060302u);  // high halves
      swap16(p, q);
      out[4 * i + b / 2] = p;      // quarter 2i:     elements 4 * (2i) + b, + b + 1
      out[4 * i + 2 + b / 2] = q;  // quarter 2i + 1
    }
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

// The argument block is read field by field, each read a scalar load that the next instructions wait for, and at the start of
// a launch each of them misses the scalar cache.  One load from every 64-byte line that the kernel will want (the pool, and
// everything behind the pointer tables), waited for once, brings those lines in together.
__device__ __forceinline__ void touch_args(const RequantArgs& a) {
#if defined(__HIP_DEVICE_COMPILE__)  // (the builtin exists in the device pass only)
  const uint32_t* args = static_cast<const uint32_t*>(__builtin_amdgcn_kernarg_segment_ptr());
  constexpr unsigned kTail = offsetof(RequantArgs, b.q_sh) / 4, kLast = (sizeof(RequantArgs) - 4) / 4;
  static_assert(kLast - kTail <= 64, "four lines cover the tail");
  const uint32_t w0 = args[0], w1 = args[16], w2 = args[kTail], w3 = args[kTail + 16], w4 = args[kTail + 32], w5 = args[kLast];
  asm volatile("" ::"s"(w0), "s"(w1), "s"(w2), "s"(w3), "s"(w4), "s"(w5));
#endif
}

constexpr int kWaveRows = 16;  // new positions per wave

// CARRY: RequantArgs::carry_values as a compile-time property (the default path carries no trace of the variant)
template <int BITS, int G, bool CARRY = false>
__global__ __launch_bounds__(256) void requant_kernel(const RequantArgs a) {
  constexpr int kRowDw = kD * BITS / 32;  // dwords per packed key row / value block row
  constexpr int kPer = 32 / BITS;         // elements per dword
  constexpr uint32_t kMask = (1u << BITS) - 1u;
  constexpr int kKGroups = kTile / G;     // key groups per block of 64 tokens (1 or 2)
  constexpr int kVGroups = kD / G;        // value groups per token (1 or 2)
  constexpr int kOut = kWaveRows / kPer;  // dwords of codes per lane and tensor (2 or 1)

  __shared__ float red_lo[4][kD], red_hi[4][kD];
  __shared__ float gs[kKGroups][kD], gz[kKGroups][kD], gy[kKGroups][kD];
  __shared__ __attribute__((aligned(16))) uint32_t vt[kD][kRowDw];  // the block's value codes, [channel][tokens packed]

  touch_args(a);
  const int u = blockIdx.x, h = blockIdx.y, lb = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tok = lane & 15, cq = lane >> 4;  // values: token of the wave, channels 4 * e + cq
  CachePool pool = a.pool;
  pool.bits = BITS;  // (constants from here on)
  pool.G = G;
  const int Tc = a.Tc, Tn = a.Tn, Tcap = pool.Tcap;
  const int layer = a.b.layer0 + lb;
  const int sb = a.b.src_buf(lb);
  const LayerCache src = layer_cache(pool, sb, layer);
  const LayerCache dst = layer_cache(pool, pool.buffers == 1 ? sb : sb ^ 1, layer);
  const int32_t* keep = a.ws.keep + list_index(a.ws.sets, layer, h) * a.ws.scores_stride;
  const int nv = min(kTile, Tn - u * kTile);  // valid new positions in this block

  // A block that holds the same cached rows as before the step and has already reproduced itself is final.
  const bool candidate = u < a.stable_blocks;  // the same for the whole workgroup
  uint8_t* const stable = a.stable_flag + ((size_t)layer * a.pool.H + h) * (Tcap / kTile) + u;
  if (candidate && *stable) return;
  unsigned changed = 0;  // candidate blocks: some code or parameter written differs from what was read

  // source row: arithmetic where the keep list is known without reading it (no dependent load in front of the gather)
  const int r = wave * kWaveRows + tok, pos = u * kTile + r;
  int s_row = -1;
  if (r < nv) s_row = pos < a.identity_end ? pos : (pos >= Tn - a.n ? pos - (Tn - a.n) + Tc : keep[pos]);
  const bool row_valid = s_row >= 0;
  const bool from_cache = row_valid && s_row < Tc;
  const bool wave_valid = wave * kWaveRows < nv;  // the wave holds at least one position
  const bool all_cache = __all(from_cache), any_cache = __any(from_cache);

  // values: all loads are issued here, ahead of the key phase, so that the kernel pays one memory
  // round trip for both; vraw = 16 gathered dwords (cache) or the 8 dwords of the frame row
  uint32_t vraw[16], vfrm[8];
  float v_ps[kVGroups] = {}, v_pz[kVGroups] = {};
  int v_shift = 0;
  if (from_cache) {
    const int blk = s_row / kTile, col = s_row % kTile;
    const uint32_t* vh = reinterpret_cast<const uint32_t*>(src.vc) + (size_t)h * Tcap * kRowDw;
    const uint32_t off = (uint32_t)(blk * kTile + cq) * kRowDw + col / kPer;
    v_shift = (col % kPer) * BITS;
#pragma unroll
    for (int e = 0; e < 16; ++e) vraw[e] = vh[off + e * 4 * kRowDw];
    const float* ps = src.vs + (size_t)h * Tcap * kVGroups;
    const float* pz = src.vz + (size_t)h * Tcap * kVGroups;
#pragma unroll
    for (int g = 0; g < kVGroups; ++g) {
      v_ps[g] = ps[(uint32_t)(s_row * kVGroups + g)];
      v_pz[g] = pz[(uint32_t)(s_row * kVGroups + g)];
    }
  } else {
#pragma unroll
    for (int e = 0; e < 16; ++e) vraw[e] = 0u;
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) vfrm[e] = 0u;
  if (!all_cache && row_valid && !from_cache) {
    const uint4* p = reinterpret_cast<const uint4*>(a.b.v[lb] + (size_t)h * a.b.v_sh + (size_t)(s_row - Tc) * a.b.v_st + cq * 16);
    const uint4 v0 = p[0], v1 = p[1];
    vfrm[0] = v0.x; vfrm[1] = v0.y; vfrm[2] = v0.z; vfrm[3] = v0.w;
    vfrm[4] = v1.x; vfrm[5] = v1.y; vfrm[6] = v1.z; vfrm[7] = v1.w;
  }

  // ---------------- keys: lane = channel ----------------
  float x[kWaveRows];
  float lo = INFINITY, hi = -INFINITY;
  if (wave_valid) {
    // buffer loads: the lane's offset never changes and the row's is a scalar, so a load costs no vector instruction
    // (a head's rows lie within 2 GiB: the cache's by its largest size, the frame's by the host's check)
    const auto codes = buffer_of(src.kc + (size_t)h * Tcap * (kRowDw * 4), (uint32_t)Tcap * (kRowDw * 4));
    const uint32_t prm_bytes = (uint32_t)(Tcap / G) * (kD * 4);
    const auto scales = buffer_of(src.ks + (size_t)h * (Tcap / G) * kD, prm_bytes);
    const auto zeros = buffer_of(src.kz + (size_t)h * (Tcap / G) * kD, prm_bytes);
    const uint32_t k_row = (uint32_t)a.b.k_st * 2u;  // bytes
    const auto frame = buffer_of(a.b.k[lb] + (size_t)h * a.b.k_sh, (uint32_t)(a.n - 1) * k_row + kD * 2u);
    const uint32_t dw4 = (unsigned)lane / kPer * 4u, lane4 = (unsigned)lane * 4u, sh = ((unsigned)lane % kPer) * BITS;
    auto code_word = [&](uint32_t row) { return __builtin_amdgcn_raw_buffer_load_b32(codes, dw4, row * (kRowDw * 4u), 0); };
    auto scale_of = [&](uint32_t row) { return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(scales, lane4, row / G * (kD * 4u), 0)); };
    auto zero_of = [&](uint32_t row) { return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(zeros, lane4, row / G * (kD * 4u), 0)); };
    auto frame_word = [&](uint32_t row) { return (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(frame, lane4 >> 1, row * k_row, 0); };
    if (all_cache) {
      uint32_t w[kWaveRows];
      float s[kWaveRows], z[kWaveRows];
#pragma unroll
      for (int t = 0; t < kWaveRows; ++t) {
        const uint32_t row = (uint32_t)__builtin_amdgcn_readlane(s_row, t);
        w[t] = code_word(row);
        s[t] = scale_of(row);
        z[t] = zero_of(row);
      }
#pragma unroll
      for (int t = 0; t < kWaveRows; t += 2) {
        const uint32_t pk = pack_bf16(((float)((w[t] >> sh) & kMask) - z[t]) * s[t], ((float)((w[t + 1] >> sh) & kMask) - z[t + 1]) * s[t + 1]);
        x[t] = bf16_lo(pk);
        x[t + 1] = bf16_hi(pk);
      }
    } else {
      // (positions past the end repeat the wave's first row: no new minimum or maximum)
      const int row0 = __builtin_amdgcn_readlane(s_row, 0);
      if (!any_cache) {
        uint32_t w[kWaveRows];
#pragma unroll
        for (int t = 0; t < kWaveRows; ++t) {
          const int row = __builtin_amdgcn_readlane(s_row, t);
          w[t] = frame_word((uint32_t)((row < 0 ? row0 : row) - Tc));
        }
#pragma unroll
        for (int t = 0; t < kWaveRows; ++t) x[t] = bf16_lo(w[t]);
      } else {
#pragma unroll
        for (int t = 0; t < kWaveRows; ++t) {
          int row = __builtin_amdgcn_readlane(s_row, t);
          if (row < 0) row = row0;
          if (row < Tc) x[t] = round_bf16(((float)((code_word(row) >> sh) & kMask) - zero_of(row)) * scale_of(row));
          else x[t] = bf16_lo(frame_word((uint32_t)(row - Tc)));
        }
      }
    }
#pragma unroll
    for (int t = 0; t < kWaveRows; ++t) {
      lo = fminf(lo, x[t]);
      hi = fmaxf(hi, x[t]);
    }
  }
  // token ids travel with the rows (one copy per index set: head 0 writes the shared one)
  if ((h == 0 || a.ws.sets > 1) && cq == 0 && row_valid) {
    const size_t row0 = a.ws.sets > 1 ? (size_t)h * Tcap : 0;
    dst.tok_frame[row0 + pos] = from_cache ? src.tok_frame[row0 + s_row] : a.frame_id;
    dst.tok_index[row0 + pos] = from_cache ? src.tok_index[row0 + s_row] : s_row - Tc;
  }
  red_lo[wave][lane] = lo;
  red_hi[wave][lane] = hi;
  __syncthreads();
  if (wave < kKGroups && wave * G < nv) {  // one wave works out a group's parameters, the others go on to the values
    constexpr int parts = 4 / kKGroups;    // waves per group
    float l = red_lo[wave * parts][lane], m = red_hi[wave * parts][lane];
#pragma unroll
    for (int p = 1; p < parts; ++p) {
      l = fminf(l, red_lo[wave * parts + p][lane]);
      m = fmaxf(m, red_hi[wave * parts + p][lane]);
    }
    const QParam q = group_param<BITS>(l, m);
    gs[wave][lane] = q.s;
    gz[wave][lane] = q.z;
    gy[wave][lane] = q.y;
    const size_t gidx = ((size_t)h * (Tcap / G) + (size_t)u * kKGroups + wave) * kD + lane;
    if (candidate) changed |= (__float_as_uint(src.ks[gidx]) ^ __float_as_uint(q.s)) | (__float_as_uint(src.kz[gidx]) ^ __float_as_uint(q.z));
    dst.ks[gidx] = q.s;
    dst.kz[gidx] = q.z;
  }

  // ---------------- values: lane = (token, every fourth channel) ----------------
  // "quantize once" (carry_values): a row that comes from the cache keeps its codes and parameters; a wave whose rows
  // all do skips the arithmetic altogether
  uint32_t vw[kOut];
  if (wave_valid) {
    QParam q[kVGroups];
    if (!(CARRY && all_cache)) {
      float v[16];
      if (all_cache || any_cache) {
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
          const int g = e * 4 / G;
          const uint32_t pk = pack_bf16(((float)((vraw[e] >> v_shift) & kMask) - v_pz[g]) * v_ps[g],
                                        ((float)((vraw[e + 1] >> v_shift) & kMask) - v_pz[g]) * v_ps[g]);
          v[e] = bf16_lo(pk);
          v[e + 1] = bf16_hi(pk);
        }
      }
      if (!all_cache) {
        uint32_t d[8];
        deal_channels(vfrm, d);
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
          v[e] = any_cache && from_cache ? v[e] : bf16_lo(d[e / 2]);
          v[e + 1] = any_cache && from_cache ? v[e + 1] : bf16_hi(d[e / 2]);
        }
      }
      bool fast = true;
#pragma unroll
      for (int g = 0; g < kVGroups; ++g) {
        constexpr int n = 16 / kVGroups;
        float l = v[g * n], m = v[g * n];
#pragma unroll
        for (int e = 1; e < n; ++e) {
          l = fminf(l, v[g * n + e]);
          m = fmaxf(m, v[g * n + e]);
        }
        q[g] = group_param<BITS>(min_quarters(l), max_quarters(m));
        fast = fast && q[g].y != 0.0f;
      }
      fast = __all(fast);
      const uint32_t w0 = quant8<BITS>(v, q[0], fast), w1 = quant8<BITS>(v + 8, q[kVGroups - 1], fast);
      if constexpr (BITS == 4) { vw[0] = w0; vw[kOut - 1] = w1; }
      else vw[0] = w0 | (w1 << 16);
    }
    if constexpr (CARRY) {  // the row's own codes and parameters, as read
      uint32_t cw[kOut];
#pragma unroll
      for (int i = 0; i < kOut; ++i) cw[i] = 0;
#pragma unroll
      for (int e = 0; e < 16; ++e) cw[e / kPer] |= ((vraw[e] >> v_shift) & kMask) << (BITS * (e % kPer));
#pragma unroll
      for (int i = 0; i < kOut; ++i) vw[i] = all_cache || from_cache ? cw[i] : vw[i];
#pragma unroll
      for (int g = 0; g < kVGroups; ++g) {
        q[g].s = all_cache || from_cache ? v_ps[g] : q[g].s;
        q[g].z = all_cache || from_cache ? v_pz[g] : q[g].z;
      }
    }
    if (row_valid && cq < kVGroups) {
      const int g = kVGroups == 1 ? 0 : cq;
      const float s = kVGroups > 1 && cq ? q[kVGroups - 1].s : q[0].s, z = kVGroups > 1 && cq ? q[kVGroups - 1].z : q[0].z;
      const size_t gidx = ((size_t)h * Tcap + (size_t)u * kTile + r) * kVGroups + g;
      if (candidate) {
        const float s0 = kVGroups > 1 && cq ? v_ps[kVGroups - 1] : v_ps[0], z0 = kVGroups > 1 && cq ? v_pz[kVGroups - 1] : v_pz[0];
        changed |= (__float_as_uint(s0) ^ __float_as_uint(s)) | (__float_as_uint(z0) ^ __float_as_uint(z));
      }
      dst.vs[gidx] = s;
      dst.vz[gidx] = z;
    }
  }
#pragma unroll
  for (int d = 0; d < kOut; ++d) {
    // (positions past the end of the cache hold zeros)
    const uint32_t w = transpose_codes<BITS>(wave_valid && row_valid ? vw[d] : 0u, lane);
    const int e = d * kPer + (lane & (kPer - 1));  // the lane's element after the transposition: channel 4 * e + cq
    vt[4 * e + cq][wave * kOut + (BITS == 4 ? tok >> 3 : 0)] = w;
  }
  __syncthreads();

  // ---------------- keys, second half: codes ----------------
  if (wave_valid) {
    const int gi = wave * kWaveRows / G;
    QParam q;
    q.s = gs[gi][lane];
    q.z = gz[gi][lane];
    q.y = gy[gi][lane];
    const bool fast = __all(q.y != 0.0f);
    const uint32_t w0 = quant8<BITS>(x, q, fast), w1 = quant8<BITS>(x + 8, q, fast);
    uint32_t kw[kOut];
    if constexpr (BITS == 4) { kw[0] = w0; kw[kOut - 1] = w1; }
    else kw[0] = w0 | (w1 << 16);
    const size_t base = ((size_t)h * Tcap + (size_t)u * kTile) * kRowDw;
    uint32_t* out = reinterpret_cast<uint32_t*>(dst.kc) + base;
    const uint32_t* old = reinterpret_cast<const uint32_t*>(src.kc) + base;
#pragma unroll
    for (int d = 0; d < kOut; ++d) {
      const uint32_t w = transpose_codes<BITS>(kw[d], lane);
      const int row = wave * kWaveRows + d * kPer + (lane & (kPer - 1));
      const unsigned at = (unsigned)row * kRowDw + (unsigned)lane / kPer;
      if (row < nv) {
        if (candidate) changed |= w ^ old[at];
        out[at] = w;
      }
    }
  }
  {  // the value block, whole lines
    const size_t base = ((size_t)h * Tcap + (size_t)u * kTile) * kRowDw;
    const unsigned at = tid * (kRowDw / 4);
    uint32_t* out = reinterpret_cast<uint32_t*>(dst.vc) + base;
    const uint32_t* old = reinterpret_cast<const uint32_t*>(src.vc) + base;
#pragma unroll
    for (int i = 0; i < kRowDw / 4; ++i) {
      const uint32_t w = (&vt[0][0])[at + i];
      if (candidate) changed |= w ^ old[at + i];
      out[at + i] = w;
    }
  }
  if (candidate) {  // did the block reproduce itself?
    const int any = __syncthreads_or(changed != 0);
    if (tid == 0) *stable = any ? 0 : 1;
  } else if (tid == 0) {
    *stable = 0;  // a block whose rows may move carries no flag into a later step in which they do not
  }
}

// A 16-bit cache: the kept rows copied to their new places.  Thread = (token tid/4 of the block, channel quarter tid%4); a
// value row is gathered from the transposed blocks and goes through LDS to come out transposed again.  In a cache that is never
// pruned that is the frame's rows and the block they begin in; blocks that an earlier step has flagged are not launched at all
// (four layers, 16 frames of 16 x 1374 tokens: up to 5504 workgroups of which 352 have something to do took 8.5 us a step, 704 take 5.8).
__global__ __launch_bounds__(256) void move_kernel(const RequantArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t vt[kD][kTile + 8];  // [channel][token]
  const int u = blockIdx.x + a.first_block, h = blockIdx.y, lb = blockIdx.z;
  const int tid = threadIdx.x, r = tid >> 2, cq = tid & 3;
  const int Tc = a.Tc, Tn = a.Tn, Tcap = a.pool.Tcap;
  const int layer = a.b.layer0 + lb;
  const int sb = a.b.src_buf(lb);
  const LayerCache src = layer_cache(a.pool, sb, layer);
  const LayerCache dst = layer_cache(a.pool, a.pool.buffers == 1 ? sb : sb ^ 1, layer);
  const int32_t* keep = a.ws.keep + list_index(a.ws.sets, layer, h) * a.ws.scores_stride;
  const int nv = min(kTile, Tn - u * kTile);
  const bool candidate = u < a.stable_blocks;  // (a copied block always reproduces itself: the flag is set by its first step)
  uint8_t* const stable = a.stable_flag + ((size_t)layer * a.pool.H + h) * (Tcap / kTile) + u;
  if (candidate && *stable) return;
  if (candidate && a.pool.buffers == 1) {  // (its rows are where they belong)
    if (tid == 0) *stable = 1;
    return;
  }
  const int pos = u * kTile + r;
  int s_row = -1;
  if (r < nv) s_row = pos < a.identity_end ? pos : (pos >= Tn - a.n ? pos - (Tn - a.n) + Tc : keep[pos]);
  const bool row_valid = s_row >= 0;
  const bool from_cache = row_valid && s_row < Tc;
  if ((h == 0 || a.ws.sets > 1) && cq == 0 && row_valid) {
    const size_t row0 = a.ws.sets > 1 ? (size_t)h * Tcap : 0;
    dst.tok_frame[row0 + pos] = from_cache ? src.tok_frame[row0 + s_row] : a.frame_id;
    dst.tok_index[row0 + pos] = from_cache ? src.tok_index[row0 + s_row] : s_row - Tc;
  }
  uint4 k0 = make_uint4(0, 0, 0, 0), k1 = k0;
  uint16_t v[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) v[e] = 0;
  if (row_valid) {
    const uint16_t* kr = from_cache ? reinterpret_cast<const uint16_t*>(src.kc) + ((size_t)h * Tcap + s_row) * kD
                                    : a.b.k[lb] + (size_t)h * a.b.k_sh + (size_t)(s_row - Tc) * a.b.k_st;
    const uint4* p = reinterpret_cast<const uint4*>(kr + cq * 16);
    k0 = p[0];
    k1 = p[1];
  }
  if (from_cache) {
    const uint16_t* rows = reinterpret_cast<const uint16_t*>(src.vc) + ((size_t)h * Tcap + (size_t)(s_row / kTile) * kTile) * kD + s_row % kTile;
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = rows[(size_t)(cq * 16 + e) * kD];
  } else if (row_valid) {
    const uint4* p = reinterpret_cast<const uint4*>(a.b.v[lb] + (size_t)h * a.b.v_sh + (size_t)(s_row - Tc) * a.b.v_st + cq * 16);
    const uint4 v0 = p[0], v1 = p[1];
    const uint32_t ww[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) { v[2 * e] = (uint16_t)ww[e]; v[2 * e + 1] = (uint16_t)(ww[e] >> 16); }
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) vt[cq * 16 + e][r] = v[e];
  __syncthreads();  // (one buffer: every row of the block has been read)
  if (row_valid) {
    uint4* out = reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(dst.kc) + ((size_t)h * Tcap + (size_t)u * kTile + r) * kD + cq * 16);
    out[0] = k0;
    out[1] = k1;
  }
  {  // thread = (channel tid/4, token quarter tid%4)
    const int c = tid >> 2, tq = tid & 3;
    uint4* out = reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(dst.vc) + ((size_t)h * Tcap + (size_t)u * kTile + c) * kD + tq * 16);
    out[0] = *reinterpret_cast<const uint4*>(&vt[c][tq * 16]);
    out[1] = *reinterpret_cast<const uint4*>(&vt[c][tq * 16 + 8]);
  }
  if (tid == 0) *stable = candidate ? 1 : 0;
}

// Clears the block flags (a kernel rather than a memset node: a caller may capture the stream, and memset nodes in
// captured graphs have replayed wrongly on this platform).
__global__ __launch_bounds__(256) void zero_bytes_kernel(uint8_t* p, size_t n) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0;
}

hipError_t launch_zero_bytes(uint8_t* p, size_t n, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(zero_bytes_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, p, n);
  return hipGetLastError();
}

hipError_t launch_requant(const RequantArgs& a, hipStream_t stream) {
  if (a.Tn <= 0) return hipSuccess;
  const dim3 grid((a.Tn + kTile - 1) / kTile - a.first_block, a.pool.H, a.b.n_layers);
  const int bits = a.pool.bits, G = a.pool.G;
  const bool carry = a.carry_values != 0 && bits != 16;
  if (bits == 16) hipLaunchKernelGGL(move_kernel, grid, dim3(256), 0, stream, a);
  else if (bits == 4 && G == 64 && !carry) hipLaunchKernelGGL((requant_kernel<4, 64>), grid, dim3(256), 0, stream, a);
  else if (bits == 4 && G == 32 && !carry) hipLaunchKernelGGL((requant_kernel<4, 32>), grid, dim3(256), 0, stream, a);
  else if (bits == 2 && G == 64 && !carry) hipLaunchKernelGGL((requant_kernel<2, 64>), grid, dim3(256), 0, stream, a);
  else if (bits == 2 && G == 32 && !carry) hipLaunchKernelGGL((requant_kernel<2, 32>), grid, dim3(256), 0, stream, a);
  else if (bits == 4 && G == 64) hipLaunchKernelGGL((requant_kernel<4, 64, true>), grid, dim3(256), 0, stream, a);
  else if (bits == 4 && G == 32) hipLaunchKernelGGL((requant_kernel<4, 32, true>), grid, dim3(256), 0, stream, a);
  else if (bits == 2 && G == 64) hipLaunchKernelGGL((requant_kernel<2, 64, true>), grid, dim3(256), 0, stream, a);
  else if (bits == 2 && G == 32) hipLaunchKernelGGL((requant_kernel<2, 32, true>), grid, dim3(256), 0, stream, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// ---- the stateless quantizers ------------------------------------------------------------------------
// A plain bf16 tensor [H][T][64] straight to canonical codes (a byte each), scales and zero points: one workgroup per
// (block of 64 tokens, head), thread = (token tid/4, 16 channels), one read of the tensor and one write of the result.
// The arithmetic is requant_kernel's.  The order of the elements in a min / max is not, and need not be: the hardware takes -0
// for smaller than +0, so a group of zeros of both signs has the same extremes, and zero point, in any order.  Bound: memory, in
// principle - at 16 heads x 4096 tokens a launch moves 13 MB and takes less time than launching it and waiting for it (the calls
// are synchronous).  Keys and values of that size take 51 us, and took 1.2 to 5.7 ms as a throw-away context that was filled,
// re-quantized and unpacked (its allocations vary by that much).
// `wide`: the codes' address allows 16-byte stores (any address is accepted).
__device__ __forceinline__ void load_row16(const uint16_t* p, float* x) {
  const uint4* p4 = reinterpret_cast<const uint4*>(p);
  const uint4 v0 = p4[0], v1 = p4[1];
  const uint32_t ww[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
  for (int e = 0; e < 8; ++e) { x[2 * e] = bf16_lo(ww[e]); x[2 * e + 1] = bf16_hi(ww[e]); }
}

__device__ __forceinline__ void store_codes16(uint8_t* out, const uint32_t* code, bool wide) {
  if (wide) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = code[4 * i] | (code[4 * i + 1] << 8) | (code[4 * i + 2] << 16) | (code[4 * i + 3] << 24);
    *reinterpret_cast<uint4*>(out) = make_uint4(w[0], w[1], w[2], w[3]);
  } else {
#pragma unroll
    for (int e = 0; e < 16; ++e) out[e] = (uint8_t)code[e];
  }
}

template <int BITS, int G>
__global__ __launch_bounds__(256) void quantize_keys_kernel(const QuantizeArgs a) {
  constexpr int kKGroups = kTile / G;
  __shared__ float xk[kTile][kD + 1];
  __shared__ float red_lo[4][kD], red_hi[4][kD];
  __shared__ float gs[kKGroups][kD], gz[kKGroups][kD], gy[kKGroups][kD];
  __shared__ int k_unsafe;
  const int u = blockIdx.x, h = blockIdx.y, tid = threadIdx.x, r = tid >> 2, cq = tid & 3;
  const int nv = min(kTile, a.T - u * kTile);
  const size_t row = (size_t)h * a.T + (size_t)u * kTile + r;
  if (tid == 0) k_unsafe = 0;
  float x[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) x[e] = 0.f;
  if (r < nv) load_row16(a.x + row * kD + cq * 16, x);
#pragma unroll
  for (int e = 0; e < 16; ++e) xk[r][cq * 16 + e] = x[e];
  __syncthreads();
  {
    const int c = tid & 63, part = tid >> 6;
    float lo = INFINITY, hi = -INFINITY;
    for (int i = part * 16; i < min(nv, part * 16 + 16); ++i) {
      lo = fminf(lo, xk[i][c]);
      hi = fmaxf(hi, xk[i][c]);
    }
    red_lo[part][c] = lo;
    red_hi[part][c] = hi;
  }
  __syncthreads();
  if (tid < kKGroups * kD) {
    const int c = tid & 63, gi = tid >> 6;
    constexpr int parts = 4 / kKGroups;
    if (gi * G < nv) {
      float lo = red_lo[gi * parts][c], hi = red_hi[gi * parts][c];
#pragma unroll
      for (int p = 1; p < parts; ++p) {
        lo = fminf(lo, red_lo[gi * parts + p][c]);
        hi = fmaxf(hi, red_hi[gi * parts + p][c]);
      }
      const QParam q = group_param<BITS>(lo, hi);
      gs[gi][c] = q.s;
      gz[gi][c] = q.z;
      gy[gi][c] = q.y;
      if (q.y == 0.0f) k_unsafe = 1;
      const size_t gidx = ((size_t)h * ((a.T + G - 1) / G) + (size_t)u * kKGroups + gi) * kD + c;
      a.scale[gidx] = q.s;
      a.zero[gidx] = q.z;
    }
  }
  __syncthreads();
  if (r >= nv) return;
  const int gi = r / G;
  uint32_t code[16];
  if (!k_unsafe) {
#pragma unroll
    for (int e = 0; e < 16; ++e) code[e] = quant_code_fast<BITS>(x[e], gs[gi][cq * 16 + e], gy[gi][cq * 16 + e], gz[gi][cq * 16 + e]);
  } else {
#pragma unroll
    for (int e = 0; e < 16; ++e) code[e] = quant_code<BITS>(x[e], gs[gi][cq * 16 + e], gz[gi][cq * 16 + e]);
  }
  store_codes16(a.codes + row * kD + cq * 16, code, a.wide);
}

template <int BITS, int G>
__global__ __launch_bounds__(256) void quantize_values_kernel(const QuantizeArgs a) {
  const int h = blockIdx.y, tid = threadIdx.x, r = tid >> 2, cq = tid & 3;
  const bool valid = (long long)blockIdx.x * kTile + r < a.T;
  const size_t row = (size_t)h * a.T + (size_t)blockIdx.x * kTile + r;
  float x[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) x[e] = 0.f;
  if (valid) load_row16(a.x + row * kD + cq * 16, x);
  float lo = x[0], hi = x[0];
#pragma unroll
  for (int e = 1; e < 16; ++e) { lo = fminf(lo, x[e]); hi = fmaxf(hi, x[e]); }
  lo = fminf(lo, __shfl_xor(lo, 1));
  hi = fmaxf(hi, __shfl_xor(hi, 1));
  if (G == 64) {
    lo = fminf(lo, __shfl_xor(lo, 2));
    hi = fmaxf(hi, __shfl_xor(hi, 2));
  }
  const QParam q = group_param<BITS>(lo, hi);
  uint32_t code[16];
  if (__all(q.y != 0.0f)) {
#pragma unroll
    for (int e = 0; e < 16; ++e) code[e] = quant_code_fast<BITS>(x[e], q.s, q.y, q.z);
  } else {
#pragma unroll
    for (int e = 0; e < 16; ++e) code[e] = quant_code<BITS>(x[e], q.s, q.z);
  }
  if (!valid) return;
  if ((cq * 16) % G == 0) {
    const size_t gidx = row * (kD / G) + (cq * 16) / G;
    a.scale[gidx] = q.s;
    a.zero[gidx] = q.z;
  }
  store_codes16(a.codes + row * kD + cq * 16, code, a.wide);
}

template <int BITS, int G>
static hipError_t launch_quantize_t(const QuantizeArgs& a, bool keys, hipStream_t stream) {
  const dim3 grid((a.T + kTile - 1) / kTile, a.H);
  if (keys) hipLaunchKernelGGL((quantize_keys_kernel<BITS, G>), grid, dim3(256), 0, stream, a);
  else hipLaunchKernelGGL((quantize_values_kernel<BITS, G>), grid, dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_quantize_plain(const QuantizeArgs& a, int bits, int G, bool keys, hipStream_t stream) {
  if (bits == 4 && G == 64) return launch_quantize_t<4, 64>(a, keys, stream);
  if (bits == 4 && G == 32) return launch_quantize_t<4, 32>(a, keys, stream);
  if (bits == 2 && G == 64) return launch_quantize_t<2, 64>(a, keys, stream);
  if (bits == 2 && G == 32) return launch_quantize_t<2, 32>(a, keys, stream);
  return hipErrorInvalidValue;
}

// ---- canonical unpack: thread per (head, token, channel) -------------------------------------------
template <int BITS>
__global__ __launch_bounds__(256) void unpack_kernel(const UnpackArgs a) {
  constexpr bool kQuant = BITS != 16;
  constexpr int kRowDw = kD * BITS / 32;
  constexpr int kPer = kQuant ? 32 / BITS : 2;
  constexpr uint32_t kMask = kQuant ? (1u << (BITS & 15)) - 1u : 0xffffu;
  const int H = a.pool.H, T = a.T, Tcap = a.pool.Tcap, G = a.pool.G;
  const size_t gid = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (gid >= (size_t)H * T * kD) return;
  const int c = (int)(gid % kD);
  const int t = (int)((gid / kD) % T);
  const int h = (int)(gid / ((size_t)kD * T));
  const LayerCache lc = layer_cache(a.pool, a.buf, a.layer);
  const uint32_t* krow = reinterpret_cast<const uint32_t*>(lc.kc) + ((size_t)h * Tcap + t) * kRowDw;
  const uint32_t* vrow = reinterpret_cast<const uint32_t*>(lc.vc) + ((size_t)h * Tcap + (size_t)(t / kTile) * kTile + c) * kRowDw;
  const uint32_t kcode = (krow[c / kPer] >> ((c % kPer) * BITS)) & kMask;
  const int col = t % kTile;
  const uint32_t vcode = (vrow[col / kPer] >> ((col % kPer) * BITS)) & kMask;
  if constexpr (kQuant) {
    const int ng = (T + G - 1) / G, vg = kD / G;
    const float ks = lc.ks[((size_t)h * (Tcap / G) + t / G) * kD + c], kz = lc.kz[((size_t)h * (Tcap / G) + t / G) * kD + c];
    const float vs = lc.vs[((size_t)h * Tcap + t) * vg + c / G], vz = lc.vz[((size_t)h * Tcap + t) * vg + c / G];
    if (a.k_codes) a.k_codes[gid] = (uint8_t)kcode;
    if (a.v_codes) a.v_codes[gid] = (uint8_t)vcode;
    if (t % G == 0) {
      if (a.k_scale) a.k_scale[((size_t)h * ng + t / G) * kD + c] = ks;
      if (a.k_zero) a.k_zero[((size_t)h * ng + t / G) * kD + c] = kz;
    }
    if (c % G == 0) {
      if (a.v_scale) a.v_scale[((size_t)h * T + t) * vg + c / G] = vs;
      if (a.v_zero) a.v_zero[((size_t)h * T + t) * vg + c / G] = vz;
    }
    if (a.k_bf16) a.k_bf16[gid] = bf16_bits(((float)kcode - kz) * ks);
    if (a.v_bf16) a.v_bf16[gid] = bf16_bits(((float)vcode - vz) * vs);
  } else {
    if (a.k_bf16) a.k_bf16[gid] = (uint16_t)kcode;
    if (a.v_bf16) a.v_bf16[gid] = (uint16_t)vcode;
  }
}

hipError_t launch_unpack(const UnpackArgs& a, hipStream_t stream) {
  const size_t total = (size_t)a.pool.H * a.T * kD;
  if (total == 0) return hipSuccess;
  const dim3 grid((unsigned)((total + 255) / 256));
  if (a.pool.bits == 16) hipLaunchKernelGGL((unpack_kernel<16>), grid, dim3(256), 0, stream, a);
  else if (a.pool.bits == 4) hipLaunchKernelGGL((unpack_kernel<4>), grid, dim3(256), 0, stream, a);
  else if (a.pool.bits == 2) hipLaunchKernelGGL((unpack_kernel<2>), grid, dim3(256), 0, stream, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace xsv
