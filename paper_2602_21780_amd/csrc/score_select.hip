// Token importance and keep-list selection (paper Sec. 3.2) for gfx950.
//
// The importance  S_j = (1/N_pooled) sum_i (Qbar Kbar^T)[i][j]  is linear in the pooled queries, so
// it is evaluated as  S_j = qtilde . Kbar_j  with  qtilde = (1/N_pooled) sum_i Qbar_i.  Three parts:
//   pool    one pass over Q: weighted row sums (weight 1/(H N_pooled) for a special
//           row, 1/(H N_pooled |group|) for a patch row), two workgroups and kPoolParts partials per head, added up
//           by everybody who needs qtilde in one fixed order: reproducible bit for bit, no atomics on floats.
//   score   one pass over the packed keys of the prunable middle: dequantized view,
//           head mean, dot product with qtilde.  64 tokens x all heads per workgroup, 8 channels per thread, all loads of a
//           workgroup issued before any use.  (Per-head lists: 256 tokens x one head.)
//   select  exact top-k by radix select on order-preserving integer keys held in
//           registers (digits of 11, 11 and 10 bits, histograms in LDS), ties at the threshold resolved toward smaller
//           positions, then an ordered compaction that emits the keep list ascending.
// front_kernel is all three in one launch for one layer, a role per workgroup.  Each part takes a few microseconds, most of it the latency of
// a kernel's start, of its arguments and of one or two trips to memory: one layer of 16 heads x 1374 tokens with 2722 middle
// positions took 21.2 us as three kernels with nothing beside them, and takes 13.8 as one.  Beside attention, as a step runs it,
// the kernel takes 17.2 us where 64 compute units are free, the three took 7.9 + 8.9 + 10.2 (medians of traces).  (61 registers, three
// workgroups to a compute unit; with the pool of last resort unrolled like the first, 120 to 139, and steps that wait for the chain are 1
// to 2 % slower.  So few registers that a workgroup fits beside attention's 32-row shapes, which does harm: launch_attend_t.)
// Nothing in it waits without end, whatever else is on the chip.  The workgroup that completes a list's scores goes on to select
// it.  A score workgroup does wait for the pool (only at the end, with the key means in registers), which has smaller indices and
// as a rule has been started before it; but launches of several streams may hold the places each other's pools need, so the wait
// is bounded (FrontCommon::polls) and a workgroup that runs out of patience pools the queries itself, in the same order.  What is
// handed over goes through agent-scope stores and loads (past the caches that the dies of the chip do not share) and one counter
// per list, which the last workgroup to arrive puts back to zero.
//   Per-head variant (FrontCommon::per_head, not the paper's): the averages over heads are left out,
//   qtilde_h comes from head h's partials alone and head h's keys give head h's own score vector and list.
// Compiled with -ffp-contract=off: the dequantized view must be (code - zero) * scale with one
// rounding per operation.
#include <type_traits>

#include "xsv_internal.h"

namespace xsv {

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

constexpr int kThreads = 512;    // of pool, select and (but for plain keys) score
constexpr int kHeadChunk = 16;   // heads whose keys a score workgroup holds in registers at a time

// ---- handing over between workgroups ------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ T load_agent(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ __forceinline__ void store_agent(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// FrontLayer::sync, one per list: pool workgroups that are done in the low half, score workgroups in the high half.
constexpr uint64_t kPoolArrived = 1, kScoreArrived = 1ull << 32;
// This workgroup's part is done; to thread 0 (only): the counter before that.  The last to arrive leaves zero.
// (A wave's agent-scope stores have reached memory when its count of outstanding ones is zero.)
__device__ __forceinline__ uint64_t arrive(uint64_t* counter, uint64_t mine, uint64_t all) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  uint64_t before = 0;
  if (threadIdx.x == 0) {
    before = __hip_atomic_fetch_add(counter, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (before + mine == all) store_agent(counter, (uint64_t)0);
  }
  return before;
}
// `n` pool workgroups are done; false if they were not in the time that `polls` looks take.
__device__ __forceinline__ bool wait_for_pool(const uint64_t* counter, uint32_t n, int polls) {
  bool done = false;
  for (int i = 0; i < polls && !done; ++i) {
    done = (uint32_t)load_agent(counter) == n;
    if (!done) __builtin_amdgcn_s_sleep(1);
  }
  asm volatile("" ::: "memory");
  return done;
}
// A list's arrivals.
__device__ __forceinline__ uint32_t pools_of(const FrontCommon& a, bool per_head) { return per_head ? 2u : 2u * a.H; }
__device__ __forceinline__ uint64_t all_of(const FrontCommon& a, bool per_head) {
  return pools_of(a, per_head) * kPoolArrived + (uint64_t)a.blocks * kScoreArrived;
}

// ---- pool ----------------------------------------------------------------------------------------------
constexpr int kPoolLds = (kThreads / 8) * (kD + 1);
// Thread = (row lane, channel run).  A head has 128 row lanes (lane i: rows i, i + 128, ..), 64 to each of its two workgroups,
// and each 32 lanes' sum is a partial: returned by threads tid < 128 for partial 2 * half + tid / 64, channel tid % 64.
template <int ROWS>
__device__ __forceinline__ float pool_partial(const FrontLayer& ly, const FrontCommon& a, int h, int half, float* lds) {
  float(*red)[kD + 1] = reinterpret_cast<float(*)[kD + 1]>(lds);
  const int H = a.H, n = a.n, n_s = a.n_special, g = a.pool_size;
  const int n_groups = (n - n_s + g - 1) / g, n_pooled = n_s + n_groups;
  const int tid = threadIdx.x, rl = tid >> 3, o = tid & 7;
  const uint16_t* qh = ly.q + (size_t)h * a.q_sh + o * 8;
  const float base = a.per_head ? (float)n_pooled : (float)(H * n_pooled);
  // a special row, a row of a whole group, a row of the last group
  const int last = n_s + (n_groups - 1) * g;  // its first row
  const float w_special = 1.0f / base, w_whole = 1.0f / (base * (float)min(g, n - n_s)), w_last = 1.0f / (base * (float)(n - last));
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // ROWS rows of a row lane are in flight together (rows past the frame: weight 0); with six, 1374 rows take two trips to
  // memory (an unrolled loop and its rest took two and one for every row of the rest: 4.8 us alone, 4.2 like this)
  for (int r0 = half * 64 + rl; r0 < n; r0 += 128 * ROWS) {
    uint4 v[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      const int r = r0 + 128 * i;
      v[i] = r < n ? *reinterpret_cast<const uint4*>(qh + (size_t)r * a.q_st) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      const int r = r0 + 128 * i;
      const float w = r < n_s ? w_special : (r < last ? w_whole : (r < n ? w_last : 0.f));
      const uint32_t ww[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[2 * e] += w * bf16_lo(ww[e]);
        acc[2 * e + 1] += w * bf16_hi(ww[e]);
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[rl][o * 8 + e] = acc[e];
  __syncthreads();
  float s = 0.f;
  if (tid < 2 * kD) {
    const int sg = tid >> 6, c = tid & 63;
#pragma unroll
    for (int i = 0; i < 32; ++i) s += red[sg * 32 + i][c];
  }
  return s;
}
template <bool SYNC>
__device__ __forceinline__ void pool_part(const FrontLayer& ly, const FrontCommon& a, int h, int half, float* lds) {
  // (rows that are not there cost arithmetic all the same: a step of 14 x 58 tokens 24.3 us with six, 23.8 with two)
  const float s = a.n > 256 ? pool_partial<6>(ly, a, h, half, lds) : pool_partial<2>(ly, a, h, half, lds);
  const int tid = threadIdx.x;
  if (tid < 2 * kD) {
    float* out = ly.qpart + ((size_t)h * kPoolParts + half * 2) * kD + tid;
    if (SYNC) store_agent(out, s);
    else *out = s;
  }
  if (SYNC) arrive(ly.sync + (a.per_head ? h : 0), kPoolArrived, all_of(a, a.per_head));
}

static_assert(kPoolParts == 4, "the order of the sums");
__device__ __forceinline__ float add_partials(const float* x) { return ((x[0] + x[1]) + x[2]) + x[3]; }
// Channel c of head h's pooled query: its partials in order.
template <bool SYNC>
__device__ __forceinline__ float head_query(const FrontLayer& ly, int h, int c) {
  const float* p = ly.qpart + (size_t)h * kPoolParts * kD + c;
  float x[kPoolParts];
#pragma unroll
  for (int i = 0; i < kPoolParts; ++i) x[i] = SYNC ? load_agent(p + i * kD) : p[i * kD];
  return add_partials(x);
}

// The sum of the pooled queries of heads [h0, h1) without the pool workgroups' help, to qtilde; `lds`: kPoolLds + kPoolParts * kD.
__device__ __forceinline__ void pool_alone(const FrontLayer& ly, const FrontCommon& a, int h0, int h1, float* qtilde, float* lds) {
  const int tid = threadIdx.x;
  float* parts = lds + kPoolLds;
  float sum = 0.f;
  for (int h = h0; h < h1; ++h) {
    for (int half = 0; half < 2; ++half) {
      const float s = pool_partial<1>(ly, a, h, half, lds);  // (a score workgroup has its registers full of keys)
      if (tid < 2 * kD) parts[half * 2 * kD + tid] = s;
      __syncthreads();
    }
    if (tid < kD) {
      const float x[kPoolParts] = {parts[tid], parts[kD + tid], parts[2 * kD + tid], parts[3 * kD + tid]};
      sum += add_partials(x);
    }
  }
  if (tid < kD) qtilde[tid] = sum;
  __syncthreads();
}

// ---- score ---------------------------------------------------------------------------------------------
constexpr int kHeadTiles = 4;  // tiles of a score workgroup that works on one head
template <bool PER_HEAD>
constexpr int kScoreItems = PER_HEAD ? kHeadTiles : kHeadChunk;  // (head, tile) pairs whose keys a workgroup holds in registers
template <int BITS, int G, bool PER_HEAD>
constexpr int score_lds() {
  return kD + (BITS == 16 ? 0 : kScoreItems<PER_HEAD> * (kTile / G) * 2 * kD);
}
// Thread = (token tid/8 of the workgroup's THREADS/8, channels 8 * (tid%8) ..).  Everything a workgroup needs is requested up
// front (one memory round trip): the group parameters of all its items (staged in LDS, they are shared by a tile's tokens) and the
// thread's codes of all items.  An item is a head's keys of the workgroup's tile, or a tile of the workgroup's head.
// `lds`: score_lds(), and what pool_alone takes behind the first kD floats.
// A caller's plain keys may begin at any bf16: their 16-byte loads promise no more than that (same instruction, same time).
typedef __attribute__((ext_vector_type(4), aligned(2))) uint32_t KeyPiece;
template <int BITS, int G, bool PER_HEAD, int THREADS, bool SYNC>
__device__ __forceinline__ void score_part(const FrontLayer& ly, const FrontCommon& a, int list, int block, float* lds) {
  constexpr bool kQuant = BITS != 16;
  constexpr int kRows = THREADS / 8;
  static_assert(!kQuant || kRows == kTile, "the block's parameters are those of one tile");
  constexpr int kItems = kScoreItems<PER_HEAD>;
  constexpr int kGroups = kQuant ? kTile / G : 1;      // key groups inside a block of 64 positions
  constexpr int kRowDw = kD * BITS / 32;               // dwords per key row
  constexpr int kDwT = kQuant ? 1 : 4;                 // dwords per thread (2 bits: shared by two threads)
  float* qtilde = lds;
  float* prm = lds + kD;                               // [item][group][scale|zero][channel]
  __shared__ int pooled;

  const int H = a.H, tid = threadIdx.x, r = tid >> 3, c8 = tid & 7;
  const int first = (a.T_first / kRows + block * (PER_HEAD ? kItems : 1)) * kRows;  // cache position of the first row
  auto position = [&](int item) { return first + r + (PER_HEAD ? item * kRows : 0); };
  auto in_middle = [&](int pos) { return pos >= a.T_first && pos < a.T_first + a.P; };
  const uint32_t* src = reinterpret_cast<const uint32_t*>(ly.kc) + (size_t)(first + r) * kRowDw + (kQuant ? c8 * kRowDw / 8 : 4 * c8);
  const size_t head_stride = (size_t)a.head_rows * kRowDw;

  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
  // sum over the thread's 16 channels' worth of products in channel order: the odd lanes go on from their neighbours
  auto dot16 = [&](const float* qt, const float* x) {
    float d = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) d += qt[e] * x[e];
    const float even = __shfl_xor(d, 1);
    d = even;
#pragma unroll
    for (int e = 0; e < 8; ++e) d += qt[e] * x[e];
    d += __shfl_xor(d, 2);
    d += __shfl_xor(d, 4);
    return d;  // (in odd lanes)
  };
  auto store_score = [&](int pos, float s) {
    float* out = ly.scores + (size_t)list * a.stride + (pos - a.T_first);
    if (in_middle(pos) && c8 == 1) {
      if (SYNC) store_agent(out, s);
      else *out = s;
    }
  };
  // qtilde of heads [h0, h1), at a point where nobody needs the parameters behind it any more (or yet)
  auto pooled_query = [&](int h0, int h1) {
    if (tid < kD) {
      const bool done = !SYNC || __all(wait_for_pool(ly.sync + list, pools_of(a, PER_HEAD), a.polls));
      float s = 0.f;
      if (done) {
#pragma unroll 8
        for (int h = h0; h < h1; ++h) s += head_query<SYNC>(ly, h, tid);
      }
      qtilde[tid] = s;
      if (SYNC && tid == 0) pooled = done;
    }
    __syncthreads();
    if constexpr (SYNC) {
      if (!pooled) pool_alone(ly, a, h0, h1, qtilde, lds + kD);
    }
  };
  const int head_begin = PER_HEAD ? list : 0, head_end = PER_HEAD ? list + 1 : H;
  for (int h0 = head_begin; h0 < head_end; h0 += kHeadChunk) {  // (one chunk for H <= kHeadChunk)
    const int hn = PER_HEAD ? kItems : min(kHeadChunk, H - h0);  // items of this chunk
    uint32_t w[kItems][kDwT];
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      const uint32_t* p = src + (PER_HEAD ? h0 * head_stride + (size_t)(i * kRows * kRowDw) : (h0 + i) * head_stride);
      const bool valid = in_middle(position(i)) && i < hn;
      if constexpr (kQuant) {
        w[i][0] = valid ? *p : 0u;
      } else {
        const KeyPiece v = valid ? *reinterpret_cast<const KeyPiece*>(p) : KeyPiece{0, 0, 0, 0};
        w[i][0] = v.x; w[i][1] = v.y; w[i][2] = v.z; w[i][3] = v.w;
      }
    }
    constexpr int kPrmIter = kQuant ? kItems * kGroups * 2 * kD / THREADS : 1;
    float pr[kPrmIter];
    if constexpr (kQuant) {
#pragma unroll
      for (int it = 0; it < kPrmIter; ++it) {
        const int i = tid + it * THREADS;
        const int c = i % kD, sz = (i / kD) & 1, gi = (i / (2 * kD)) % kGroups, item = i / (2 * kD * kGroups);
        const int h = PER_HEAD ? h0 : h0 + item, row = first + (PER_HEAD ? item * kRows : 0);
        const bool valid = item < hn && row < a.T_first + a.P;
        pr[it] = valid ? (sz ? ly.kz : ly.ks)[((size_t)h * (a.head_rows / G) + row / G + gi) * kD + c] : 0.f;
      }
    }
    if (h0 > head_begin) __syncthreads();  // the previous chunk's parameters are no longer read
    if constexpr (PER_HEAD) pooled_query(h0, h0 + 1);
    if constexpr (kQuant) {
#pragma unroll
      for (int it = 0; it < kPrmIter; ++it) prm[tid + it * THREADS] = pr[it];
      __syncthreads();
    }
#pragma unroll
    for (int h = 0; h < kItems; ++h) {
      if (h < hn) {
        float x[8];  // the item's key row (this thread's 8 channels), dequantized view
        if constexpr (kQuant) {
          const float* ks = prm + ((h * kGroups + (r / G) % kGroups) * 2) * kD + c8 * 8;
          const float* kz = ks + kD;
          // codes to floats by bytes: one mask per 4 (2-bit: 2) codes, then one byte-to-float conversion each,
          // instead of a bit-field extract and a conversion per code
          constexpr int kPerByte = 8 / BITS;
          const uint32_t codes = BITS == 4 ? w[h][0] : w[h][0] >> (16 * (c8 & 1));
          float code[8];
#pragma unroll
          for (int sft = 0; sft < kPerByte; ++sft) {  // code e sits in byte e / kPerByte of (codes >> BITS * (e % kPerByte)) & mask
            uint32_t t = (codes >> (BITS * sft)) & (BITS == 4 ? 0x0f0f0f0fu : 0x03030303u);
            asm volatile("" : "+v"(t));  // (keeps the mask shared by the conversions below)
#pragma unroll
            for (int b = 0; b < 8 / kPerByte; ++b) code[b * kPerByte + sft] = (float)((t >> (8 * b)) & 0xffu);
          }
          // canonical view, rounded to bf16 in pairs (one packed conversion per two values)
#pragma unroll
          for (int e = 0; e < 8; e += 2) {
            typedef __attribute__((ext_vector_type(2))) float f2;
            typedef __attribute__((ext_vector_type(2))) __bf16 b2;
            const f2 v = {(code[e] - kz[e]) * ks[e], (code[e + 1] - kz[e + 1]) * ks[e + 1]};
            const uint32_t pk = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, b2));
            x[e] = bf16_lo(pk);
            x[e + 1] = bf16_hi(pk);
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            x[2 * e] = bf16_lo(w[h][e]);
            x[2 * e + 1] = bf16_hi(w[h][e]);
          }
        }
        if constexpr (PER_HEAD) {
          store_score(position(h), dot16(qtilde + c8 * 8, x));
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[e] += x[e];
        }
      }
    }
  }
  if constexpr (!PER_HEAD) {
    const float fH = (float)H;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] /= fH;
    pooled_query(0, H);
    store_score(first + r, dot16(qtilde + c8 * 8, acc));
  }
}

// ---- select --------------------------------------------------------------------------------------------

// float → unsigned key with the same order (larger score ↔ larger key); -0 and +0 stay distinct
// neighbours, which only matters for exact-zero scores.
__device__ __forceinline__ uint32_t order_key(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// inclusive sum over the lanes up to this one, by lane shifts of the ALU
__device__ __forceinline__ uint32_t wave_prefix(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true);   // row_shr:1
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true);   // row_shr:2
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true);   // row_shr:4
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true);   // row_shr:8
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
  return x;
}

constexpr int kBins = 2048, kBinsT = kBins / kThreads;  // bins, and bins per thread
constexpr int kSelWaves = kThreads / 64;
constexpr int kSelLds = kBins + 2 * kSelWaves + 4 + 2 * 64;

// One list.  A wave holds chunks of 64 consecutive scores, one per lane: chunk c belongs to wave c % kSelWaves.  KPT: scores per
// thread; lists longer than KPT * kThreads are read again in every pass, a segment of so many at a time.
template <int KPT, bool SYNC>
__device__ __forceinline__ void select_part(const SelectArgs& a, int list, uint32_t* lds) {
  static_assert(KPT * kSelWaves <= 128, "two chunks per lane in the prefix sums of the compaction");
  uint32_t* hist = lds;
  uint32_t* wave_tot = hist + kBins;           // [2][kSelWaves]: by the parity of the pass
  uint32_t* found = wave_tot + 2 * kSelWaves;  // digit, rank inside it, keys in it; keys put on the list of candidates
  uint32_t* counts = found + 4;                // per chunk of a segment: kept | equal << 16
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float* scores = a.scores + (size_t)list * a.scores_stride;
  int32_t* keep = a.keep + (size_t)list * a.keep_stride;
  const int P = a.P, k = a.k;
  constexpr int kSegment = KPT * kThreads;
  const int segments = (P + kSegment - 1) / kSegment;

  uint32_t keys[KPT];
  auto at = [&](int segment, int i) { return segment * kSegment + 64 * (i * kSelWaves + wave) + lane; };
  auto load = [&](int segment) {
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
      const int j = at(segment, i);
      keys[i] = j < P ? order_key(SYNC ? load_agent(scores + j) : scores[j]) : 0u;
    }
  };
  load(0);
  if (tid == 0) found[3] = 0;
  for (int i = tid; i < a.T_first; i += kThreads) keep[i] = i;
  for (int i = tid; i < a.T_cur; i += kThreads) keep[a.T_first + k + i] = a.T_first + P + i;

  // k-th largest key by radix select, most significant digit first
  uint32_t prefix = 0;
  uint32_t need = k;  // rank still to find inside the current prefix class (1-based from the top)
#pragma unroll
  for (int pass = 0; pass < 3; ++pass) {
    const int shift = pass == 0 ? 21 : (pass == 1 ? 10 : 0);
    const uint32_t digits = pass == 2 ? 1023u : 2047u, hi_mask = pass == 0 ? 0u : ~((digits << shift) | ((1u << shift) - 1u));
#pragma unroll
    for (int b = 0; b < kBinsT; ++b) hist[b * kThreads + tid] = 0;
    __syncthreads();
    for (int s = 0; s < segments; ++s) {
      if (segments > 1) load(s);
#pragma unroll
      for (int i = 0; i < KPT; ++i)
        if (at(s, i) < P && (keys[i] & hi_mask) == prefix) atomicAdd(&hist[(keys[i] >> shift) & digits], 1u);
    }
    __syncthreads();
    // thread t looks at the t-th kBinsT bins from the top; the wanted rank lies in bin b iff
    // (#keys in bins above b) < need <= (that + hist[b])
    uint32_t h[kBinsT], mine = 0;
#pragma unroll
    for (int b = 0; b < kBinsT; ++b) {
      h[b] = hist[kBins - 1 - (tid * kBinsT + b)];
      mine += h[b];
    }
    const uint32_t incl = wave_prefix(mine);
    uint32_t* tot = wave_tot + (pass & 1) * kSelWaves;
    if (lane == 63) tot[wave] = incl;
    __syncthreads();
    uint32_t above = incl - mine;
    for (int w = 0; w < wave; ++w) above += tot[w];
#pragma unroll
    for (int b = 0; b < kBinsT; ++b) {
      if (above < need && need <= above + h[b]) {
        found[0] = kBins - 1 - (tid * kBinsT + b);
        found[1] = need - above;
        found[2] = h[b];
      }
      above += h[b];
    }
    __syncthreads();
    prefix |= found[0] << shift;
    need = found[1];
    // What is left of the class, if it is little, is ranked by comparing all with all, instead of further passes: a pass of four
    // barriers takes about 0.65 us, a candidate 0.04.  (Every wave does it, so that nobody waits for the result.)  2722 scores
    // around zero of which 1348 are kept, 9 candidates, the kernel by itself: 7.9 and 6.6 us; around a third of their spread, 56
    // candidates, 6.7 with passes and 7.7 by comparing.
    const uint32_t left = found[2];
    if (pass < 2 && segments == 1 && left <= (pass == 0 ? 32u : 16u)) {
#pragma unroll
      for (int i = 0; i < KPT; ++i)
        if (at(0, i) < P && (keys[i] & (hi_mask | digits << shift)) == prefix) hist[atomicAdd(&found[3], 1u)] = keys[i];
      __syncthreads();
      const uint32_t mine = lane < (int)left ? hist[lane] : 0u;
      uint32_t gt = 0, ge = 0;
      for (uint32_t i = 0; i < left; ++i) {
        const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)i);
        gt += x > mine;
        ge += x >= mine;
      }
      const unsigned long long hit = __ballot(lane < (int)left && gt < need && need <= ge);
      const int at_hit = __builtin_ctzll(hit);
      prefix = (uint32_t)__builtin_amdgcn_readlane((int)mine, at_hit);
      need -= (uint32_t)__builtin_amdgcn_readlane((int)gt, at_hit);
      break;
    }
  }
  const uint32_t thr = prefix;  // key of the k-th largest score; `need` of the scores equal to it are kept (smallest positions)

  // ordered compaction
  uint32_t gt_before = 0, eq_before = 0;  // in the segments before
  for (int s = 0; s < segments; ++s) {
    if (segments > 1) {
      __syncthreads();  // (the counts of the segment before have been read)
      load(s);
    }
    unsigned long long gt[KPT], eq[KPT];
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
      const bool in = at(s, i) < P;
      gt[i] = __ballot(in && keys[i] > thr);
      eq[i] = __ballot(in && keys[i] == thr);
      if (lane == 0) counts[i * kSelWaves + wave] = (uint32_t)__popcll(gt[i]) | (uint32_t)__popcll(eq[i]) << 16;
    }
    __syncthreads();
    // (a segment holds at most 8192 scores, so that neither half overflows)
    const uint32_t c0 = 2 * lane < KPT * kSelWaves ? counts[2 * lane] : 0u, c1 = 2 * lane < KPT * kSelWaves ? counts[2 * lane + 1] : 0u;
    const uint32_t incl = wave_prefix(c0 + c1);
    const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
      const int chunk = i * kSelWaves + wave;
      uint32_t before = (uint32_t)__builtin_amdgcn_readlane((int)(incl - c0 - c1), chunk >> 1);
      if (chunk & 1) before += (uint32_t)__builtin_amdgcn_readlane((int)c0, chunk >> 1);
      const uint32_t g = gt_before + (before & 0xffffu) + (uint32_t)__popcll(gt[i] & below);
      const uint32_t e = eq_before + (before >> 16) + (uint32_t)__popcll(eq[i] & below);
      const bool take = ((gt[i] >> lane) & 1) || (((eq[i] >> lane) & 1) && e < need);
      if (take) keep[a.T_first + g + min(e, need)] = a.T_first + at(s, i);
    }
    const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    gt_before += all & 0xffffu;
    eq_before += all >> 16;
  }
}

// ---- kernels -------------------------------------------------------------------------------------------
constexpr int max_of(int a, int b) { return a > b ? a : b; }

// One layer: 2 H pool workgroups, then a.blocks score workgroups per list.
template <int BITS, int G, bool PER_HEAD, int KPT>
__global__ __launch_bounds__(kThreads) void front_kernel(const FrontArgsT<1> args) {
  constexpr int kLds = max_of(max_of(kD + kPoolLds + kPoolParts * kD, score_lds<BITS, G, PER_HEAD>()), kSelLds);
  __shared__ __attribute__((aligned(16))) float lds[kLds];
  __shared__ int last;
  static_assert(sizeof(lds) > kLdsBesideAttention, "it stays off the compute units of attention's 32-row shapes");
#if defined(__HIP_DEVICE_COMPILE__)
  {
    // every field of the arguments that is read further down would wait for its own line of them: all lines at once
    const uint32_t* w = static_cast<const uint32_t*>(__builtin_amdgcn_kernarg_segment_ptr());
    static_assert(sizeof(args) > 128 && sizeof(args) <= 4 * 64, "four loads reach every line");
    const uint32_t w0 = w[0], w1 = w[16], w2 = w[32], w3 = w[sizeof(args) / 4 - 1];
    asm volatile("" ::"s"(w0), "s"(w1), "s"(w2), "s"(w3));
  }
#endif
  const FrontCommon& a = args.c;
  const FrontLayer& ly = args.layer[0];
  const int b = blockIdx.x;
  if (b < 2 * a.H) {
    pool_part<true>(ly, a, b >> 1, b & 1, lds);
    return;
  }
  const int list = PER_HEAD ? (b - 2 * a.H) / a.blocks : 0;
  score_part<BITS, G, PER_HEAD, kThreads, true>(ly, a, list, b - 2 * a.H - list * a.blocks, lds);
  const uint64_t before = arrive(ly.sync + list, kScoreArrived, all_of(a, PER_HEAD));
  if (threadIdx.x == 0) last = (int)(before >> 32) == a.blocks - 1;
  __syncthreads();
  if (last) {
    const SelectArgs s{ly.scores, ly.keep, a.stride, a.stride, a.P, a.k, a.T_first, a.T_cur};
    select_part<KPT, true>(s, list, reinterpret_cast<uint32_t*>(lds));
  }
}

// The parts by themselves, for many layers at a time and for plain bf16 keys.
template <int LAYERS>
__global__ __launch_bounds__(kThreads) void pool_kernel(const FrontArgsT<LAYERS> args) {
  __shared__ float lds[kPoolLds];
  pool_part<false>(args.layer[blockIdx.y], args.c, blockIdx.x >> 1, blockIdx.x & 1, lds);
}
template <int BITS, int G, bool PER_HEAD, int THREADS, int LAYERS>
__global__ __launch_bounds__(THREADS) void score_kernel(const FrontArgsT<LAYERS> args) {
  __shared__ __attribute__((aligned(16))) float lds[score_lds<BITS, G, PER_HEAD>()];
  const int list = PER_HEAD ? blockIdx.x / args.c.blocks : 0;
  score_part<BITS, G, PER_HEAD, THREADS, false>(args.layer[blockIdx.y], args.c, list, blockIdx.x - list * args.c.blocks, lds);
}
template <int KPT>
__global__ __launch_bounds__(kThreads) void select_kernel(const SelectArgs a) {
  __shared__ uint32_t lds[kSelLds];
  select_part<KPT, false>(a, blockIdx.x, lds);
}

// blocks of `rows` positions that the middle touches
static int score_blocks(const FrontCommon& c, int rows) { return (c.T_first + c.P - 1) / rows - c.T_first / rows + 1; }

constexpr int kPlainThreads = 128;  // 16 positions: a list of 2722 is then spread over 170 workgroups (pool and score of
// 16 heads: 28.6 us with 43, 10.0 with 170)
hipError_t launch_score(const FrontArgs& a, hipStream_t stream) {
  FrontArgsT<1> one{a.c, {a.layer[0]}};
  one.c.blocks = score_blocks(a.c, kPlainThreads / 8);
  hipLaunchKernelGGL(pool_kernel<1>, dim3(2 * a.c.H), dim3(kThreads), 0, stream, one);
  hipLaunchKernelGGL((score_kernel<16, 64, false, kPlainThreads, 1>), dim3(one.c.blocks), dim3(kPlainThreads), 0, stream, one);
  return hipGetLastError();
}

// Scores per thread of a select workgroup: 8 while they do (4096 scores), since all of them are looked at in every pass.
static bool few_scores(int P) { return P <= 8 * kThreads; }

hipError_t launch_select(const SelectArgs& a, int n_lists, hipStream_t stream) {
  if (few_scores(a.P)) hipLaunchKernelGGL(select_kernel<8>, dim3(n_lists), dim3(kThreads), 0, stream, a);
  else hipLaunchKernelGGL(select_kernel<16>, dim3(n_lists), dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

template <int BITS, int G, bool PER_HEAD>
static hipError_t launch_front_t(FrontArgs& a, hipStream_t stream) {
  FrontCommon& c = a.c;
  const int tiles = score_blocks(c, kTile), lists = PER_HEAD ? c.H : 1;
  c.blocks = PER_HEAD ? (tiles + kHeadTiles - 1) / kHeadTiles : tiles;
  if (c.n_layers == 1) {
    const dim3 grid(2 * c.H + c.blocks * lists);
    const FrontArgsT<1> one{c, {a.layer[0]}};
    if (few_scores(c.P)) hipLaunchKernelGGL((front_kernel<BITS, G, PER_HEAD, 8>), grid, dim3(kThreads), 0, stream, one);
    else hipLaunchKernelGGL((front_kernel<BITS, G, PER_HEAD, 16>), grid, dim3(kThreads), 0, stream, one);
    return hipGetLastError();
  }
  // Many layers: their parts fill the chip by themselves, and workgroups that wait only hold places that others could use
  // (24 layers of the sizes above: 104 us as one launch, 46 as three).
  hipLaunchKernelGGL(pool_kernel<kMaxBatch>, dim3(2 * c.H, c.n_layers), dim3(kThreads), 0, stream, a);
  hipLaunchKernelGGL((score_kernel<BITS, G, PER_HEAD, kThreads, kMaxBatch>), dim3(c.blocks * lists, c.n_layers), dim3(kThreads), 0, stream, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // (the lists of consecutive layers follow each other)
  return launch_select(SelectArgs{a.layer[0].scores, a.layer[0].keep, c.stride, c.stride, c.P, c.k, c.T_first, c.T_cur}, c.n_layers * lists, stream);
}

hipError_t launch_front(FrontArgs& a, int bits, int G, hipStream_t stream) {
  auto launch = [&](auto b, auto g) {
    constexpr int BITS = decltype(b)::value, GROUP = decltype(g)::value;
    return a.c.per_head ? launch_front_t<BITS, GROUP, true>(a, stream) : launch_front_t<BITS, GROUP, false>(a, stream);
  };
  using std::integral_constant;
  if (bits == 16) return launch(integral_constant<int, 16>{}, integral_constant<int, 64>{});
  if (bits == 4 && G == 64) return launch(integral_constant<int, 4>{}, integral_constant<int, 64>{});
  if (bits == 4 && G == 32) return launch(integral_constant<int, 4>{}, integral_constant<int, 32>{});
  if (bits == 2 && G == 64) return launch(integral_constant<int, 2>{}, integral_constant<int, 64>{});
  if (bits == 2 && G == 32) return launch(integral_constant<int, 2>{}, integral_constant<int, 32>{});
  return hipErrorInvalidValue;
}

// keep = [0, T_first) ∪ (middle, if kept) ∪ current
__global__ __launch_bounds__(256) void fill_keep_kernel(int32_t* keep, int T_first, int P, int T_cur, int keep_middle) {
  const int total = T_first + (keep_middle ? P : 0) + T_cur;
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < total) keep[i] = (keep_middle || i < T_first) ? i : i + P;
}

hipError_t launch_fill_keep(int32_t* keep, int T_first, int P, int T_cur, bool keep_middle, hipStream_t stream) {
  const int total = T_first + (keep_middle ? P : 0) + T_cur;
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_keep_kernel, dim3((total + 255) / 256), dim3(256), 0, stream, keep, T_first, P, T_cur, keep_middle ? 1 : 0);
  return hipGetLastError();
}

}  // namespace xsv
