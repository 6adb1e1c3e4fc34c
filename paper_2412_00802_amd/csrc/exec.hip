// Kernels and the executor of libhthedl.
//
// Work decomposition (all bit rows are uint64 words, 64 individuals each):
//   k_threshold  numeric restriction (Algorithms 9/10): one lane per individual,
//                one wave ballot per output word.
//   k_region     n-ary and/or/not over bit rows (Algorithms 1/2): one lane per
//                word, the region's postfix bytecode interpreted with a value
//                stack in LDS; coverage (Algorithm 15) fused: popcount against
//                the example rows, wave reduction, one atomic per wave.
//   k_role       role restrictions (Algorithms 3-8) over a CSR direction: one
//                wave per 64 consecutive subjects; the wave walks the subjects'
//                concatenated assertion range in chunks of 64 (coalesced target
//                loads, eight chunks' loads in flight), tests each object against
//                the child row, and each subject lane counts its own assertions
//                in a chunk as popcount(ballot & its lane range).  Skewed degrees
//                are balanced inside the wave by construction; rows stop
//                contributing once their count decides the predicate, and the
//                walk jumps past chunks that hold only decided rows.  Rows above
//                the heavy-row threshold are counted on many blocks instead
//                (k_role_heavy).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <memory>
#include <set>
#include <utility>
#include <vector>

#include "kb_handle.h"
#include "plan.h"

namespace hth {

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

// ---------------------------------------------------------------------------
// numeric thresholds
// ---------------------------------------------------------------------------
// All thresholds requested on one property in one pass over its column: one
// lane per individual over 8 consecutive words (values loaded once, kept in
// registers), one wave ballot per threshold and word; lanes 0..7 then store
// the 8 words of a threshold's row together (a full 64-byte line).  Bound by
// the vector unit: a compare and two lane writes per threshold and word (the
// comparison is chosen once per threshold, and an individual past the end is a
// missing value, so that nothing else is done per word).  VIEW: the column is
// read at the examples (list), 64 of them a word.
// 576 thresholds over 32M individuals 2.1 ms, where a select on the
// comparison and on the lane per word took 7.6.
__device__ __forceinline__ void put_lane(uint32_t& lo, uint32_t& hi, uint64_t m, int lane) {
  // (a vector instruction may read a scalar that another one wrote two wait
  // states later)
  asm("s_nop 1\n\tv_writelane_b32 %0, %2, %4\n\tv_writelane_b32 %1, %3, %4"
      : "+v"(lo), "+v"(hi)
      : "s"((uint32_t)m), "s"((uint32_t)(m >> 32)), "n"(lane));
}
template <bool VIEW>
__global__ void __launch_bounds__(256)
k_threshold(DevKB kb, const ThrGroup* __restrict__ groups, const ThrTask* __restrict__ tasks, uint32_t bpt,
            const uint32_t* __restrict__ list) {
  uint32_t gi = blockIdx.x / bpt, b = blockIdx.x % bpt;
  if (VIEW) {
    const ViewBlock v = view_block(blockIdx.x, gridDim.x / bpt, bpt, (kb.view[1] + 31) / 32);
    gi = v.item, b = v.b;
  }
  const ThrGroup G = groups[gi];
  const float* col = kb.data + (size_t)G.prop * kb.N;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint32_t N = VIEW ? kb.view[0] : kb.N, W = VIEW ? kb.view[1] : kb.W;
  const uint32_t n_blk = (W + 7) / 8;
  for (uint32_t blk = b * 4 + wv; blk < n_blk; blk += bpt * 4) {
    const uint32_t w0 = blk * 8;
    float f[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t x = (w0 + j) * 64 + lane;
      const bool in = w0 + j < W && x < N;
      const uint32_t at = in ? x : 0u;
      const float v = col[VIEW ? list[at] : at];
      f[j] = in ? v : __builtin_nanf("");       // NaN (no value) compares false
    }
    for (uint32_t i = 0; i < G.n; ++i) {
      const ThrTask T = tasks[G.first + i];
      uint32_t lo = 0, hi = 0;
      auto words = [&](auto pass) {
        put_lane(lo, hi, __ballot(pass(f[0])), 0);
        put_lane(lo, hi, __ballot(pass(f[1])), 1);
        put_lane(lo, hi, __ballot(pass(f[2])), 2);
        put_lane(lo, hi, __ballot(pass(f[3])), 3);
        put_lane(lo, hi, __ballot(pass(f[4])), 4);
        put_lane(lo, hi, __ballot(pass(f[5])), 5);
        put_lane(lo, hi, __ballot(pass(f[6])), 6);
        put_lane(lo, hi, __ballot(pass(f[7])), 7);
      };
      if (T.cmp == 0) words([&](float v) { return v >= T.t; });
      else if (T.cmp == 1) words([&](float v) { return v <= T.t; });
      else words([&](float v) { return v == T.t; });
      if (lane < 8 && w0 + lane < W) out_ptr(kb, T.out_row)[w0 + lane] = ((uint64_t)hi << 32) | lo;
    }
  }
}

// The ballots of a round of chunks (64 values each), held across the wave:
// lane c keeps chunk c's ballot and the number of passing values before it.  A
// subject's count in the round is the difference of two prefix counts, each
// one lookup by lane: work per subject and round, where taking every chunk's
// part of the subject's range is work per subject and chunk.
template <class F, int... C>
__device__ __forceinline__ void unrolled(F&& f, std::integer_sequence<int, C...>) {
  (f(std::integral_constant<int, C>()), ...);
}
template <int N, class F>
__device__ __forceinline__ void unrolled(F&& f) {   // f of each constant 0 .. N - 1
  unrolled(f, std::make_integer_sequence<int, N>());
}
struct ChunkSums {
  uint32_t lo = 0, hi = 0, before = 0, total = 0;   // total: so far, the same on every lane
  template <int C>
  __device__ __forceinline__ void put(uint64_t m) {   // (the wait states: see put_lane)
    asm("s_nop 1\n\tv_writelane_b32 %0, %3, %6\n\tv_writelane_b32 %1, %4, %6\n\tv_writelane_b32 %2, %5, %6"
        : "+v"(lo), "+v"(hi), "+v"(before)
        : "s"(__builtin_amdgcn_readfirstlane((uint32_t)m)), "s"(__builtin_amdgcn_readfirstlane((uint32_t)(m >> 32))),
          "s"(__builtin_amdgcn_readfirstlane(total)), "n"(C));
    total += (uint32_t)__popcll(m);
  }
  // passing values among the round's first p (p <= span, the round's values)
  __device__ __forceinline__ uint32_t prefix(uint32_t p) const {
    const int c = (int)(p >> 6);
    const uint64_t m = (uint64_t)(uint32_t)__shfl((int)hi, c, 64) << 32 | (uint32_t)__shfl((int)lo, c, 64);
    return (uint32_t)__shfl((int)before, c, 64) + (uint32_t)__popcll(m & ((1ull << (p & 63)) - 1ull));
  }
  // those of values [r0, r1) (absolute; the round holds [i0, i0 + span))
  template <int CHUNKS>
  __device__ __forceinline__ uint32_t count(uint32_t r0, uint32_t r1, uint32_t i0) {
    constexpr uint32_t span = CHUNKS * 64;
    put<CHUNKS>(0);
    const uint32_t a = r0 > i0 ? min(r0 - i0, span) : 0u, z = r1 > i0 ? min(r1 - i0, span) : 0u;
    const uint32_t pa = prefix(a), pz = prefix(z);
    return z > a ? pz - pa : 0u;
  }
};

// ---------------------------------------------------------------------------
// multi-valued numeric concrete roles (Algorithms 9/10)
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool num_pass(float v, uint32_t cmp, float t) {
  return cmp == 0 ? v >= t : cmp == 1 ? v <= t : v == t;
}

// Value roles (numeric and string concrete roles): one wave per 64 consecutive
// subjects, as in the role pass.  The wave walks the subjects' concatenated
// values in chunks of 64 (eight chunks' loads in flight), a subject's passing
// values are the difference of two prefix counts (ChunkSums), and the walk
// stops once every subject with values left has found one.  Up to value_tasks()
// tasks of one role share a walk, and a round has as many chunks as the values
// left need (2, 4 or 8).  Rows above the heavy-row threshold are left to
// value_heavy (their bits here are 0).  About 60 restrictions on 4 roles over
// 1M individuals: numeric 173 us, string 167 (348 and 334 with 8 chunks in
// every round, 437 and 372 with a walk for each task).
constexpr int kNumChunks = 8;
constexpr uint32_t kValPerPass = 16;
// off: the role's 32-bit offsets relative to vals, its first value.
template <typename V, class Pass, class Out>
__device__ __forceinline__ void value_walk(const DevKB& kb, const uint32_t* __restrict__ off,
                                           const V* __restrict__ vals, uint32_t n, Pass pass, Out out, uint32_t b,
                                           uint32_t bpt) {
  const int lane = threadIdx.x & 63;
  for (uint32_t w = b * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); w < kb.W; w += bpt * 4) {
    const uint32_t x = w * 64 + lane;
    const bool in = x < kb.N;
    const uint32_t olo = off[in ? x : kb.N];
    uint32_t ohi = in ? off[x + 1] : olo;
    const bool heavy = ohi - olo > kb.heavy_min;
    if (heavy) ohi = olo;
    const uint32_t ee = (uint32_t)__builtin_amdgcn_readlane((int)ohi, 63);
    uint32_t i0 = (uint32_t)__builtin_amdgcn_readlane((int)olo, 0);
    uint32_t hits = 0;           // bit j: task j has a passing value
    const uint32_t all = (1u << n) - 1u;
    // a round of `chunks` chunks from i0 on
    auto round = [&](auto chunks) {
      constexpr int C = chunks.value;
      V v[C];
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const uint64_t e = (uint64_t)i0 + 64 * c + lane;
        v[c] = vals[e < ee ? (uint32_t)e : i0];
      }
      for (uint32_t j = 0; j < n; ++j) {
        const auto test = pass(j);
        ChunkSums sums;
        unrolled<C>([&](auto c) {   // (values past ee: past every subject's range)
          sums.template put<c.value>(__ballot(test(v[c.value])));
        });
        hits |= (uint32_t)(sums.template count<C>(olo, ohi, i0) != 0) << j;
      }
    };
    while (i0 < ee) {
      if (ee - i0 <= 128) round(std::integral_constant<int, 2>());
      else if (ee - i0 <= 256) round(std::integral_constant<int, 4>());
      else round(std::integral_constant<int, kNumChunks>());
      const uint64_t step = 64 * kNumChunks;
      const uint64_t pend = __ballot(in && hits != all && ohi > i0 + step);
      if (!pend) break;
      const int l = __ffsll((unsigned long long)pend) - 1;
      const uint32_t nxt = (uint32_t)__builtin_amdgcn_readlane((int)olo, l);
      i0 = (uint32_t)max((uint64_t)i0 + step, (uint64_t)nxt);
    }
    for (uint32_t j = 0; j < n; ++j) {
      const uint64_t word = __ballot(in && !heavy && ((hits >> j) & 1u));
      if (lane == 0) out(j)[w] = word;
    }
  }
}

// One chunk of kHeavyChunk values of one heavy row per block: a passing value
// sets the row's bit (after the walk wrote the word; an existential result
// only ever gains bits, so blocks need no ordering among themselves).  Chunk
// blocks that find the bit already set skip the atomic.
template <typename V, class Pass>
__device__ __forceinline__ void value_heavy(const DevKB& kb, const uint32_t* __restrict__ off,
                                            const V* __restrict__ vals, Pass pass, uint64_t* __restrict__ out,
                                            uint32_t x, uint32_t k) {
  __shared__ uint32_t s_any[4];
  const uint32_t e0 = off[x] + k * kHeavyChunk;
  const uint32_t e1 = min(off[x + 1], e0 + kHeavyChunk);
  bool any = false;
#pragma unroll
  for (uint32_t j = 0; j < kHeavyChunk / 256; ++j) {
    const uint32_t e = e0 + j * 256 + threadIdx.x;
    if (e < e1) any |= pass(vals[e]);
  }
  const uint64_t m = __ballot(any);
  if ((threadIdx.x & 63) == 0) s_any[threadIdx.x >> 6] = m != 0;
  __syncthreads();
  if (threadIdx.x == 0 && (s_any[0] | s_any[1] | s_any[2] | s_any[3])) {
    unsigned long long* word = reinterpret_cast<unsigned long long*>(out) + (x >> 6);
    const unsigned long long bit = 1ull << (x & 63);
    if (!(__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit)) atomicOr(word, bit);
  }
}

// the task of heavy block b: the last task whose first block is <= b
template <class Task>
__device__ __forceinline__ uint32_t value_task(const Task* __restrict__ tasks, uint32_t n, uint32_t b) {
  uint32_t lo = 0, hi = n;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (tasks[mid].h_first <= b) lo = mid;
    else hi = mid;
  }
  return lo;
}

__global__ void __launch_bounds__(256)
k_numrole(DevKB kb, const ThrGroup* __restrict__ groups, const NumTask* __restrict__ tasks, uint32_t bpt) {
  const ThrGroup G = groups[blockIdx.x / bpt];
  const NumTask T0 = tasks[G.first];
  value_walk<float>(
      kb, kb.num_roff + (size_t)G.prop * (kb.N + 1), kb.num_val + ((uint64_t)T0.base_hi << 32 | T0.base_lo), G.n,
      [&](uint32_t j) {
        const uint32_t cmp = tasks[G.first + j].cmp;
        const float t = tasks[G.first + j].t;
        return [=](float v) { return num_pass(v, cmp, t); };
      },
      [&](uint32_t j) { return out_ptr(kb, tasks[G.first + j].out_row); }, blockIdx.x % bpt, bpt);
}

__global__ void __launch_bounds__(256)
k_numrole_heavy(DevKB kb, const NumTask* __restrict__ tasks, uint32_t n_tasks, uint32_t b0) {
  const uint32_t b = b0 + blockIdx.x;
  const NumTask T = tasks[value_task(tasks, n_tasks, b)];
  const HeavyChunk c = kb.num_heavy_chunks[T.hc0 + (b - T.h_first)];
  const float* vals = kb.num_val + ((uint64_t)T.base_hi << 32 | T.base_lo);
  value_heavy<float>(kb, kb.num_roff + (size_t)T.role * (kb.N + 1), vals,
                     [&](float v) { return num_pass(v, T.cmp, T.t); }, out_ptr(kb, T.out_row),
                     kb.num_heavy_rows[c.hrow], c.k);
}

// CONTAIN, first step: for every dictionary string, whether it holds the
// task's pattern (one lane per string, a plain scan of the string; the empty
// pattern is in every string).  A wave ballot writes one word of the task's
// id set per 64 strings.  The per-assertion test then reads one bit.
__global__ void __launch_bounds__(256)
k_contains(DevKB kb, const StrTask* __restrict__ tasks, uint32_t tiles) {
  const StrTask T = tasks[blockIdx.x / tiles];
  const uint32_t s = (blockIdx.x % tiles) * 256 + threadIdx.x;
  const int64_t p0 = kb.pat_off[T.q], pl = kb.pat_off[T.q + 1] - p0;
  const uint8_t* pat = kb.pat_chars + p0;
  bool hit = false;
  if (s < kb.n_strings) {
    const int64_t s0 = kb.dict_off[s], sl = kb.dict_off[s + 1] - s0;
    const uint8_t* str = kb.dict_chars + s0;
    for (int64_t i = 0; i + pl <= sl && !hit; ++i) {
      int64_t j = 0;
      while (j < pl && str[i + j] == pat[j]) ++j;
      hit = j == pl;
    }
  }
  const uint64_t m = __ballot(hit);
  const uint32_t w = s >> 6;
  if ((threadIdx.x & 63) == 0 && (uint64_t)w * 64 < kb.n_strings) kb.idsets[T.set_word + w] = m;
}

__global__ void __launch_bounds__(256)
k_strrole(DevKB kb, const ThrGroup* __restrict__ groups, const StrTask* __restrict__ tasks, uint32_t bpt) {
  const ThrGroup G = groups[blockIdx.x / bpt];
  const StrTask T0 = tasks[G.first];
  value_walk<int32_t>(
      kb, kb.str_roff + (size_t)G.prop * (kb.N + 1), kb.str_ids + ((uint64_t)T0.base_hi << 32 | T0.base_lo), G.n,
      [&](uint32_t j) {
        const StrTask T = tasks[G.first + j];
        const uint64_t* set = kb.idsets + T.set_word;
        return [=](int32_t id) {
          return T.kind == 0 ? (uint32_t)id == T.q : (bool)((set[(uint32_t)id >> 6] >> (id & 63)) & 1);
        };
      },
      [&](uint32_t j) { return out_ptr(kb, tasks[G.first + j].out_row); }, blockIdx.x % bpt, bpt);
}

__global__ void __launch_bounds__(256)
k_strrole_heavy(DevKB kb, const StrTask* __restrict__ tasks, uint32_t n_tasks, uint32_t b0) {
  const uint32_t b = b0 + blockIdx.x;
  const StrTask T = tasks[value_task(tasks, n_tasks, b)];
  const HeavyChunk c = kb.str_heavy_chunks[T.hc0 + (b - T.h_first)];
  const uint32_t* off = kb.str_roff + (size_t)T.role * (kb.N + 1);
  const int32_t* ids = kb.str_ids + ((uint64_t)T.base_hi << 32 | T.base_lo);
  const uint32_t x = kb.str_heavy_rows[c.hrow];
  uint64_t* out = out_ptr(kb, T.out_row);
  if (T.kind == 0) {
    value_heavy<int32_t>(kb, off, ids, [&](int32_t id) { return (uint32_t)id == T.q; }, out, x, c.k);
  } else {
    const uint64_t* set = kb.idsets + T.set_word;
    value_heavy<int32_t>(kb, off, ids, [&](int32_t id) { return (set[(uint32_t)id >> 6] >> (id & 63)) & 1; },
                         out, x, c.k);
  }
}

// Restrictions that only coverage reads, at the examples alone: one wave per
// kExWords words of the example rows.  Their set bits are listed in LDS; a
// lane takes one example after another and walks its row, a wave together
// those longer than kExLane.  test(value): the value counts; the result, lo <=
// count <= hi, decided at sat.  Every word of the output row is written, zeros
// outside the examples.  Bound by the latency of three dependent loads (the
// row's offsets, its values, what they select), so that a task over 1M
// individuals costs 11 us with 62,000 examples (16 with 32 words a wave), where
// every individual's row takes 18.
constexpr uint32_t kExWords = 8, kExLane = 32;
template <typename V, class Test>
__device__ __forceinline__ void example_walk(const DevKB& kb, const uint32_t* __restrict__ off,
                                             const V* __restrict__ vals, Test test, uint32_t lo, uint32_t hi,
                                             uint32_t sat, uint64_t* __restrict__ out, uint32_t tile) {
  __shared__ uint16_t s_list[kExWords * 64];
  __shared__ uint32_t s_out[2 * kExWords];
  const uint32_t lane = threadIdx.x, half = tile * 2 * kExWords + lane;   // a lane per 32 individuals
  const bool mine = lane < 2 * kExWords && half < 2 * kb.W;
  uint32_t m = 0;
  if (mine)
    m = reinterpret_cast<const uint32_t*>(kb.pos)[half] | reinterpret_cast<const uint32_t*>(kb.neg)[half];
  uint32_t inc = (uint32_t)__popc(m);
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t u = (uint32_t)__shfl_up((int)inc, d, 64);
    if (lane >= (uint32_t)d) inc += u;
  }
  const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
  if (lane < 2 * kExWords) s_out[lane] = 0;
  for (uint32_t at = inc - (uint32_t)__popc(m); m; m &= m - 1) s_list[at++] = (uint16_t)(lane * 32 + __builtin_ctz(m));
  __syncthreads();
  for (uint32_t i0 = 0; i0 < n; i0 += 64) {
    const uint32_t s = i0 + lane < n ? s_list[i0 + lane] : 0u, x = tile * kExWords * 64 + s;
    const bool in = i0 + lane < n && x < kb.N;
    const uint32_t r0 = in ? off[x] : 0u, r1 = in ? off[x + 1] : 0u;
    uint32_t cnt = 0;
    const bool wide = r1 - r0 > kExLane;
    if (!wide)
      for (uint32_t e = r0; e < r1 && cnt < sat; e += 8) {
        V v[8];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) v[u] = vals[min(e + u, r1 - 1)];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) cnt += (uint32_t)(test(v[u]) && e + u < r1);
      }
    for (uint64_t w = __ballot(wide); w; w &= w - 1) {
      const int l = __builtin_ctzll(w);
      const uint32_t e1 = (uint32_t)__builtin_amdgcn_readlane((int)r1, l);
      uint32_t c = 0;
      for (uint32_t e0 = (uint32_t)__builtin_amdgcn_readlane((int)r0, l); e0 < e1 && c < sat; e0 += 512) {
        V v[8];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) v[u] = vals[min(e0 + u * 64 + lane, e1 - 1)];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) c += (uint32_t)__popcll(__ballot(e0 + u * 64 + lane < e1 && test(v[u])));
      }
      if (lane == (uint32_t)l) cnt = c;
    }
    if (in && cnt >= lo && cnt <= hi) atomicOr(s_out + (s >> 5), 1u << (s & 31));
  }
  __syncthreads();
  if (mine) reinterpret_cast<uint32_t*>(out)[half] = s_out[lane];
}

__global__ void __launch_bounds__(64)
k_numrole_ex(DevKB kb, const NumTask* __restrict__ tasks, uint32_t tiles) {
  const NumTask T = tasks[blockIdx.x / tiles];
  example_walk<float>(kb, kb.num_roff + (size_t)T.role * (kb.N + 1),
                      kb.num_val + ((uint64_t)T.base_hi << 32 | T.base_lo),
                      [&](float v) { return num_pass(v, T.cmp, T.t); }, 1, kNone, 1, out_ptr(kb, T.out_row),
                      blockIdx.x % tiles);
}

__global__ void __launch_bounds__(64)
k_strrole_ex(DevKB kb, const StrTask* __restrict__ tasks, uint32_t tiles) {
  const StrTask T = tasks[blockIdx.x / tiles];
  const uint64_t* set = kb.idsets + T.set_word;
  example_walk<int32_t>(kb, kb.str_roff + (size_t)T.role * (kb.N + 1),
                        kb.str_ids + ((uint64_t)T.base_hi << 32 | T.base_lo),
                        [&](int32_t id) {
                          return T.kind == 0 ? (uint32_t)id == T.q : (bool)((set[(uint32_t)id >> 6] >> (id & 63)) & 1);
                        },
                        1, kNone, 1, out_ptr(kb, T.out_row), blockIdx.x % tiles);
}

__global__ void __launch_bounds__(64)
k_role_ex(DevKB kb, const RoleTask* __restrict__ tasks, uint32_t tiles) {
  const RoleTask T = tasks[blockIdx.x / tiles];
  const uint32_t* child = reinterpret_cast<const uint32_t*>(row_ptr(kb, T.child_row));
  example_walk<int32_t>(kb, (T.inv ? kb.inv_off : kb.fwd_off) + (size_t)T.role * (kb.N + 1),
                        (T.inv ? kb.inv_tg : kb.fwd_tg) + kb.role_base[T.role],
                        [&](int32_t y) { return (((child[(uint32_t)y >> 5] >> (y & 31)) & 1u) ^ T.neg) != 0; },
                        T.lo, T.hi, T.sat, out_ptr(kb, T.out_row), blockIdx.x % tiles);
}

// ---------------------------------------------------------------------------
// boolean regions (+ coverage)
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kRegionThreads)
k_region(DevKB kb, const RegionTask* __restrict__ tasks, const uint32_t* __restrict__ code,
         uint32_t n_tasks, uint32_t tiles) {
  __shared__ uint64_t stk[kStackDepth][kRegionThreads];
  const uint32_t task = blockIdx.x % n_tasks;
  const RegionTask T = tasks[task];
  if (T.out_row == kNone && T.cover == kNone) return;   // a root whose coverage a shared pass adds
  const uint32_t tid = threadIdx.x;
  const uint32_t W = span_w(kb), S = kb.view ? W : kb.S;
  const uint64_t tail = span_tail(kb);
  for (uint32_t tile = blockIdx.x / n_tasks; tile * kRegionThreads < S; tile += tiles) {
    const uint32_t w = tile * kRegionThreads + tid;
    const bool live = w < W;
    uint64_t top = 0;
    int sp = 0;
    for (uint32_t pc = 0; pc < T.code_len; ++pc) {
      const uint32_t ins = code[T.code_off + pc];
      const uint32_t op = ins & 15u, arg = ins >> 5;
      const uint64_t negm = (ins & 16u) ? ~0ull : 0ull;
      switch (op) {
        case RP_LEAF:
        case RP_TOP:
        case RP_BOT: {
          uint64_t v;
          if (op == RP_LEAF) v = live ? (row_ptr(kb, arg)[w] ^ negm) : 0ull;
          else v = op == RP_TOP ? ~0ull : 0ull;
          if (pc) stk[sp++][tid] = top;
          top = v;
          break;
        }
        case RP_NOT: top = ~top; break;
        case RP_AND: top &= stk[--sp][tid]; break;
        default: top |= stk[--sp][tid]; break;
      }
    }
    if (!live) top = 0;
    else if (w == W - 1) top &= tail;
    if (T.out_row != kNone && w < kb.S) {
      // kInstances: the caller's rows, one per covered hypothesis
      uint64_t* o = T.out_row == kInstances ? kb.instances + (size_t)T.cover * kb.S : out_ptr(kb, T.out_row);
      o[w] = top;
    }
    if (T.cover != kNone) {
      uint32_t p = live ? (uint32_t)__popcll(top & kb.pos[w]) : 0u;
      uint32_t q = live ? (uint32_t)__popcll(top & kb.neg[w]) : 0u;
      p = wave_sum(p);
      q = wave_sum(q);
      if ((tid & 63) == 0 && (p | q)) {
        if (p) atomicAdd(kb.counts + 2 * T.cover, p);
        if (q) atomicAdd(kb.counts + 2 * T.cover + 1, q);
      }
    }
  }
}

// The same regions with the value stack in registers (a shift register of
// depth D, enough for most programs) and R words per lane, so that no LDS
// limits occupancy.  A block takes one task and a run of `tpb` consecutive
// tiles (256 R words each) and walks them in order: while it evaluates one
// tile, the words of the program's first kRegLeaves leaves and the example
// words of the next tile are already in flight.  The program runs leaf by
// leaf from registers; leaves beyond the first kRegLeaves are loaded where
// they occur.  An operand directly followed by AND or OR is combined with
// the top at once, so flat conjunctions and disjunctions never move the stack.  Lane t handles words tile*256R + R*t + r (consecutive: 16-byte loads).
// Coverage is summed over the block's tiles and added with one atomic pair.
// A root whose coverage a shared pass adds has an empty task: its blocks
// leave at once.
constexpr int kRegDepth = 6;     // D: most stack entries a program may need
constexpr int kRegLeaves = 2;    // leaves whose words are loaded ahead
template <int D, int R>
__global__ void __launch_bounds__(256)
k_region_reg(DevKB kb, const RegionTask* __restrict__ tasks, const uint32_t* __restrict__ code,
             uint32_t n_tasks, uint32_t tiles, uint32_t tpb, uint32_t runs) {
  __shared__ uint32_t s_pq[2][4];
  const uint32_t run = blockIdx.x / n_tasks, task = blockIdx.x % n_tasks;
  const RegionTask T = tasks[task];
  if (T.out_row == kNone && T.cover == kNone) return;
  const uint32_t W = span_w(kb);
  const uint64_t tail = span_tail(kb);
  if (kb.view) {                // the launch's runs share the words there are
    tiles = (W + 256 * R - 1) / (256 * R);
    tpb = (tiles + runs - 1) / runs;
    if (run * tpb >= tiles) return;
  }
  const uint32_t tid = threadIdx.x;
  const uint32_t* prog = code + T.code_off;
  const uint32_t len = T.code_len;
  // the first kRegLeaves leaves' rows (a program with fewer reads the example
  // row in their place and never uses it)
  const uint64_t* lrow[kRegLeaves];
  {
    uint32_t pc = 0;
#pragma unroll
    for (int j = 0; j < kRegLeaves; ++j) {
      while (pc < len && (prog[pc] & 15u) != RP_LEAF) ++pc;
      lrow[j] = pc < len ? row_ptr(kb, prog[pc] >> 5) : kb.pos;
      if (pc < len) ++pc;
    }
  }
  const bool cover = T.cover != kNone;
  uint64_t* out = T.out_row == kNone ? nullptr
                  : T.out_row == kInstances ? kb.instances + (size_t)T.cover * kb.S
                                            : out_ptr(kb, T.out_row);
  // loads of one tile: a lane's R consecutive words, at an index clamped into
  // the row (rows hold S words, S a multiple of 8; words past W are masked
  // later), R-word vector loads with no branch around them
  auto load_words = [&](const uint64_t* row, uint32_t wc, uint64_t (&v)[R]) {
    if constexpr (R == 1) {
      v[0] = row[wc];
    } else {
#pragma unroll
      for (int r = 0; r < R; r += 2) {
        const ulonglong2 q = *reinterpret_cast<const ulonglong2*>(row + wc + r);
        v[r] = q.x;
        v[r + 1] = q.y;
      }
    }
  };
  auto fetch = [&](uint32_t tile, uint64_t (&lv)[kRegLeaves][R], uint64_t (&ep)[R], uint64_t (&en)[R]) {
    const uint32_t wc = min(tile * (256 * R) + tid * R, kb.S - R);
#pragma unroll
    for (int j = 0; j < kRegLeaves; ++j) load_words(lrow[j], wc, lv[j]);
    load_words(kb.pos, wc, ep);
    load_words(kb.neg, wc, en);
  };
  const uint32_t t_end = min((run + 1) * tpb, tiles);
  uint64_t lv[kRegLeaves][R], ep[R], en[R];
  fetch(run * tpb, lv, ep, en);
  uint32_t p = 0, q = 0;
  for (uint32_t tile = run * tpb; tile < t_end; ++tile) {
    uint64_t nlv[kRegLeaves][R], nep[R], nen[R];
    if (tile + 1 < t_end) fetch(tile + 1, nlv, nep, nen);
    const uint32_t w0 = tile * (256 * R) + tid * R;
    uint64_t top[R], st[D > 1 ? D - 1 : 1][R];
#pragma unroll
    for (int r = 0; r < R; ++r) top[r] = 0;
    uint32_t pc = 0;
    // segment j runs the program up to and including its j-th leaf; the last
    // segment runs the rest, loading its leaves itself
#pragma unroll
    for (int j = 0; j <= kRegLeaves; ++j) {
      while (pc < len) {
        const uint32_t ins = prog[pc++];
        const uint32_t op = ins & 15u, arg = ins >> 5;
        if (op <= RP_BOT) {
          uint64_t val[R];                        // the operand's words
          const bool ahead = op == RP_LEAF && j < kRegLeaves;
          if (op == RP_LEAF) {
            const uint64_t negm = (ins & 16u) ? ~0ull : 0ull;
            if (ahead) {
#pragma unroll
              for (int r = 0; r < R; ++r) val[r] = lv[j < kRegLeaves ? j : 0][r] ^ negm;
            } else {
              const uint64_t* row = row_ptr(kb, arg);
#pragma unroll
              for (int r = 0; r < R; ++r) {
                const uint32_t w = w0 + r;
                val[r] = w < W ? (row[w] ^ negm) : 0ull;
              }
            }
          } else {
#pragma unroll
            for (int r = 0; r < R; ++r) val[r] = op == RP_TOP ? ~0ull : 0ull;
          }
          // an operand followed by AND / OR folds into the top: no push, no pop
          // (every operand of a flattened conjunction or disjunction but the first)
          const uint32_t nop = pc < len ? (prog[pc] & 15u) : (uint32_t)RP_LEAF;
          if (pc > 1 && (nop == RP_AND || nop == RP_OR)) {
#pragma unroll
            for (int r = 0; r < R; ++r) top[r] = nop == RP_AND ? (top[r] & val[r]) : (top[r] | val[r]);
            ++pc;
          } else {
            if (pc > 1) {                         // push: shift the stack down
#pragma unroll
              for (int i = D - 2; i > 0; --i)
#pragma unroll
                for (int r = 0; r < R; ++r) st[i][r] = st[i - 1][r];
#pragma unroll
              for (int r = 0; r < R; ++r) st[0][r] = top[r];
            }
#pragma unroll
            for (int r = 0; r < R; ++r) top[r] = val[r];
          }
          if (ahead) break;
        } else if (op == RP_NOT) {
#pragma unroll
          for (int r = 0; r < R; ++r) top[r] = ~top[r];
        } else {                                  // pop b, top = top op b
          const bool conj = op == RP_AND;
#pragma unroll
          for (int r = 0; r < R; ++r) top[r] = conj ? (top[r] & st[0][r]) : (top[r] | st[0][r]);
#pragma unroll
          for (int i = 0; i + 1 < D - 1; ++i)
#pragma unroll
            for (int r = 0; r < R; ++r) st[i][r] = st[i + 1][r];
        }
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint32_t w = w0 + r;
      uint64_t v = top[r];
      if (w >= W) v = 0;
      else if (w == W - 1) v &= tail;
      if (out && w < kb.S) out[w] = v;
      if (cover) {
        p += (uint32_t)__popcll(v & ep[r]);
        q += (uint32_t)__popcll(v & en[r]);
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      ep[r] = nep[r];
      en[r] = nen[r];
#pragma unroll
      for (int j = 0; j < kRegLeaves; ++j) lv[j][r] = nlv[j][r];
    }
  }
  if (cover) {
    p = wave_sum(p);
    q = wave_sum(q);
    if ((tid & 63) == 0) {
      s_pq[0][tid >> 6] = p;
      s_pq[1][tid >> 6] = q;
    }
    __syncthreads();
    if (tid == 0) {
      const uint32_t P = s_pq[0][0] + s_pq[0][1] + s_pq[0][2] + s_pq[0][3];
      const uint32_t Q = s_pq[1][0] + s_pq[1][1] + s_pq[1][2] + s_pq[1][3];
      if (P) atomicAdd(kb.counts + 2 * T.cover, P);
      if (Q) atomicAdd(kb.counts + 2 * T.cover + 1, Q);
    }
  }
}

// ---------------------------------------------------------------------------
// single role restriction, one wave per 64 subjects
// ---------------------------------------------------------------------------
// A wave walks its words of the direction's list as a pipeline: while one
// word is counted, the targets of the next and the offsets of the one after
// are in flight.  A word's assertions are one range, taken in rounds of
// kRoleChunks chunks of 64 (the first round's loads are the ones in flight;
// at 8 assertions a subject a second is rare); a subject's count is the
// difference of two prefix counts over the ballots of child members.  The child row is
// staged in LDS where it fits, with 16-byte loads, all of a lane's in flight.
// One node over 1M individuals and 8.3M assertions: 18 us, where one word
// at a time, counted chunk by chunk, and 8-byte staging took 36 (8 chunks a
// round 21, 12 19).
constexpr int kRoleChunks = 10;   // 64-assertion chunks whose loads a wave issues together
struct RoleRows {                 // a word's subjects: their rows, heavy ones left out
  uint32_t w, olo, ohi, i0, ee;
  bool in, heavy;
};
__device__ __forceinline__ RoleRows role_rows(const DevKB& kb, const uint32_t* __restrict__ off, uint32_t w, int lane) {
  RoleRows q;
  q.w = w;
  const uint32_t x = w * 64 + lane;
  q.in = x < kb.N;
  q.olo = off[q.in ? x : kb.N];
  q.ohi = off[q.in ? x + 1 : kb.N];
  return q;
}
__device__ __forceinline__ void role_range(const DevKB& kb, RoleRows& q) {
  q.heavy = q.ohi - q.olo > kb.heavy_min;   // counted by k_role_heavy instead
  if (q.heavy) q.ohi = q.olo;
  q.ee = (uint32_t)__builtin_amdgcn_readlane((int)q.ohi, 63);
  q.i0 = (uint32_t)__builtin_amdgcn_readlane((int)q.olo, 0);
}
__device__ __forceinline__ void role_targets(const int32_t* __restrict__ tg, uint32_t i0, uint32_t ee, int lane,
                                             int32_t (&t)[kRoleChunks]) {
#pragma unroll
  for (int c = 0; c < kRoleChunks; ++c) {
    const uint32_t e = i0 + 64 * c + lane;   // (a listed word's role has a target 0)
    t[c] = tg[e < ee ? e : 0u];
  }
}

template <bool STAGE>
__global__ void __launch_bounds__(STAGE ? 1024 : 256)
k_role(DevKB kb, const RoleTask* __restrict__ tasks, uint32_t bpt) {
  extern __shared__ uint64_t lds_child[];
  const uint32_t task = blockIdx.x / bpt, b = blockIdx.x % bpt;
  const RoleTask T = tasks[task];
  const uint32_t* child = reinterpret_cast<const uint32_t*>(row_ptr(kb, T.child_row));
  const size_t ro = (size_t)T.role * (kb.N + 1);
  const uint32_t* off = (T.inv ? kb.inv_off : kb.fwd_off) + ro;
  const int32_t* tg = (T.inv ? kb.inv_tg : kb.fwd_tg) + kb.role_base[T.role];
  uint64_t* out = out_ptr(kb, T.out_row);
  const uint32_t* words = kb.words + (size_t)(2 * T.role + T.inv) * kb.W;
  const uint32_t nw = blockDim.x >> 6, step = bpt * nw;
  const int lane = threadIdx.x & 63;
  uint32_t i = b * nw + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool any = i < T.n_words;
  auto word = [&](uint32_t j) { return scalar_u32(words + min(j, T.n_words - 1)); };
  RoleRows q{}, qn{};
  int32_t t[kRoleChunks];
  if (any) {
    q = role_rows(kb, off, word(i), lane);
    qn = role_rows(kb, off, word(i + step), lane);
    role_range(kb, q);
    role_targets(tg, q.i0, q.ee, lane, t);
  }
  if (STAGE) {
    constexpr uint32_t kFly = 8;
    typedef uint32_t U4 __attribute__((ext_vector_type(4)));
    const U4* src = reinterpret_cast<const U4*>(child);
    U4* dst = reinterpret_cast<U4*>(lds_child);
    const uint32_t n2 = (kb.W + 1) / 2;      // (rows are a multiple of 8 words long)
    for (uint32_t j0 = threadIdx.x; j0 < n2; j0 += kFly * blockDim.x) {
      U4 v[kFly];
#pragma unroll
      for (uint32_t j = 0; j < kFly; ++j) v[j] = src[min(j0 + j * blockDim.x, n2 - 1)];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (uint32_t j = 0; j < kFly; ++j)
        if (j0 + j * blockDim.x < n2) dst[j0 + j * blockDim.x] = v[j];
    }
    __syncthreads();
    child = reinterpret_cast<const uint32_t*>(lds_child);
  }
  for (; i < T.n_words; i += step) {
    RoleRows qnn = role_rows(kb, off, word(i + 2 * step), lane);
    role_range(kb, qn);
    int32_t tn[kRoleChunks];
    role_targets(tg, qn.i0, i + step < T.n_words ? qn.ee : qn.i0, lane, tn);
    __builtin_amdgcn_sched_barrier(0);
    uint32_t cnt = 0, i0 = q.i0;
    while (i0 < q.ee) {
      ChunkSums sums;
      uint32_t v[kRoleChunks];
#pragma unroll
      for (int c = 0; c < kRoleChunks; ++c) v[c] = child[(uint32_t)t[c] >> 5];
      // (values past ee lie past every subject's range)
      unrolled<kRoleChunks>([&](auto c) {
        sums.template put<c.value>(__ballot(((v[c.value] >> (t[c.value] & 31)) & 1u) != T.neg));
      });
      cnt += sums.template count<kRoleChunks>(q.olo, q.ohi, i0);
      const uint32_t round = 64 * kRoleChunks;
      const uint64_t pend = __ballot(q.in && cnt < T.sat && q.ohi > i0 + round);
      if (!pend) break;
      const int l = __ffsll((unsigned long long)pend) - 1;
      const uint32_t nxt = (uint32_t)__builtin_amdgcn_readlane((int)q.olo, l);
      i0 = max(i0 + round, nxt);
      role_targets(tg, i0, q.ee, lane, t);
    }
    const bool res = q.in && !q.heavy && cnt >= T.lo && cnt <= T.hi;
    const uint64_t bits = __ballot(res);
    if (lane == 0) out[q.w] = bits;
    q = qn;
    qn = qnn;
#pragma unroll
    for (int c = 0; c < kRoleChunks; ++c) t[c] = tn[c];
  }
}

// The task of heavy-row block b or counter i: the last task whose first block
// (counter) is <= b; tasks without heavy rows own empty ranges.
template <bool BLOCKS>
__device__ __forceinline__ uint32_t heavy_task(const RoleTask* __restrict__ tasks, uint32_t n, uint32_t b) {
  uint32_t lo = 0, hi = n;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if ((BLOCKS ? tasks[mid].h_first : tasks[mid].c_first) <= b) lo = mid;
    else hi = mid;
  }
  return lo;
}

// One chunk of kHeavyChunk assertions of one heavy row per block: the count
// of child members among them goes to partial[block] (no early exit: every
// chunk is counted, so that no two blocks touch the same word).
__global__ void __launch_bounds__(256)
k_role_heavy(DevKB kb, const RoleTask* __restrict__ tasks, uint32_t n_tasks, uint32_t b0,
             uint32_t* __restrict__ partial) {
  __shared__ uint32_t s_part[4];
  const uint32_t b = b0 + blockIdx.x;
  const RoleTask T = tasks[heavy_task<true>(tasks, n_tasks, b)];
  const HeavyChunk c = kb.heavy_chunks[T.hc0 + (b - T.h_first)];
  const uint32_t x = kb.heavy_rows[c.hrow];
  const uint32_t* off = (T.inv ? kb.inv_off : kb.fwd_off) + (size_t)T.role * (kb.N + 1);
  const int32_t* tg = (T.inv ? kb.inv_tg : kb.fwd_tg) + kb.role_base[T.role];
  const uint64_t* child = row_ptr(kb, T.child_row);
  const uint32_t e0 = off[x] + c.k * kHeavyChunk;
  const uint32_t e1 = min(off[x + 1], e0 + kHeavyChunk);
  uint32_t cnt = 0;
#pragma unroll
  for (uint32_t j = 0; j < kHeavyChunk / 256; ++j) {
    const uint32_t e = e0 + j * 256 + threadIdx.x;
    if (e < e1) {
      const uint32_t t = (uint32_t)tg[e];
      cnt += ((uint32_t)(child[t >> 6] >> (t & 63)) & 1u) ^ T.neg;
    }
  }
  cnt = wave_sum(cnt);
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) partial[b] = s_part[0] + s_part[1] + s_part[2] + s_part[3];
}

// One block per (task, heavy row): the sum of the row's chunk partials gives
// the row's bit.  Runs after k_role has written the rows' words (with the
// heavy bits clear).
__global__ void __launch_bounds__(256)
k_role_heavy_fix(DevKB kb, const RoleTask* __restrict__ tasks, uint32_t n_tasks, uint32_t i0,
                 const uint32_t* __restrict__ partial) {
  __shared__ uint32_t s_part[4];
  const uint32_t i = i0 + blockIdx.x;
  const RoleTask T = tasks[heavy_task<false>(tasks, n_tasks, i)];
  const uint32_t hrow = T.hr0 + (i - T.c_first);
  const uint32_t c0 = kb.heavy_chunk0[hrow], n = kb.heavy_chunk0[hrow + 1] - c0;
  const uint32_t* p = partial + T.h_first + (c0 - T.hc0);
  uint32_t cnt = 0;
#pragma unroll 8
  for (uint32_t c = threadIdx.x; c < n; c += 256) cnt += p[c];
  cnt = wave_sum(cnt);
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    cnt = s_part[0] + s_part[1] + s_part[2] + s_part[3];
    const uint32_t x = kb.heavy_rows[hrow];
    const unsigned long long bit = 1ull << (x & 63);
    unsigned long long* word = reinterpret_cast<unsigned long long*>(out_ptr(kb, T.out_row) + (x >> 6));
    if (cnt >= T.lo && cnt <= T.hi) atomicOr(word, bit);
    else atomicAnd(word, ~bit);
  }
}

// A single ∃ρ.A (lo = 1, hi unbounded) or ¬∃ρ.A (lo = hi = 0) whose atomic
// child A is sparse, pushed from A's members: every y in A takes the subjects
// x that reach it (its row in the opposite direction) and sets (∃) or clears
// (¬∃) their bits in the output row, which a fill task has set to all zeros
// or all ones before.  One wave per word of A, a lane per member walking its
// row alone, so it is only chosen where every row of the opposite direction
// is short (kPushMaxDeg).
__global__ void __launch_bounds__(256)
k_push(DevKB kb, const RoleTask* __restrict__ tasks, uint32_t tiles) {
  const uint32_t t = blockIdx.x / tiles, tile = blockIdx.x % tiles;
  const uint32_t w = tile * 4 + (threadIdx.x >> 6);
  if (w >= kb.W) return;
  const RoleTask T = tasks[t];
  const int lane = threadIdx.x & 63;
  const uint64_t cw = row_ptr(kb, T.child_row)[w];
  if (!((cw >> lane) & 1ull)) return;
  const uint32_t y = w * 64 + lane;
  const uint32_t* off = (T.inv ? kb.fwd_off : kb.inv_off) + (size_t)T.role * (kb.N + 1);
  const int32_t* tg = (T.inv ? kb.fwd_tg : kb.inv_tg) + kb.role_base[T.role];
  unsigned long long* out = reinterpret_cast<unsigned long long*>(out_ptr(kb, T.out_row));
  const uint32_t e1 = off[y + 1];
  const bool mark = T.lo == 1;
#pragma unroll 4
  for (uint32_t e = off[y]; e < e1; ++e) {
    const uint32_t x = (uint32_t)tg[e];
    const unsigned long long bit = 1ull << (x & 63);
    if (mark) atomicOr(out + (x >> 6), bit);
    else atomicAnd(out + (x >> 6), ~bit);
  }
}

// Zero-count results for the words of a role direction without assertions:
// the whole row, four words (two 16-byte stores) per thread.  Rows are
// stride_words apart, a multiple of 8, so a thread's words never cross a row.
constexpr uint32_t kFillWords = 4;
inline uint32_t fill_tiles(uint32_t S) { return (S + 256 * kFillWords - 1) / (256 * kFillWords); }
__global__ void __launch_bounds__(256)
k_fill_rows(DevKB kb, const FillTask* __restrict__ tasks, uint32_t tiles) {
  const uint32_t t = blockIdx.x / tiles, tile = blockIdx.x % tiles;
  const FillTask F = tasks[t];
  const uint32_t w0 = (tile * 256 + threadIdx.x) * kFillWords;
  if (w0 >= kb.S) return;
  uint64_t v[kFillWords];
#pragma unroll
  for (uint32_t i = 0; i < kFillWords; ++i) {
    const uint32_t w = w0 + i;
    v[i] = F.ones && w < kb.W ? (w == kb.W - 1 ? kb.tail : ~0ull) : 0ull;
  }
  ulonglong2* q = reinterpret_cast<ulonglong2*>(out_ptr(kb, F.out_row) + w0);
  q[0] = make_ulonglong2(v[0], v[1]);
  q[1] = make_ulonglong2(v[2], v[3]);
}

}  // namespace hth

#include "group_kernels.h"

namespace hth {

// ---------------------------------------------------------------------------
// executor
// ---------------------------------------------------------------------------
// The T rows of the groups of one launch stay within kb.tune.t_budget bytes so
// that the random T fetches of a launch stay in the last-level caches.
inline uint32_t t_width_bytes(uint32_t k) { return k <= 8 ? 1 : k <= 16 ? 2 : k <= 32 ? 4 : 8; }
inline size_t t_area_bytes(const hth_kb_s& kb) {
  return std::max<size_t>(kb.tune.t_budget, align_up(kb.N, 64) * 8);
}
// T rows of a group: the objects of its direction (compact) or all individuals
inline uint64_t t_rows(const hth_kb_s& kb, const GroupTask& g) {
  return align_up(g.compact ? kb.n_obj[2 * g.role + g.inv] : kb.N, 64);
}

// Consecutive groups of a level share a launch while their T rows, at the
// widest T width among them, fit the budget; sets each group's T offset.
struct GroupChunk {
  size_t first;
  uint32_t n, wb;
  uint32_t rounds;     // XCD-local: rounds of the slot table (0 = chip-wide launch)
  size_t slot_off;     // its first entry in the plan's slot table
  uint32_t build;      // groups whose T rows its launch builds: its own, the next chunk's too, or none
};
// XCD-local placement of a chunk's groups: longest first onto the least loaded
// XCD (cost ~ assertions + 64 per visited word); slot (round, xcd) -> group.
void place_on_xcds(const hth_kb_s& kb, const std::vector<GroupTask>& gs, GroupChunk& c,
                   std::vector<uint32_t>& xslots) {
  std::vector<std::pair<double, uint32_t>> cost;
  for (uint32_t i = 0; i < c.n; ++i) {
    const GroupTask& g = gs[c.first + i];
    const double e = (double)(kb.role_base[g.role + 1] - kb.role_base[g.role]);
    cost.push_back({e + 64.0 * kb.n_words[2 * g.role + g.inv], i});
  }
  std::stable_sort(cost.begin(), cost.end(), [](const auto& a, const auto& b) { return a.first > b.first; });
  double load[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  std::vector<uint32_t> per[8];
  for (const auto& [w, i] : cost) {
    const int x = (int)(std::min_element(load, load + 8) - load);
    load[x] += w;
    per[x].push_back(i);
  }
  size_t rounds = 0;
  for (int x = 0; x < 8; ++x) rounds = std::max(rounds, per[x].size());
  c.rounds = (uint32_t)rounds;
  c.slot_off = xslots.size();
  xslots.resize(xslots.size() + rounds * 8, kNone);
  for (int x = 0; x < 8; ++x)
    for (size_t r = 0; r < per[x].size(); ++r) xslots[c.slot_off + r * 8 + x] = per[x][r];
}

// groups per launch stay few enough for the pass's grid (at most 8 x 256
// blocks per XCD round) to stay far below 2^31 work-items
constexpr size_t kMaxGroupsPerLaunch = 2048;

// Role direction rd = 2 role + inv holds only short rows: its shared passes
// walk one subject per lane (k_group_short)
inline bool short_rows(const hth_kb_s& kb, uint32_t rd) {
  return kb.tune.short_rows && kb.max_deg[rd & 1][rd >> 1] <= kb.tune.short_rows;
}

std::vector<GroupChunk> chunk_groups(const hth_kb_s& kb, std::vector<GroupTask>& gs) {
  std::vector<GroupChunk> out;
  size_t i = 0;
  while (i < gs.size()) {
    uint32_t wb = t_width_bytes(gs[i].k);
    uint64_t rows = t_rows(kb, gs[i]);
    size_t j = i + 1;
    while (j < gs.size() && j - i < kMaxGroupsPerLaunch && gs[j].short_rows == gs[i].short_rows) {
      const uint32_t nwb = std::max(wb, t_width_bytes(gs[j].k));
      if ((rows + t_rows(kb, gs[j])) * nwb > kb.tune.t_budget) break;
      rows += t_rows(kb, gs[j]);
      wb = nwb;
      ++j;
    }
    uint64_t off = 0;
    for (size_t q = i; q < j; ++q) {
      gs[q].t_off = off;
      off += t_rows(kb, gs[q]);
    }
    out.push_back({i, (uint32_t)(j - i), wb, 0, 0, (uint32_t)(j - i)});
    i = j;
  }
  // the last short-row chunk and the first of the others build their T rows in
  // one launch where that makes neither's wider, or over few words (a launch
  // less per level, 4 to 6 us each: a batch of 256 hypotheses over 10,000
  // individuals, 44 launches before, takes 292 us, 320 with two builds a level)
  constexpr uint32_t kMixWords = 1024;
  constexpr uint64_t kMixBytes = 64ull << 20;   // T rows of both, still in the last-level cache for the second pass
  for (size_t c = 0; c + 1 < out.size(); ++c) {
    GroupChunk& a = out[c];
    GroupChunk& b = out[c + 1];
    if (!gs[a.first].short_rows || gs[b.first].short_rows) continue;
    auto rows = [&](const GroupChunk& x) { return gs[x.first + x.n - 1].t_off + t_rows(kb, gs[x.first + x.n - 1]); };
    const uint32_t wb = std::max(a.wb, b.wb);
    const uint64_t ra = rows(a);
    if ((a.wb != b.wb && kb.W > kMixWords) || (ra + rows(b)) * wb > std::min<uint64_t>(kb.tune.t_budget, kMixBytes) ||
        a.n + b.n > kMaxGroupsPerLaunch)
      continue;
    for (uint32_t g = 0; g < b.n; ++g) gs[b.first + g].t_off += ra;
    a.wb = b.wb = wb;
    a.build = a.n + b.n;
    b.build = 0;
  }
  return out;
}

// T bytes the chunks of one level use at most: a chunk's rows run from its
// first group's t_off (0) to the end of its last group's, at the chunk's width.
inline size_t chunks_t_bytes(const hth_kb_s& kb, const std::vector<GroupTask>& gs,
                             const std::vector<GroupChunk>& cs) {
  size_t most = 0;
  for (const GroupChunk& c : cs) {
    const GroupTask& last = gs[c.first + c.n - 1];
    most = std::max<size_t>(most, (size_t)(last.t_off + t_rows(kb, last)) * c.wb);
  }
  return align_up(most, 256);
}

// Target segments of a chunk: its passes cover T rows in ranges of at most
// t_segment bytes (at the chunk's T width), when that takes 2..kMaxSegments
// passes; otherwise one pass over all rows.  seg_rows: T rows per pass.
constexpr uint32_t kMaxSegments = 4;
uint32_t chunk_segments(const hth_kb_s& kb, const std::vector<GroupTask>& gs, const GroupChunk& c,
                        uint64_t* seg_rows) {
  uint64_t rows = 0;
  for (uint32_t i = 0; i < c.n; ++i) rows = std::max(rows, t_rows(kb, gs[c.first + i]));
  *seg_rows = rows;
  const uint64_t seg = (uint64_t)kb.tune.t_segment_kb << 10;
  if (!seg || rows * c.wb <= seg) return 1;
  const uint64_t P = (rows * c.wb + seg - 1) / seg;
  if (P > kMaxSegments) return 1;
  *seg_rows = align_up((rows + P - 1) / P, 64);
  return (uint32_t)P;
}
// partial counts carried between the passes of a segmented chunk
inline size_t chunk_partial_bytes(const hth_kb_s& kb, const std::vector<GroupTask>& gs, const GroupChunk& c) {
  uint64_t sr;
  return chunk_segments(kb, gs, c, &sr) > 1 ? (size_t)c.n * kb.W * 256 * c.wb : 0;
}

namespace {

struct Blob {
  std::vector<char> bytes;
  template <class T>
  size_t add(const std::vector<T>& v) {
    size_t at = align_up(bytes.size(), 256);
    if (v.empty()) return at;
    bytes.resize(at + v.size() * sizeof(T));
    std::memcpy(bytes.data() + at, v.data(), v.size() * sizeof(T));
    return at;
  }
};

size_t table_bound(uint32_t max_nodes, uint32_t max_hyps) {
  const size_t n = max_nodes + 2;
  size_t b = 0;
  b += align_up(n * sizeof(ThrTask), 256);
  b += align_up(n * sizeof(ThrGroup), 256);
  b += align_up(n * sizeof(NumTask), 256);
  b += align_up(n * sizeof(StrTask), 256);
  b += align_up(n * sizeof(ThrGroup), 256);                // num and string tasks by role
  b += align_up((n + max_hyps) * sizeof(RegionTask), 256);
  b += align_up(n * sizeof(RoleTask), 256);
  b += align_up(n * sizeof(RoleTask), 256);                // pushed role tasks
  b += align_up(n * sizeof(GroupTask), 256);
  b += align_up(n * sizeof(GroupMember), 256);
  b += align_up(n * sizeof(FillTask), 256);
  b += align_up((4 * n + 16) * sizeof(uint32_t), 256);
  b += align_up((9 * n + 8) * sizeof(uint32_t), 256);     // XCD slot tables
  return b + 4096;
}

DevKB dev_view(const hth_kb_s& kb) {
  DevKB d{};
  d.concepts = kb.d.concept_bits;
  d.data = kb.d.data;
  d.fwd_off = kb.fwd_off;
  d.inv_off = kb.inv_off;
  d.fwd_tg = kb.d.role_targets;
  d.inv_tg = kb.inv_tg;
  d.role_base = kb.role_base_dev;
  d.words = kb.words;
  d.objmask = kb.objmask;
  d.objbase = kb.objbase;
  d.ctg_fwd = kb.ctg_fwd;
  d.ctg_inv = kb.ctg_inv;
  d.heavy_rows = kb.heavy_rows;
  d.heavy_chunks = kb.heavy_chunks;
  d.heavy_chunk0 = kb.heavy_chunk0;
  d.heavy_min = kb.heavy_min;
  d.pos = kb.pos;
  d.neg = kb.neg;
  d.n_concepts = kb.d.n_concepts;
  d.n_fixed = kb.d.n_concepts;
  d.N = kb.N;
  d.W = kb.W;
  d.S = kb.S;
  d.tail = kb.tail;
  return d;
}

// words of the example view as counted at load: its kernels' grids are sized for
// them, and for view_fill blocks at least
inline uint32_t view_words_hint(const hth_kb_s& kb) { return (kb.ex_hint + 63) / 64 + 1; }

// Blocks for each of n items so that a launch over the view fills the chip
// however many examples there are by then (the rows may be other ones than at
// load, or rewritten; a block beyond the view's words leaves at once).  Loaded
// with one example and given 25,000 of 400,000 individuals, 64 hypotheses took
// 1,076 us with grids by the count at load, 106 with these, 106 loaded
// with all of them.
inline uint32_t view_fill(const hth_kb_s& kb, uint64_t n) { return (uint32_t)((4 * (uint64_t)kb.n_cu + n - 1) / n); }

// Kernel launches, each optionally bracketed by timing events.
struct Launcher {
  hth_kb_s& kb;
  hipStream_t st;
  // the (role, direction) CSRs already counted in this sweep (one role-nesting
  // level): the byte model reads each once per sweep however many passes use it
  std::vector<uint32_t> csr_seen;

  double csr_once(uint32_t role, uint32_t inv);

  hth_status event(hipEvent_t* e) {
    if (!kb.event_pool.empty()) {
      *e = kb.event_pool.back();
      kb.event_pool.pop_back();
      return HTH_OK;
    }
    HTH_HIP(hipEventCreate(e));
    return HTH_OK;
  }
  template <class F>
  hth_status run(int kind, double bytes, F&& launch) {
    hipEvent_t a = nullptr, b = nullptr;
    if (kb.prof) {
      hth_status s = event(&a);
      if (!s) s = event(&b);
      if (s) return s;
      HTH_HIP(hipEventRecord(a, st));
    }
    launch();
    HTH_HIP(hipGetLastError());
    if (kb.prof) {
      HTH_HIP(hipEventRecord(b, st));
      kb.prof_recs.push_back({kind, bytes, a, b});
    }
    return HTH_OK;
  }
};

// Launches of `items` work items, `per` blocks of `threads` lanes each, split
// so that no dispatch holds 2^31 work-items or more (a dispatch counts its
// grid in work-items in 32 bits; a larger grid would wrap, not fail).
// launch(first_item, item_count, blocks) issues one of them.
template <class F>
hth_status split_launch(Launcher& L, int kind, double bytes, uint64_t items, uint64_t per, uint32_t threads,
                        F&& launch) {
  const uint64_t max_blocks = (1ull << 31) / threads - 1;
  const uint64_t chunk = std::max<uint64_t>(1, max_blocks / std::max<uint64_t>(per, 1));
  for (uint64_t i0 = 0; i0 < items; i0 += chunk) {
    const uint64_t m = std::min(chunk, items - i0);
    hth_status s = L.run(kind, i0 ? 0.0 : bytes, [&] { launch((uint32_t)i0, (uint32_t)m, (uint32_t)(per * m)); });
    if (s) return s;
  }
  return HTH_OK;
}

// algorithmic bytes of the region tasks of one sweep (byte model): every
// distinct row they read once, each output row once, the two example rows
// once and 8 bytes of counts per hypothesis whose coverage they take
double region_bytes(const hth_kb_s& kb, const std::vector<RegionTask>& tasks, const std::vector<uint32_t>& code) {
  const double w8 = (double)kb.W * 8;
  std::vector<uint32_t> leaves;
  double b = 0;
  bool cover = false;
  for (const RegionTask& t : tasks) {
    for (uint32_t i = 0; i < t.code_len; ++i) {
      const uint32_t ins = code[t.code_off + i];
      if ((ins & 15u) == RP_LEAF) leaves.push_back(ins >> 5);
    }
    if (t.out_row != kNone) b += w8;
    if (t.cover != kNone) {
      b += 8;
      cover = true;
    }
  }
  std::sort(leaves.begin(), leaves.end());
  leaves.erase(std::unique(leaves.begin(), leaves.end()), leaves.end());
  return b + leaves.size() * w8 + (cover ? 2 * w8 : 0.0);
}

// a CSR direction scanned once: 32-bit row offsets and the role's targets
double csr_bytes(const hth_kb_s& kb, uint32_t role, uint32_t inv) {
  const double words = kb.n_words.empty() ? kb.W : kb.n_words[2 * role + inv];
  return 4.0 * std::min<double>((double)kb.N + 1, 65.0 * words) +
         4.0 * (double)(kb.role_base[role + 1] - kb.role_base[role]);
}

double Launcher::csr_once(uint32_t role, uint32_t inv) {
  const uint32_t key = 2 * role + inv;
  if (std::find(csr_seen.begin(), csr_seen.end(), key) != csr_seen.end()) return 0.0;
  csr_seen.push_back(key);
  return csr_bytes(kb, role, inv);
}

// tiles one block of the register region kernel walks (with the next tile's
// loads in flight while it evaluates one)
constexpr uint32_t kRegionTilesPerBlock = 16;
constexpr uint64_t kRegionMinBlocks = 16384;

// Blocks per threshold group over W words: about 32 words per wave, enough
// independent column loads in flight; fewer, down to the 8 a wave takes at
// once, while the launch would leave compute units idle (7 groups of 30
// thresholds over 157 words 28 us at 32 words a wave, 13 at 8).
inline uint32_t threshold_blocks(const hth_kb_s& kb, uint32_t n, uint32_t W) {
  return std::max<uint32_t>(1, std::min((W + 31) / 32, std::max((W + 127) / 128, 4 * kb.n_cu / n)));
}

// A plan's fills, every level's at once before the first: a launch less for
// each further level (3 % of a round over 200,000 individuals).  Far beyond the
// last-level cache too: 13.4 GB of fills on 17 levels (65,536 hypotheses over 4M
// individuals) take 2.78 ms at once and 2.65 level by level, which leaves part
// of them in the cache, but the T builds next to them 10.40 and 10.71, and the
// whole step 52.9 and 53.2.
hth_status launch_fills(Launcher& L, const DevKB& d, const FillTask* tasks, size_t n, double bytes) {
  if (!n) return HTH_OK;
  const uint32_t tiles = fill_tiles(L.kb.S);
  return split_launch(L, HTH_K_FILL, bytes, n, tiles, 256, [&](uint32_t i0, uint32_t, uint32_t blocks) {
    hipLaunchKernelGGL(k_fill_rows, dim3(blocks), dim3(256), 0, L.st, d, tasks + i0, tiles);
  });
}

// Tasks that share a walk of a value role's values, of `tasks` in all: one up to
// 2^14 words of results, and in proportion beyond.  Few words leave the chip
// room for a walk each, where a shared walk is a chain of its tasks; many fill
// it, and a walk of its own is another read of the values.  Batches, 1 / 2 / 4 /
// 8 / 16 a walk, us (words): 5,000 individuals 24.7 / 25.9 / 28.9 / 35.0 / 47.7
// (3,160), 131,073 29.2 / 27.7 / 29.6 / 35.4 / 35.4 (31,000), 262,145 41.6 / 36.9 /
// 36.3 / 41.1 / 40.7 (61,000), 524,289 63.3 / 57.9 / 53.9 / 52.2 / 52.9 (123,000),
// 1M 91.1 / 81.0 / 75.9 / 73.7 / 73.4 (234,000).
inline uint32_t value_tasks(const hth_kb_s& kb, size_t tasks) {
  return (uint32_t)std::min<uint64_t>(kValPerPass, std::max<uint64_t>(1, ((uint64_t)tasks * kb.W + (1u << 13)) >> 14));
}
inline uint32_t value_blocks(const hth_kb_s& kb, uint32_t n) {
  return std::max<uint32_t>(1, std::min<uint32_t>((kb.W + 7) / 8, (32 * kb.n_cu + n - 1) / n));
}

// n region tasks whose programs need at most `depth` stack entries
hth_status launch_regions_n(Launcher& L, const DevKB& d, const RegionTask* tasks, const uint32_t* code,
                            uint32_t n, int depth, double bytes) {
  if (!n) return HTH_OK;
  // the register kernel when every program's stack fits its shift register
  // (the view: as many words as the load's examples fill, and blocks for the
  // whole chip; the kernels cover however many there are)
  const uint32_t S = d.view ? std::min(d.S, view_words_hint(L.kb)) : d.S;
  if (depth <= kRegDepth && L.kb.tune.region_reg) {
    const uint32_t rw = L.kb.tune.region_reg;     // words per lane: 1, 2 or 4
    const uint32_t tiles = (S + 256 * rw - 1) / (256 * rw);
    // a block walks up to kRegionTilesPerBlock tiles of its task, fewer when
    // the launch would otherwise have under kRegionMinBlocks blocks
    const uint64_t per = std::max<uint64_t>(1, (uint64_t)n * tiles / kRegionMinBlocks);
    const uint32_t tpb = (uint32_t)std::min<uint64_t>(std::min<uint64_t>(tiles, kRegionTilesPerBlock), per);
    const uint32_t most = (d.S + 256 * rw - 1) / (256 * rw);
    const uint32_t runs = std::max((tiles + tpb - 1) / tpb, d.view ? std::min(most, view_fill(L.kb, n)) : 0u);
    return split_launch(L, HTH_K_REGION, bytes, n, runs, 256, [&](uint32_t t0, uint32_t m, uint32_t blocks) {
      const dim3 grid(blocks), block(256);
      if (rw == 1)
        hipLaunchKernelGGL((k_region_reg<kRegDepth, 1>), grid, block, 0, L.st, d, tasks + t0, code, m, tiles, tpb, runs);
      else if (rw == 2)
        hipLaunchKernelGGL((k_region_reg<kRegDepth, 2>), grid, block, 0, L.st, d, tasks + t0, code, m, tiles, tpb, runs);
      else
        hipLaunchKernelGGL((k_region_reg<kRegDepth, 4>), grid, block, 0, L.st, d, tasks + t0, code, m, tiles, tpb, runs);
    });
  }
  const uint32_t most = (d.S + kRegionThreads - 1) / kRegionThreads;
  const uint32_t tiles = std::max((S + kRegionThreads - 1) / kRegionThreads, d.view ? std::min(most, view_fill(L.kb, n)) : 0u);
  return split_launch(L, HTH_K_REGION, bytes, n, tiles, kRegionThreads, [&](uint32_t t0, uint32_t m, uint32_t blocks) {
    hipLaunchKernelGGL(k_region, dim3(blocks), dim3(kRegionThreads), 0, L.st, d, tasks + t0, code, m, tiles);
  });
}

hth_status launch_regions(Launcher& L, const DevKB& d, const RegionTask* tasks, const uint32_t* code,
                          const std::vector<RegionTask>& host, const std::vector<uint32_t>& hcode) {
  const double bytes = L.kb.prof ? region_bytes(L.kb, host, hcode) : 0.0;
  int depth = 0;
  for (const RegionTask& t : host) {
    int sp = 0;
    for (uint32_t i = 0; i < t.code_len; ++i) {
      const uint32_t op = hcode[t.code_off + i] & 15u;
      if (op <= RP_BOT) sp += i ? 1 : 0;
      else if (op != RP_NOT) --sp;
      depth = std::max(depth, sp + 1);
    }
  }
  return launch_regions_n(L, d, tasks, code, (uint32_t)host.size(), depth, bytes);
}

hth_status launch_roles_n(Launcher& L, const DevKB& d, const RoleTask* tasks, uint32_t n, double bytes) {
  const hth_kb_s& kb = L.kb;
  if (!n) return HTH_OK;
  const size_t lds = align_up((size_t)kb.W * 8, 16);
  if (lds <= kb.lds_per_block) {
    // one 1024-lane block per CU holds the child row in LDS: one round of blocks,
    // so that each CU stages the row once
    uint32_t bpt = std::max<uint32_t>(1, (kb.n_cu + n - 1) / n);
    bpt = std::min<uint32_t>(bpt, (kb.W + 15) / 16);
    return split_launch(L, HTH_K_ROLE, bytes, n, bpt, 1024, [&](uint32_t t0, uint32_t, uint32_t blocks) {
      hipLaunchKernelGGL(k_role<true>, dim3(blocks), dim3(1024), lds, L.st, d, tasks + t0, bpt);
    });
  }
  uint32_t bpt = std::max<uint32_t>(1, (8 * kb.n_cu + n - 1) / n);
  bpt = std::min<uint32_t>(bpt, (kb.W + 3) / 4);
  return split_launch(L, HTH_K_ROLE, bytes, n, bpt, 256, [&](uint32_t t0, uint32_t, uint32_t blocks) {
    hipLaunchKernelGGL(k_role<false>, dim3(blocks), dim3(256), 0, L.st, d, tasks + t0, bpt);
  });
}

hth_status launch_roles(Launcher& L, const DevKB& d, const RoleTask* tasks,
                        const std::vector<RoleTask>& host) {
  // per node: its CSR once per sweep, its child row in, its listed words out
  double bytes = 0;
  for (const RoleTask& t : host)
    bytes += L.csr_once(t.role, t.inv) + 8.0 * L.kb.W + 8.0 * L.kb.n_words[2 * t.role + t.inv];
  return launch_roles_n(L, d, tasks, (uint32_t)host.size(), bytes);
}

// vd, passes: the example view and its tasks, whose T rows are built from the
// groups' real directions (d, groups); null: the pass runs on those too.
template <typename TW>
hth_status launch_group_chunk(Launcher& L, const DevKB& d, const GroupTask* groups,
                              const GroupMember* members, const std::vector<GroupTask>& host,
                              const GroupChunk& c, const uint32_t* xslots_all, void* tarea, void* parea,
                              const DevKB* vd, const GroupTask* passes) {
  const hth_kb_s& kb = L.kb;
  const size_t g0 = c.first;
  const uint32_t n = c.n;
  // byte model: the transpose reads the members' child rows (T is an
  // intermediate of this design, not counted); the pass reads its CSR once per
  // sweep and writes the members' listed words (the other words are filled)
  double tb = 0, gb = 0;
  for (uint32_t i = 0; i < c.build; ++i) tb += (double)host[g0 + i].k * kb.W * 8;
  for (uint32_t i = 0; i < n; ++i) {
    const GroupTask& G = host[g0 + i];
    // (the view: the examples' share of both)
    gb += vd ? L.csr_once(G.role, G.inv) * kb.ex_hint / kb.N + (double)G.k * view_words_hint(kb) * 8
             : L.csr_once(G.role, G.inv) + (double)G.k * G.n_words * 8;
  }
  TW* T = static_cast<TW*>(tarea);
  hth_status s = HTH_OK;
  if (c.build) {
    // 256 words per block: every word, or the object words of a compact group
    uint32_t span = 1;
    for (uint32_t i = 0; i < c.build; ++i) {
      const GroupTask& G = host[g0 + i];
      span = std::max(span, G.compact ? G.n_obj_words : kb.W);
    }
    const uint32_t tiles = (span + 255) / 256;
    s = split_launch(L, HTH_K_TBUILD, tb, c.build, tiles, 256, [&](uint32_t i0, uint32_t, uint32_t blocks) {
      hipLaunchKernelGGL(k_tbuild<TW>, dim3(blocks), dim3(256), 0, L.st, d, groups + g0 + i0, members, T, tiles);
    });
    if (s) return s;
  }
  const uint32_t* xslots = c.rounds ? xslots_all + c.slot_off : nullptr;
  const uint32_t most_b = (kb.W + 3) / 4;       // blocks that have a word each, at most
  uint32_t bpg, nblocks;
  if (xslots) {
    bpg = std::min<uint32_t>(std::max<uint32_t>(1, kb.n_cu / 8 * 8), most_b);
    if (vd) bpg = std::min(bpg, std::max((view_words_hint(kb) + 3) / 4, view_fill(kb, 8ull * c.rounds)));
    nblocks = 8 * bpg * c.rounds;
  } else {
    bpg = std::max<uint32_t>(1, (8 * kb.n_cu + n - 1) / n);
    if (vd) bpg = std::min(bpg, std::max((view_words_hint(kb) + 3) / 4, view_fill(kb, n)));
    bpg = std::min<uint32_t>(bpg, most_b);
    nblocks = bpg * n;
  }
  const DevKB& pd = vd ? *vd : d;
  const GroupTask* pg = (vd ? passes : groups) + g0;
  // several list words per wave iteration where words hold few assertions
  double ew = 0, nwd = 0;
  for (uint32_t i = 0; i < n; ++i) {
    const GroupTask& G = host[g0 + i];
    ew += (double)(kb.role_base[G.role + 1] - kb.role_base[G.role]);
    nwd += G.n_words;
  }
  const bool multi = nwd > 0 && ew < 96.0 * nwd;
  if (host[g0].short_rows) {   // every row short: a lane per subject, one pass
    // exact 3-bit counts when no row of the launch's directions holds 8 assertions
    uint32_t most = 0;
    for (uint32_t i = 0; i < n; ++i) {
      const GroupTask& G = host[g0 + i];
      most = std::max(most, kb.max_deg[G.inv][G.role]);
    }
    auto go = [&](auto view) {
      constexpr bool VIEW = decltype(view)::value;
      if (most < kGroupMaxCount)
        hipLaunchKernelGGL((k_group_short<TW, kShortWords, kShortSub, kShortFly<TW>, true, VIEW>), dim3(nblocks), dim3(256),
                           0, L.st, pd, pg, members, T, bpg, xslots);
      else
        hipLaunchKernelGGL((k_group_short<TW, kShortWords, kShortSub, kShortFly<TW>, false, VIEW>), dim3(nblocks), dim3(256),
                           0, L.st, pd, pg, members, T, bpg, xslots);
    };
    return L.run(HTH_K_GROUP_SHORT, gb, [&] {
      if (vd) go(std::true_type());
      else go(std::false_type());
    });
  }
  uint64_t seg_rows = 0;
  const uint32_t P = vd ? 1 : chunk_segments(kb, host, c, &seg_rows);
  for (uint32_t sg = 0; sg < P; ++sg) {
    SegPass<TW> sp{0, 0xFFFFFFFFu, 1, 1, nullptr, (size_t)kb.W * 256};
    if (P > 1) {
      sp.lo = (uint32_t)(sg * seg_rows);
      sp.hi = (uint32_t)std::min<uint64_t>((sg + 1) * seg_rows, 0xFFFFFFFFu);
      sp.first = sg == 0;
      sp.last = sg == P - 1;
      sp.part = static_cast<TW*>(parea);
    }
    s = L.run(HTH_K_GROUP, sg ? 0.0 : gb, [&] {
      const dim3 grid(nblocks), block(256);
      const bool u16 = kb.tune.group_unroll >= 16;
      auto go = [&](auto view) {
        constexpr bool VIEW = decltype(view)::value;
        if (multi)    // few assertions per lane: 8 in flight
          hipLaunchKernelGGL((k_group<TW, 8, 4, VIEW>), grid, block, 0, L.st, pd, pg, members, T, bpg, xslots, sp);
        else if (u16)
          hipLaunchKernelGGL((k_group<TW, 16, 1, VIEW>), grid, block, 0, L.st, pd, pg, members, T, bpg, xslots, sp);
        else
          hipLaunchKernelGGL((k_group<TW, 8, 1, VIEW>), grid, block, 0, L.st, pd, pg, members, T, bpg, xslots, sp);
      };
      if (vd) go(std::true_type());
      else go(std::false_type());
    });
    if (s) return s;
  }
  return HTH_OK;
}

hth_status launch_groups(Launcher& L, const DevKB& d, const GroupTask* groups,
                         const GroupMember* members, const std::vector<GroupTask>& host,
                         const std::vector<GroupChunk>& chunks, const uint32_t* xslots, void* tarea,
                         void* parea, const DevKB* vd = nullptr, const GroupTask* passes = nullptr) {
  for (const GroupChunk& c : chunks) {
    hth_status s;
    switch (c.wb) {
      case 1: s = launch_group_chunk<uint8_t>(L, d, groups, members, host, c, xslots, tarea, parea, vd, passes); break;
      case 2: s = launch_group_chunk<uint16_t>(L, d, groups, members, host, c, xslots, tarea, parea, vd, passes); break;
      case 4: s = launch_group_chunk<uint32_t>(L, d, groups, members, host, c, xslots, tarea, parea, vd, passes); break;
      default: s = launch_group_chunk<uint64_t>(L, d, groups, members, host, c, xslots, tarea, parea, vd, passes); break;
    }
    if (s) return s;
  }
  return HTH_OK;
}

}  // namespace
}  // namespace hth

#include "view.h"

namespace hth {
namespace {

// heavy-row scratch of a plan: a partial count per (role task, chunk of its
// direction), the largest level's worth (levels run one after the other)
size_t heavy_counter_bytes(const hth_kb_s& kb, const Plan& P) {
  size_t most = 0;
  for (const PlanLevel& PL : P.levels) {
    size_t nb = 0;
    for (const RoleTask& t : PL.roles)
      nb += kb.chunk_first[2 * t.role + t.inv + 1] - kb.chunk_first[2 * t.role + t.inv];
    most = std::max(most, nb);
  }
  return align_up(most * 4, 256);
}

// A single role node evaluated by k_push: ∃ρ.A or ¬∃ρ.A over an atomic A with
// fewer than push_pct percent of the individuals, where no row of the
// opposite direction is longer than kPushMaxDeg (a member's row is walked by
// one lane).  Otherwise it is counted per subject (k_role).
constexpr uint32_t kPushMaxDeg = 64;
inline bool pushed(const hth_kb_s& kb, const RoleTask& t) {
  if (!kb.tune.push_pct || t.neg || t.child_row >= kb.d.n_concepts) return false;
  const bool exists = t.lo == 1 && t.hi == 0xFFFFFFFFu, none = t.lo == 0 && t.hi == 0;
  if (!exists && !none) return false;
  if (kb.max_deg[t.inv ? 0 : 1][t.role] > kPushMaxDeg) return false;
  return (uint64_t)kb.concept_pop[t.child_row] * 100 < (uint64_t)kb.tune.push_pct * kb.N;
}

// The shared passes of a level as launched: word counts and T layout set.
// Short-row groups first, so that a launch holds groups of one kind.
std::vector<GroupTask> level_groups(const hth_kb_s& kb, const PlanLevel& PL) {
  std::vector<GroupTask> out;
  for (GroupTask g : PL.groups) {
    g.n_words = kb.n_words[2 * g.role + g.inv];
    g.n_obj_words = kb.n_words[(2 * g.role + g.inv) ^ 1u];
    g.compact = kb.tune.t_compact && 2ull * kb.n_obj[2 * g.role + g.inv] <= kb.N;
    g.short_rows = short_rows(kb, 2 * g.role + g.inv);
    out.push_back(g);
  }
  std::stable_partition(out.begin(), out.end(), [](const GroupTask& g) { return g.short_rows != 0; });
  return out;
}

// partial counts of the segmented chunks of a plan (the largest chunk's worth)
size_t partial_bytes(const hth_kb_s& kb, const Plan& P) {
  size_t most = 0;
  for (const PlanLevel& PL : P.levels) {
    std::vector<GroupTask> gs = level_groups(kb, PL);
    for (const GroupChunk& c : chunk_groups(kb, gs)) most = std::max(most, chunk_partial_bytes(kb, gs, c));
  }
  return align_up(most, 256);
}

// the id sets of a plan's CONTAIN restrictions: one bit per dictionary string each
inline size_t idset_words(uint32_t n_strings) { return align_up(((size_t)n_strings + 63) / 64, 8); }
size_t idset_bytes(const Plan& P) {
  size_t n = 0;
  for (const StrTask& t : P.str) n += t.kind == 1;
  for (const StrTask& t : P.ex_str) n += t.kind == 1;
  return align_up(n * idset_words(P.n_strings) * 8, 256);
}

// bytes of the packed tables plus slots plus T area for a plan
// The T area a plan needs: the most any launch's chunk uses, over its levels
// (the shared passes as launched; never more than t_area_bytes)
size_t plan_t_bytes(const hth_kb_s& kb, const Plan& P) {
  size_t most = 0;
  for (const PlanLevel& PL : P.levels) {
    if (PL.groups.empty()) continue;
    std::vector<GroupTask> gs = level_groups(kb, PL);
    const std::vector<GroupChunk> cs = chunk_groups(kb, gs);
    most = std::max(most, chunks_t_bytes(kb, gs, cs));
  }
  return most;
}

size_t plan_workspace_bytes(const hth_kb_s& kb, const Plan& P) {
  size_t tables = 0;
  auto add = [&](size_t n, size_t each) { tables = align_up(tables, 256) + n * each; };
  // a root covered by its pass has a region of one instruction where instances are written
  size_t n_reg = P.roots.size(), n_cover = 0, n_role = 0, n_grp = 0, n_mem = 0, n_fill = 0, max_groups = 0;
  for (const PlanLevel& PL : P.levels) {
    for (const GroupMember& m : PL.members) n_cover += m.cover != kNone;
    n_reg += PL.mat.size();
    n_role += PL.roles.size();
    n_grp += PL.groups.size();
    n_mem += PL.members.size();
    n_fill += PL.roles.size() + PL.members.size();
    max_groups = std::max(max_groups, PL.groups.size());
  }
  add(P.thr.size(), sizeof(ThrTask));
  add(P.thr.size(), sizeof(ThrGroup));
  add(P.num.size(), sizeof(NumTask));
  add(P.str.size(), sizeof(StrTask));
  add(P.num.size() + P.str.size(), sizeof(ThrGroup));
  add(n_reg + n_cover, sizeof(RegionTask));
  add(n_role, sizeof(RoleTask));
  add(n_role, sizeof(RoleTask));            // pushed role tasks (a subset of the role nodes)
  add(n_grp, sizeof(GroupTask));
  add(n_mem, sizeof(GroupMember));
  add(n_fill, sizeof(FillTask));
  add(P.code.size() + n_cover, sizeof(uint32_t));
  add(9 * n_grp + 8, sizeof(uint32_t));     // XCD slot tables: at most 8 more than groups per chunk
  return align_up(tables, 256) + (size_t)P.n_slots * kb.S * 8 + (max_groups ? plan_t_bytes(kb, P) : 0) +
         heavy_counter_bytes(kb, P) + partial_bytes(kb, P) + idset_bytes(P);
}

std::once_flag g_attr_once;

// A compiled plan laid out for the device: the table blob with its offsets and
// the host side of the launch sequence.  Built once; uploaded into a workspace
// with one copy; launched any number of times (kernels only).
struct Prepared {
  Plan P;
  Blob blob;
  struct LevelAt { size_t mat, role, group, nrole, ngroup, nhb, nhc, push, npush; double fill_bytes; size_t ex; };
  std::vector<LevelAt> at;
  size_t root_at = 0;
  std::vector<std::vector<RoleTask>> lv_roles;
  std::vector<std::vector<RoleTask>> lv_push;
  std::vector<std::vector<GroupTask>> lv_groups;
  std::vector<std::vector<GroupChunk>> lv_chunks;
  size_t n_thr_groups = 0, n_thr_tasks = 0, n_fills = 0;
  size_t o_thr = 0, o_thg = 0, o_reg = 0, o_role = 0, o_grp = 0, o_mem = 0, o_fill = 0, o_code = 0, o_xslot = 0;
  size_t o_push = 0;
  size_t o_num = 0, n_num_blocks = 0;   // numeric concrete-role tasks, their heavy-row blocks
  size_t o_str = 0, n_str_blocks = 0, n_contains = 0;   // string concrete-role tasks
  size_t o_numg = 0, n_numg = 0, o_strg = 0, n_strg = 0;   // their tasks by role (ThrGroup: prop = role)
  size_t o_xnum = 0, o_xstr = 0, n_xcontains = 0, o_xrole = 0;   // tasks at the examples only
  ViewPlan V;                           // the example view: its tables below, its areas in V
  size_t o_vthr = 0, o_vthg = 0, o_vgrp = 0, o_vpass = 0, o_vdir = 0, o_vbase = 0, o_vcopy = 0;
  size_t o_idset = 0;                   // the CONTAIN id sets (workspace offset)
  size_t o_hcnt = 0;   // heavy-row counters (workspace offset)
  size_t o_part = 0;   // partial counts of segmented shared passes (workspace offset)
  size_t tables = 0, need = 0;
  uint32_t n_hyps = 0;
};

void prepare(const hth_kb_s& kb, Plan&& plan, uint32_t n_hyps, Prepared& X) {
  X.P = std::move(plan);
  const Plan& P = X.P;
  X.n_hyps = n_hyps;
  std::vector<RegionTask> regions;
  std::vector<RoleTask> roles;
  std::vector<GroupTask> groups;
  std::vector<GroupMember> members;
  std::vector<FillTask> fills;
  std::vector<RoleTask> pushes;
  std::vector<RoleTask> ex_roles;
  std::vector<uint32_t> xslots;
  const size_t NL = P.levels.size();
  X.at.assign(NL, {});
  X.lv_roles.assign(NL, {});
  X.lv_push.assign(NL, {});
  X.lv_groups.assign(NL, {});
  X.lv_chunks.assign(NL, {});
  for (size_t L = 0; L < NL; ++L) {
    const PlanLevel& PL = P.levels[L];
    X.at[L] = {regions.size(), roles.size(), groups.size(), 0, 0, 0, 0, pushes.size(), 0, 0.0, ex_roles.size()};
    ex_roles.insert(ex_roles.end(), PL.ex_roles.begin(), PL.ex_roles.end());
    regions.insert(regions.end(), PL.mat.begin(), PL.mat.end());
    for (RoleTask t : PL.roles) {
      const uint32_t rd = 2 * t.role + t.inv;
      t.n_words = kb.n_words[rd];
      if (pushed(kb, t)) {
        fills.push_back(FillTask{t.out_row, t.lo == 0 ? 1u : 0u});
        X.at[L].fill_bytes += 8.0 * kb.W;
        pushes.push_back(t);
        X.lv_push[L].push_back(t);
        continue;
      }
      t.hr0 = kb.heavy_first[rd];
      t.hc0 = kb.chunk_first[rd];
      t.h_first = (uint32_t)X.at[L].nhb;
      t.c_first = (uint32_t)X.at[L].nhc;
      X.at[L].nhb += kb.chunk_first[rd + 1] - kb.chunk_first[rd];
      X.at[L].nhc += kb.heavy_first[rd + 1] - kb.heavy_first[rd];
      if (t.n_words < kb.W) {
        fills.push_back(FillTask{t.out_row, t.lo == 0 ? 1u : 0u});
        X.at[L].fill_bytes += 8.0 * (kb.W - t.n_words);
      }
      roles.push_back(t);
      X.lv_roles[L].push_back(t);
    }
    const uint32_t mbase = (uint32_t)members.size();
    for (GroupTask g : level_groups(kb, PL)) {
      if (g.n_words < kb.W) {
        for (uint32_t j = 0; j < g.k; ++j) {
          const uint32_t r = PL.members[g.first + j].out_row;
          if (r == kNone) continue;              // coverage added by the pass, no row
          fills.push_back(FillTask{r, (uint32_t)((g.acc[0] >> j) & 1)});
          X.at[L].fill_bytes += 8.0 * (kb.W - g.n_words);
        }
      }
      g.first += mbase;
      X.lv_groups[L].push_back(g);
    }
    X.lv_chunks[L] = chunk_groups(kb, X.lv_groups[L]);
    for (GroupChunk& c : X.lv_chunks[L])
      if (kb.tune.xcd_local && c.n >= 8) place_on_xcds(kb, X.lv_groups[L], c, xslots);
    groups.insert(groups.end(), X.lv_groups[L].begin(), X.lv_groups[L].end());
    members.insert(members.end(), PL.members.begin(), PL.members.end());
    X.at[L].nrole = roles.size() - X.at[L].role;
    X.at[L].ngroup = groups.size() - X.at[L].group;
    X.at[L].npush = pushes.size() - X.at[L].push;
  }
  X.root_at = regions.size();
  regions.insert(regions.end(), P.roots.begin(), P.roots.end());
  // thresholds grouped by property (at most kThrPerPass per group): one column pass each
  auto by_property = [](const std::vector<ThrTask>& in, std::vector<ThrTask>& tasks) {
    tasks = in;
    std::stable_sort(tasks.begin(), tasks.end(), [](const ThrTask& a, const ThrTask& b) { return a.prop < b.prop; });
    std::vector<ThrGroup> out;
    for (uint32_t i = 0; i < tasks.size(); ++i) {
      if (out.empty() || out.back().prop != tasks[i].prop || out.back().n == kThrPerPass)
        out.push_back(ThrGroup{tasks[i].prop, i, 0, 0});
      out.back().n++;
    }
    return out;
  };
  std::vector<ThrTask> thr_tasks, vthr_tasks;
  const std::vector<ThrGroup> thr_groups = by_property(P.thr, thr_tasks), vthr_groups = by_property(P.vthr, vthr_tasks);
  // the view's shared passes, whatever their levels (every row they read is
  // complete by then), short-row directions first
  ViewPlan& V = X.V;
  V = ViewPlan();
  V.on = P.view;
  if (V.on) {
    const uint32_t gk = std::max<uint32_t>(1, std::min<uint32_t>(kb.tune.group_k, kMaxK)), mbase = (uint32_t)members.size();
    for (int want_short = 1; want_short >= 0; --want_short)
      for (const ViewBucket& q : P.vbuckets)
        if ((int)short_rows(kb, q.rd) == want_short) V.add_passes(kb, q.rd, q.count, gk, mbase + q.first, want_short);
    members.insert(members.end(), P.vmembers.begin(), P.vmembers.end());
    V.chunks = chunk_groups(kb, V.groups);
    for (GroupChunk& c : V.chunks)
      if (kb.tune.xcd_local && c.n >= 8) place_on_xcds(kb, V.groups, c, xslots);
    for (size_t i = 0; i < V.groups.size(); ++i) {
      V.passes[i].t_off = V.groups[i].t_off;
      for (uint32_t j = 0; j < V.passes[i].k; ++j) accept_bits(V.passes[i], members[V.passes[i].first + j], j);
    }
    V.n_rows = P.n_vrows;
    V.n_copies = 2 + (uint32_t)P.vcopies.size();
    V.n_thg = (uint32_t)vthr_groups.size();
    std::vector<ViewCopy> copies{{kPosRow, 0}, {kNegRow, 1}};
    copies.insert(copies.end(), P.vcopies.begin(), P.vcopies.end());
    std::vector<uint64_t> bases;
    for (const ViewDir& v : V.dirs) bases.push_back(v.base);
    X.o_vthr = X.blob.add(vthr_tasks);
    X.o_vthg = X.blob.add(vthr_groups);
    X.o_vgrp = X.blob.add(V.groups);
    X.o_vpass = X.blob.add(V.passes);
    X.o_vdir = X.blob.add(V.dirs);
    X.o_vbase = X.blob.add(bases);
    X.o_vcopy = X.blob.add(copies);
  }
  // tasks of one role share a walk of its values, up to per_walk at a time
  auto by_role = [&](auto& tasks, auto from) {
    std::stable_sort(tasks.begin() + from, tasks.end(), [](const auto& a, const auto& b) { return a.role < b.role; });
    const uint32_t per_walk = value_tasks(kb, tasks.size());
    std::vector<ThrGroup> out;
    for (uint32_t i = 0; i < tasks.size(); ++i) {
      if (out.empty() || out.back().prop != tasks[i].role || out.back().n == per_walk)
        out.push_back(ThrGroup{tasks[i].role, i, 0, 0});
      out.back().n++;
    }
    return out;
  };
  std::vector<NumTask> num(P.num);
  const std::vector<ThrGroup> num_groups = by_role(num, 0);
  for (NumTask& t : num) {
    t.base_lo = (uint32_t)P.num_bounds[t.role];
    t.base_hi = (uint32_t)(P.num_bounds[t.role] >> 32);
    t.h_first = (uint32_t)X.n_num_blocks;
    t.hc0 = P.num_chunk_first[t.role];
    X.n_num_blocks += P.num_chunk_first[t.role + 1] - P.num_chunk_first[t.role];
  }
  X.o_num = X.blob.add(num);
  X.o_numg = X.blob.add(num_groups);
  X.n_numg = num_groups.size();
  // string tasks: CONTAIN first (k_contains takes them as one range), each
  // with its id set; heavy-row blocks numbered in table order
  std::vector<StrTask> str(P.str);
  const ptrdiff_t first_equal =
      std::stable_partition(str.begin(), str.end(), [](const StrTask& t) { return t.kind == 1; }) - str.begin();
  std::stable_sort(str.begin(), str.begin() + first_equal, [](const StrTask& a, const StrTask& b) { return a.role < b.role; });
  const std::vector<ThrGroup> str_groups = by_role(str, first_equal);
  for (StrTask& t : str) {
    t.base_lo = (uint32_t)P.str_bounds[t.role];
    t.base_hi = (uint32_t)(P.str_bounds[t.role] >> 32);
    t.hc0 = P.str_chunk_first[t.role];
    t.h_first = (uint32_t)X.n_str_blocks;
    X.n_str_blocks += P.str_chunk_first[t.role + 1] - P.str_chunk_first[t.role];
    if (t.kind == 1) t.set_word = (uint32_t)(X.n_contains++ * idset_words(P.n_strings));
  }
  X.o_str = X.blob.add(str);
  X.o_strg = X.blob.add(str_groups);
  X.n_strg = str_groups.size();
  std::vector<NumTask> xnum(P.ex_num);
  for (NumTask& t : xnum) {
    t.base_lo = (uint32_t)P.num_bounds[t.role];
    t.base_hi = (uint32_t)(P.num_bounds[t.role] >> 32);
  }
  std::vector<StrTask> xstr(P.ex_str);
  std::stable_partition(xstr.begin(), xstr.end(), [](const StrTask& t) { return t.kind == 1; });
  for (StrTask& t : xstr) {
    t.base_lo = (uint32_t)P.str_bounds[t.role];
    t.base_hi = (uint32_t)(P.str_bounds[t.role] >> 32);
    if (t.kind == 1) t.set_word = (uint32_t)((X.n_contains + X.n_xcontains++) * idset_words(P.n_strings));
  }
  X.o_xnum = X.blob.add(xnum);
  X.o_xstr = X.blob.add(xstr);
  X.o_xrole = X.blob.add(ex_roles);
  X.n_thr_groups = thr_groups.size();
  X.n_thr_tasks = thr_tasks.size();
  X.o_thr = X.blob.add(thr_tasks);
  X.o_thg = X.blob.add(thr_groups);
  X.o_reg = X.blob.add(regions);
  X.o_role = X.blob.add(roles);
  X.o_grp = X.blob.add(groups);
  X.o_mem = X.blob.add(members);
  X.o_fill = X.blob.add(fills);
  X.n_fills = fills.size();
  X.o_code = X.blob.add(P.code);
  X.o_xslot = X.blob.add(xslots);
  X.o_push = X.blob.add(pushes);
  X.tables = align_up(X.blob.bytes.size(), 256);
  size_t t_bytes = 0;   // the T area: the most one chunk of the plan uses
  for (size_t L = 0; L < NL; ++L) t_bytes = std::max(t_bytes, chunks_t_bytes(kb, X.lv_groups[L], X.lv_chunks[L]));
  if (V.on) t_bytes = std::max(t_bytes, chunks_t_bytes(kb, V.groups, V.chunks));
  X.o_hcnt = X.tables + (size_t)P.n_slots * kb.S * 8 + t_bytes;
  X.o_part = X.o_hcnt + heavy_counter_bytes(kb, P);
  size_t part = 0;
  for (size_t L = 0; L < NL; ++L)
    for (const GroupChunk& c : X.lv_chunks[L]) part = std::max(part, chunk_partial_bytes(kb, X.lv_groups[L], c));
  X.o_idset = X.o_part + align_up(part, 256);
  X.need = X.o_idset + idset_bytes(P);
  const size_t rest = X.need;
  V.layout(kb, [&](size_t bytes) {
    const size_t at = X.need;
    X.need = align_up(at + bytes, 256);
    return at;
  });
  V.bytes = X.need - rest;
}

hth_status check_ws(const Prepared& X, const char* ws, size_t ws_bytes) {
  if (X.need > ws_bytes)
    return fail(HTH_E_NOMEM, "workspace too small: need " + std::to_string(X.need) + " bytes, have " +
                                 std::to_string(ws_bytes));
  if (reinterpret_cast<uintptr_t>(ws) % 256) return fail(HTH_E_INVALID, "workspace must be 256-byte aligned");
  return HTH_OK;
}

__global__ void k_zero_u32(uint32_t* __restrict__ p, uint32_t n) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// Small tables travel in the launch: one kernel writes them to the workspace
// and clears the counts, where a copy and a clearing kernel were two
// dispatches one after the other (and the copy, from pageable memory, stops
// the host): 2 to 3 us less of 22 for a hypothesis over 10,000 individuals.
constexpr uint32_t kInline = 224;     // 16-byte units of a launch's arguments
struct InlineTables {
  uint4 v[kInline];
};
__global__ void __launch_bounds__(256)
k_setup(InlineTables t, uint4* __restrict__ ws, uint32_t units, uint32_t* __restrict__ counts, uint32_t nc) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i < units) ws[i] = t.v[i];
  if (i < nc) counts[i] = 0;
}

// k_role<true> stages the child row in up to lds_per_block bytes of LDS
void role_attributes(const hth_kb_s& kb) {
  std::call_once(g_attr_once, [&] {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_role<true>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)kb.lds_per_block);
  });
}

// The kernels of a prepared plan whose tables are in ws: no copies, no
// allocation and no memset (the counts are cleared by a kernel).
hth_status launch_prepared(hth_kb_s& kb, const Prepared& X, char* ws, uint32_t* counts, uint64_t* instances,
                           hipStream_t st, bool cleared = false) {
  role_attributes(kb);
  const Plan& P = X.P;
  const size_t slot_bytes = (size_t)kb.S * 8;
  DevKB d = dev_view(kb);
  d.sets = P.sets;
  d.n_fixed = kb.d.n_concepts + P.n_sets;
  d.num_roff = P.num_roff;
  d.num_val = P.num_val;
  d.num_heavy_rows = P.num_heavy_rows;
  d.num_heavy_chunks = P.num_heavy_chunks;
  d.str_roff = P.str_roff;
  d.str_ids = P.str_ids;
  d.str_heavy_rows = P.str_heavy_rows;
  d.str_heavy_chunks = P.str_heavy_chunks;
  d.dict_off = P.dict_off;
  d.dict_chars = P.dict_chars;
  d.pat_off = P.pat_off;
  d.pat_chars = P.pat_chars;
  d.n_strings = P.n_strings;
  d.idsets = reinterpret_cast<uint64_t*>(ws + X.o_idset);
  d.slots = reinterpret_cast<uint64_t*>(ws + X.tables);
  d.counts = counts;
  d.instances = instances;
  void* tarea = ws + X.tables + (size_t)P.n_slots * slot_bytes;
  const uint32_t nc = 2 * X.n_hyps;
  if (!cleared) {
    hipLaunchKernelGGL(k_zero_u32, dim3((nc + 255) / 256), dim3(256), 0, st, counts, nc);
    HTH_HIP(hipGetLastError());
  }
  const ThrTask* thr = reinterpret_cast<const ThrTask*>(ws + X.o_thr);
  const ThrGroup* thg = reinterpret_cast<const ThrGroup*>(ws + X.o_thg);
  const RegionTask* reg = reinterpret_cast<const RegionTask*>(ws + X.o_reg);
  const RoleTask* rol = reinterpret_cast<const RoleTask*>(ws + X.o_role);
  const GroupTask* grp = reinterpret_cast<const GroupTask*>(ws + X.o_grp);
  const GroupMember* mem = reinterpret_cast<const GroupMember*>(ws + X.o_mem);
  const FillTask* fil = reinterpret_cast<const FillTask*>(ws + X.o_fill);
  const uint32_t* code = reinterpret_cast<const uint32_t*>(ws + X.o_code);
  Launcher Lc{kb, st};
  if (!P.num.empty()) {
    const uint32_t n = (uint32_t)P.num.size();
    const NumTask* nt = reinterpret_cast<const NumTask*>(ws + X.o_num);
    const uint32_t ng = (uint32_t)X.n_numg, bpt = value_blocks(kb, ng);
    const ThrGroup* gr = reinterpret_cast<const ThrGroup*>(ws + X.o_numg);
    double bytes = 0;   // per task: the role's offsets and values once, its row out
    for (const NumTask& t : P.num)
      bytes += 4.0 * (kb.N + 1) + 4.0 * (double)(P.num_bounds[t.role + 1] - P.num_bounds[t.role]) + 8.0 * kb.W;
    hth_status s = split_launch(Lc, HTH_K_THRESHOLD, bytes, ng, bpt, 256, [&](uint32_t i0, uint32_t, uint32_t blocks) {
      hipLaunchKernelGGL(k_numrole, dim3(blocks), dim3(256), 0, st, d, gr + i0, nt, bpt);
    });
    if (s) return s;
    if (X.n_num_blocks) {
      s = split_launch(Lc, HTH_K_THRESHOLD, 0.0, X.n_num_blocks, 1, 256, [&](uint32_t b0, uint32_t, uint32_t blocks) {
        hipLaunchKernelGGL(k_numrole_heavy, dim3(blocks), dim3(256), 0, st, d, nt, n, b0);
      });
      if (s) return s;
    }
  }
  // the id sets: the dictionary strings holding each pattern
  auto contains = [&](const StrTask* sk, size_t n) -> hth_status {
    if (!n) return HTH_OK;
    const uint32_t tiles = std::max<uint32_t>(1, (P.n_strings + 255) / 256);
    return split_launch(Lc, HTH_K_THRESHOLD, 0.0, n, tiles, 256, [&](uint32_t i0, uint32_t, uint32_t blocks) {
      hipLaunchKernelGGL(k_contains, dim3(blocks), dim3(256), 0, st, d, sk + i0, tiles);
    });
  };
  // tasks at the examples: their rows' offsets and about as many values of each as a row has
  const uint32_t xtiles = (kb.W + kExWords - 1) / kExWords;
  auto ex_bytes = [&](double values) { return kb.ex_hint * (8.0 + 4.0 * values / kb.N) + 8.0 * kb.W; };
  if (!P.ex_num.empty()) {
    const NumTask* nt = reinterpret_cast<const NumTask*>(ws + X.o_xnum);
    double bytes = 0;
    for (const NumTask& t : P.ex_num) bytes += ex_bytes((double)(P.num_bounds[t.role + 1] - P.num_bounds[t.role]));
    hth_status s = split_launch(Lc, HTH_K_THRESHOLD, bytes, P.ex_num.size(), xtiles, 64,
                                [&](uint32_t i0, uint32_t, uint32_t blocks) {
                                  hipLaunchKernelGGL(k_numrole_ex, dim3(blocks), dim3(64), 0, st, d, nt + i0, xtiles);
                                });
    if (s) return s;
  }
  if (!P.ex_str.empty()) {
    const StrTask* sk = reinterpret_cast<const StrTask*>(ws + X.o_xstr);
    hth_status s = contains(sk, X.n_xcontains);
    if (s) return s;
    double bytes = 0;
    for (const StrTask& t : P.ex_str) bytes += ex_bytes((double)(P.str_bounds[t.role + 1] - P.str_bounds[t.role]));
    s = split_launch(Lc, HTH_K_THRESHOLD, bytes, P.ex_str.size(), xtiles, 64,
                     [&](uint32_t i0, uint32_t, uint32_t blocks) {
                       hipLaunchKernelGGL(k_strrole_ex, dim3(blocks), dim3(64), 0, st, d, sk + i0, xtiles);
                     });
    if (s) return s;
  }
  if (!P.str.empty()) {
    const uint32_t n = (uint32_t)P.str.size();
    const StrTask* sk = reinterpret_cast<const StrTask*>(ws + X.o_str);
    hth_status s = contains(sk, X.n_contains);
    if (s) return s;
    const uint32_t ng = (uint32_t)X.n_strg, bpt = value_blocks(kb, ng);
    const ThrGroup* gr = reinterpret_cast<const ThrGroup*>(ws + X.o_strg);
    double bytes = 0;   // per task: the role's offsets and ids once, its row out
    for (const StrTask& t : P.str)
      bytes += 4.0 * (kb.N + 1) + 4.0 * (double)(P.str_bounds[t.role + 1] - P.str_bounds[t.role]) + 8.0 * kb.W;
    s = split_launch(Lc, HTH_K_THRESHOLD, bytes, ng, bpt, 256, [&](uint32_t i0, uint32_t, uint32_t blocks) {
      hipLaunchKernelGGL(k_strrole, dim3(blocks), dim3(256), 0, st, d, gr + i0, sk, bpt);
    });
    if (s) return s;
    if (X.n_str_blocks) {
      s = split_launch(Lc, HTH_K_THRESHOLD, 0.0, X.n_str_blocks, 1, 256, [&](uint32_t b0, uint32_t, uint32_t blocks) {
        hipLaunchKernelGGL(k_strrole_heavy, dim3(blocks), dim3(256), 0, st, d, sk, n, b0);
      });
      if (s) return s;
    }
  }
  if (X.n_thr_groups) {
    const uint32_t n = (uint32_t)X.n_thr_groups, bpt = threshold_blocks(kb, n, kb.W);
    std::vector<uint32_t> props;
    for (const ThrTask& t : P.thr) props.push_back(t.prop);
    std::sort(props.begin(), props.end());
    const double bytes = 4.0 * kb.N * (double)(std::unique(props.begin(), props.end()) - props.begin());
    hth_status s = split_launch(Lc, HTH_K_THRESHOLD, bytes, n, bpt, 256, [&](uint32_t i0, uint32_t, uint32_t blocks) {
      hipLaunchKernelGGL(k_threshold<false>, dim3(blocks), dim3(256), 0, st, d, thg + i0, thr, bpt, nullptr);
    });
    if (s) return s;
  }
  double fill_bytes = 0;
  for (const Prepared::LevelAt& at : X.at) fill_bytes += at.fill_bytes;
  hth_status sf = launch_fills(Lc, d, fil, X.n_fills, fill_bytes);
  if (sf) return sf;
  for (size_t L = 0; L < P.levels.size(); ++L) {
    const PlanLevel& PL = P.levels[L];
    const Prepared::LevelAt& at = X.at[L];
    Lc.csr_seen.clear();
    hth_status s = launch_regions(Lc, d, reg + at.mat, code, PL.mat, P.code);
    if (s) return s;
    if (at.npush) {   // after the fills that set their rows to all zeros / all ones
      const uint32_t n = (uint32_t)at.npush, tiles = (kb.W + 3) / 4;
      const RoleTask* pt = reinterpret_cast<const RoleTask*>(ws + X.o_push) + at.push;
      double bytes = 0;
      for (const RoleTask& t : X.lv_push[L])
        bytes += (double)kb.W * 8 * 2 + 8.0 * kb.concept_pop[t.child_row] +
                 4.0 * kb.concept_pop[t.child_row] *
                     ((double)(kb.role_base[t.role + 1] - kb.role_base[t.role]) / kb.N);
      s = split_launch(Lc, HTH_K_ROLE, bytes, n, tiles, 256, [&](uint32_t i0, uint32_t, uint32_t blocks) {
        hipLaunchKernelGGL(k_push, dim3(blocks), dim3(256), 0, st, d, pt + i0, tiles);
      });
      if (s) return s;
    }
    if (!PL.ex_roles.empty()) {
      const RoleTask* xr = reinterpret_cast<const RoleTask*>(ws + X.o_xrole) + at.ex;
      double bytes = 0;
      for (const RoleTask& t : PL.ex_roles) bytes += ex_bytes((double)(kb.role_base[t.role + 1] - kb.role_base[t.role]));
      s = split_launch(Lc, HTH_K_ROLE, bytes, PL.ex_roles.size(), xtiles, 64,
                       [&](uint32_t i0, uint32_t, uint32_t blocks) {
                         hipLaunchKernelGGL(k_role_ex, dim3(blocks), dim3(64), 0, st, d, xr + i0, xtiles);
                       });
      if (s) return s;
    }
    s = launch_roles(Lc, d, rol + at.role, X.lv_roles[L]);
    if (s) return s;
    if (at.nhc) {   // heavy rows: chunk partials, then the rows' bits
      uint32_t* partial = reinterpret_cast<uint32_t*>(ws + X.o_hcnt);
      const uint32_t nt = (uint32_t)at.nrole;
      s = split_launch(Lc, HTH_K_ROLE, 0.0, at.nhb, 1, 256, [&](uint32_t b0, uint32_t, uint32_t blocks) {
        hipLaunchKernelGGL(k_role_heavy, dim3(blocks), dim3(256), 0, st, d, rol + at.role, nt, b0, partial);
      });
      if (s) return s;
      s = split_launch(Lc, HTH_K_ROLE, 0.0, at.nhc, 1, 256, [&](uint32_t i0, uint32_t, uint32_t blocks) {
        hipLaunchKernelGGL(k_role_heavy_fix, dim3(blocks), dim3(256), 0, st, d, rol + at.role, nt, i0, partial);
      });
      if (s) return s;
    }
    s = launch_groups(Lc, d, grp + at.group, mem, X.lv_groups[L], X.lv_chunks[L],
                      reinterpret_cast<const uint32_t*>(ws + X.o_xslot), tarea, ws + X.o_part);
    if (s) return s;
  }
  if (X.V.on) {   // every full row is complete: what is left is done at the examples
    hth_status s = launch_view(Lc, d, X.V, ws, reinterpret_cast<const ViewDir*>(ws + X.o_vdir),
                               reinterpret_cast<const uint64_t*>(ws + X.o_vbase),
                               reinterpret_cast<const ViewCopy*>(ws + X.o_vcopy), 0,
                               reinterpret_cast<const ThrGroup*>(ws + X.o_vthg),
                               reinterpret_cast<const ThrTask*>(ws + X.o_vthr),
                               reinterpret_cast<const GroupTask*>(ws + X.o_vgrp),
                               reinterpret_cast<const GroupTask*>(ws + X.o_vpass), mem,
                               reinterpret_cast<const uint32_t*>(ws + X.o_xslot), tarea, &d);
    if (s) return s;
  }
  return launch_regions(Lc, d, reg + X.root_at, code, P.roots, P.code);
}

// A prepared plan's tables into the workspace, then its kernels.
hth_status upload_and_launch(hth_kb_s& kb, const Prepared& X, char* ws, uint32_t* counts, uint64_t* instances,
                             hipStream_t st) {
  const size_t n = X.blob.bytes.size();
  if (n > sizeof(InlineTables)) {
    HTH_HIP(hipMemcpyAsync(ws, X.blob.bytes.data(), n, hipMemcpyHostToDevice, st));
    return launch_prepared(kb, X, ws, counts, instances, st);
  }
  InlineTables t;
  std::memcpy(t.v, X.blob.bytes.data(), n);
  const uint32_t units = (uint32_t)((n + 15) / 16), nc = 2 * X.n_hyps;
  hipLaunchKernelGGL(k_setup, dim3((std::max(units, nc) + 255) / 256), dim3(256), 0, st, t,
                     reinterpret_cast<uint4*>(ws), units, counts, nc);
  HTH_HIP(hipGetLastError());
  return launch_prepared(kb, X, ws, counts, instances, st, true);
}

hth_status run_prepared(hth_kb_s& kb, const Prepared& X, char* ws, size_t ws_bytes, uint32_t* counts,
                        uint64_t* instances, hipStream_t st) {
  hth_status s = check_ws(X, ws, ws_bytes);
  if (s) return s;
  return upload_and_launch(kb, X, ws, counts, instances, st);
}

hth_status run_plan(hth_kb_s& kb, Plan&& P, char* ws, size_t ws_bytes, uint32_t* counts, uint32_t n_hyps,
                    uint64_t* instances, hipStream_t st) {
  Prepared X;
  prepare(kb, std::move(P), n_hyps, X);
  return run_prepared(kb, X, ws, ws_bytes, counts, instances, st);
}

// Whether a hypothesis evaluated alone takes its restrictions at the examples:
// from four times the individuals on and up to an eighth of them, since there is
// no pass to share.  Microseconds at the examples / over everyone: 6 % examples,
// 8 hypotheses over 131,072 individuals 188 / 173, over 400,000 221 / 222, 16 over
// 1M 542 / 790; 16 over 400,000, 10 % 496 / 534, 20 % 549 / 530; over 1M, 10 %
// 801 / 842, 20 % 926 / 840.
bool one_at_examples(const hth_kb_s& kb, const PlanOptions& opt) {
  return !opt.instances && kb.N / 4 >= kb.view_min && (uint64_t)kb.ex_hint * 8 <= kb.N && view_wanted(kb);
}

// Whether a host-planned batch evaluates at the examples what no filler reads.
bool batch_view(const hth_kb_s& kb, const PlanOptions& opt) {
  return !opt.instances && opt.group_min != 0xFFFFFFFFu && view_wanted(kb);
}

}  // namespace
}  // namespace hth

using namespace hth;

extern "C" hth_status hth_workspace_bytes(hth_kb kb, uint32_t max_nodes, uint32_t max_hyps,
                                          size_t* bytes) {
  if (!kb || !bytes) return fail(HTH_E_INVALID, "NULL argument");
  if (max_hyps == 0 || max_nodes < max_hyps) return fail(HTH_E_RANGE, "need max_nodes >= max_hyps >= 1");
  // a chunk's T rows: at most t_area_bytes, and at most one row of the widest
  // T word per individual for each of the plan's nodes
  const size_t t_bound = std::min(t_area_bytes(*kb), (size_t)max_nodes * align_up(kb->N, 64) * 8);
  *bytes = align_up(table_bound(max_nodes, max_hyps), 256) + (size_t)(max_nodes + 2) * kb->S * 8 +
           t_bound + align_up((size_t)(max_nodes + 2) * kb->chunk_most * 4, 256) +
           align_up((size_t)(max_nodes + 2) * idset_words(kb->n_strings) * 8, 256);
  return HTH_OK;
}

extern "C" hth_status hth_eval_one(hth_kb kb, const hth_node* nodes, uint32_t n_nodes,
                                   const uint32_t* children, uint32_t n_children, void* ws,
                                   size_t ws_bytes, uint64_t* d_instances, uint32_t* d_counts,
                                   void* stream) {
  if (!kb || !nodes || !ws || !d_counts) return fail(HTH_E_INVALID, "NULL argument");
  if (n_children && !children) return fail(HTH_E_INVALID, "children is NULL");
  uint32_t offs[2] = {0, n_nodes};
  PlanOptions opt;
  opt.instances = d_instances != nullptr;
  opt.examples = one_at_examples(*kb, opt);
  Plan P;
  hth_status s = compile_plan(*kb, nodes, offs, 1, children, n_children, opt, P);
  if (s) return s;
  std::lock_guard<std::mutex> g(kb->mu);
  return run_plan(*kb, std::move(P), static_cast<char*>(ws), ws_bytes, d_counts, 1, d_instances,
                  static_cast<hipStream_t>(stream));
}

// The workspace of hth_eval_one_noalloc: a fixed array in the code object's
// device data, one copy per GPU, held until the process ends.  Host code
// never passes the array's name to a kernel or a copy (on the host it is only
// a stand-in); it uses the device address hipGetSymbolAddress gives for the
// GPU the call runs on.
namespace hth {
namespace {
__device__ __align__(256) uint64_t scratch[HTH_NOALLOC_SCRATCH_BYTES / 8];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
char* g_scratch[kMaxDevices] = {};

// The scratch array's address on `device`, looked up once per device with
// that device current (the caller's current device is restored).
hth_status scratch_on(int device, char** out) {
  if (device < 0 || device >= kMaxDevices) return fail(HTH_E_UNSUPPORTED, "device index beyond 63");
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (!g_scratch[device]) {
    int cur = 0;
    HTH_HIP(hipGetDevice(&cur));
    if (cur != device) HTH_HIP(hipSetDevice(device));
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (cur != device) HTH_HIP(hipSetDevice(cur));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    if (!p || reinterpret_cast<uintptr_t>(p) % 256) return fail(HTH_E_DEVICE, "scratch address not 256-byte aligned");
    g_scratch[device] = static_cast<char*>(p);
  }
  *out = g_scratch[device];
  return HTH_OK;
}
}  // namespace
}  // namespace hth

extern "C" hth_status hth_eval_one_noalloc(hth_kb kb, const hth_node* nodes, uint32_t n_nodes,
                                           const uint32_t* children, uint32_t n_children,
                                           uint64_t* d_instances, uint32_t* d_counts, void* stream) {
  if (!kb || !nodes || !d_counts) return fail(HTH_E_INVALID, "NULL argument");
  if (n_children && !children) return fail(HTH_E_INVALID, "children is NULL");
  uint32_t offs[2] = {0, n_nodes};
  PlanOptions opt;
  opt.instances = d_instances != nullptr;
  opt.examples = one_at_examples(*kb, opt);
  Plan P;
  hth_status s = compile_plan(*kb, nodes, offs, 1, children, n_children, opt, P);
  if (s) return s;
  char* ws = nullptr;
  s = scratch_on(kb->device, &ws);
  if (s) return s;
  std::lock_guard<std::mutex> g(kb->mu);
  Prepared X;
  prepare(*kb, std::move(P), 1, X);
  if (X.need > (size_t)HTH_NOALLOC_SCRATCH_BYTES)
    return fail(HTH_E_NOMEM, "hth_eval_one_noalloc: this hypothesis needs " + std::to_string(X.need) +
                                 " bytes of workspace; the fixed scratch holds " +
                                 std::to_string((size_t)HTH_NOALLOC_SCRATCH_BYTES) +
                                 " (use hth_eval_one with a caller workspace)");
  const hipStream_t st = static_cast<hipStream_t>(stream);
  return upload_and_launch(*kb, X, ws, d_counts, d_instances, st);
}

namespace {
hth_status eval_batch_impl(hth_kb kb, const hth_node* nodes, const uint32_t* hyp_node_offsets,
                           uint32_t n_hyps, const uint32_t* children, uint32_t n_children, void* ws,
                           size_t ws_bytes, uint64_t* d_sets, uint32_t* d_counts, void* stream) {
  if (!kb || !nodes || !hyp_node_offsets || !ws || !d_counts)
    return fail(HTH_E_INVALID, "NULL argument");
  if (n_children && !children) return fail(HTH_E_INVALID, "children is NULL");
  if (n_hyps == 0) return HTH_OK;
  if (hyp_node_offsets[0] != 0) return fail(HTH_E_INVALID, "hyp_node_offsets[0] must be 0");
  PlanOptions opt;
  opt.group_min = kb->tune.group_min ? kb->tune.group_min : 0xFFFFFFFFu;
  opt.group_k = kb->tune.group_k;
  opt.instances = d_sets != nullptr;
  opt.examples = opt.view = batch_view(*kb, opt);
  for (;;) {
    Plan P;
    hth_status s = compile_plan(*kb, nodes, hyp_node_offsets, n_hyps, children, n_children, opt, P);
    if (s) return s;
    std::lock_guard<std::mutex> g(kb->mu);
    Prepared X;
    prepare(*kb, std::move(P), n_hyps, X);
    if (opt.view && (X.need > ws_bytes || X.V.too_large(*kb, X.need))) {   // no room for the view: every row in full
      opt.examples = opt.view = false;
      continue;
    }
    return run_prepared(*kb, X, static_cast<char*>(ws), ws_bytes, d_counts, d_sets, static_cast<hipStream_t>(stream));
  }
}
}  // namespace

extern "C" hth_status hth_eval_batch(hth_kb kb, const hth_node* nodes, const uint32_t* hyp_node_offsets,
                                     uint32_t n_hyps, const uint32_t* children, uint32_t n_children,
                                     void* ws, size_t ws_bytes, uint32_t* d_counts, void* stream) {
  return eval_batch_impl(kb, nodes, hyp_node_offsets, n_hyps, children, n_children, ws, ws_bytes,
                         nullptr, d_counts, stream);
}

extern "C" hth_status hth_eval_batch_sets(hth_kb kb, const hth_node* nodes,
                                          const uint32_t* hyp_node_offsets, uint32_t n_hyps,
                                          const uint32_t* children, uint32_t n_children, void* ws,
                                          size_t ws_bytes, uint64_t* d_sets, uint32_t* d_counts,
                                          void* stream) {
  if (!d_sets) return fail(HTH_E_INVALID, "d_sets is NULL");
  return eval_batch_impl(kb, nodes, hyp_node_offsets, n_hyps, children, n_children, ws, ws_bytes,
                         d_sets, d_counts, stream);
}

// The cross-batch subexpression cache (hth_cache_*): the library's LRU over
// the caller's rows, registered as the kb's set table.
struct hth_cache_s {
  hth_kb kb = nullptr;
  hth::SubexprCache* c = nullptr;
  uint64_t* rows = nullptr;
  uint32_t n_rows = 0;
  std::mutex mu;   // one cached evaluation at a time: compile, admit, launch
  ~hth_cache_s() { hth::cache_delete(c); }
};

extern "C" hth_status hth_cache_create(hth_kb kb, uint64_t* d_rows, uint32_t n_rows, hth_cache* out) {
  if (!kb || !d_rows || !out) return fail(HTH_E_INVALID, "NULL argument");
  if (n_rows == 0 || n_rows >= (1u << 24)) return fail(HTH_E_RANGE, "a cache holds 1 .. 2^24 - 1 rows");
  if (reinterpret_cast<uintptr_t>(d_rows) % 64) return fail(HTH_E_INVALID, "cache rows must be 64-byte aligned");
  hth_cache_s* c = new (std::nothrow) hth_cache_s();
  if (!c) return fail(HTH_E_NOMEM, "host allocation failed");
  c->c = cache_new(n_rows);
  if (!c->c) {
    delete c;
    return fail(HTH_E_NOMEM, "host allocation failed");
  }
  c->kb = kb;
  c->rows = d_rows;
  c->n_rows = n_rows;
  std::lock_guard<std::mutex> g(kb->mu);
  kb->sets = d_rows;
  kb->n_sets = n_rows;
  *out = c;
  return HTH_OK;
}

extern "C" hth_status hth_cache_destroy(hth_cache cache) {
  if (!cache) return HTH_OK;
  {
    std::lock_guard<std::mutex> g(cache->kb->mu);
    if (cache->kb->sets == cache->rows) {
      cache->kb->sets = nullptr;
      cache->kb->n_sets = 0;
    }
  }
  delete cache;
  return HTH_OK;
}

extern "C" hth_status hth_cache_stats(hth_cache cache, hth_cache_info* out) {
  if (!cache || !out) return fail(HTH_E_INVALID, "NULL argument");
  std::lock_guard<std::mutex> g(cache->mu);
  const CacheCounters k = cache_counters(cache->c);
  *out = hth_cache_info{k.hits, k.misses, k.admitted, k.evictions, k.batches, k.entries, k.rows};
  return HTH_OK;
}

extern "C" hth_status hth_eval_batch_cached(hth_kb kb, hth_cache cache, const hth_node* nodes,
                                            const uint32_t* hyp_node_offsets, uint32_t n_hyps,
                                            const uint32_t* children, uint32_t n_children, void* ws,
                                            size_t ws_bytes, uint32_t* d_counts, void* stream) {
  if (!kb || !cache || !nodes || !hyp_node_offsets || !ws || !d_counts) return fail(HTH_E_INVALID, "NULL argument");
  if (cache->kb != kb) return fail(HTH_E_INVALID, "the cache belongs to another kb");
  if (n_children && !children) return fail(HTH_E_INVALID, "children is NULL");
  if (n_hyps == 0) return HTH_OK;
  if (hyp_node_offsets[0] != 0) return fail(HTH_E_INVALID, "hyp_node_offsets[0] must be 0");
  std::lock_guard<std::mutex> gc(cache->mu);
  {
    std::lock_guard<std::mutex> g(kb->mu);
    if (kb->sets != cache->rows) return fail(HTH_E_STATE, "another set table replaced the cache's rows");
  }
  for (uint32_t h = 0; h < n_hyps; ++h)
    for (uint32_t i = hyp_node_offsets[h]; i < hyp_node_offsets[h + 1]; ++i)
      if (nodes[i].op == HTH_SET)
        return fail(HTH_E_UNSUPPORTED, "set-table leaves are the cache's own rows in a cached evaluation");
  PlanOptions opt;
  opt.group_min = kb->tune.group_min ? kb->tune.group_min : 0xFFFFFFFFu;
  opt.group_k = kb->tune.group_k;
  opt.cache = cache->c;
  Plan P;
  hth_status s = compile_plan(*kb, nodes, hyp_node_offsets, n_hyps, children, n_children, opt, P);
  if (s) {
    cache_rollback(cache->c);
    return s;
  }
  std::lock_guard<std::mutex> g(kb->mu);
  s = run_plan(*kb, std::move(P), static_cast<char*>(ws), ws_bytes, d_counts, n_hyps, nullptr,
               static_cast<hipStream_t>(stream));
  if (s) cache_rollback(cache->c);
  return s;
}

// A compiled batch kept for repeated launches (hth_plan_*).
struct hth_plan_s {
  hth_kb kb = nullptr;
  hth::Prepared X;
  hth_kb_s::Tuning tune;   // the schedule the tables were laid out for
  // A workspace without room for the example view gets the plan without it,
  // compiled when the first such workspace is uploaded: those it was uploaded to.
  std::function<hth_status(hth::Plan&)> without_view;
  std::unique_ptr<hth::Prepared> G;
  std::set<const void*> general;
};

namespace hth {
// The kb's schedule replaced by a plan's for the duration of its launch (the
// caller holds kb.mu): the launch sizes and the workspace areas it was laid
// out with stay consistent whatever hth_kb_set_tuning did since.
struct TuneScope {
  hth_kb_s& kb;
  hth_kb_s::Tuning saved;
  TuneScope(hth_kb_s& k, const hth_kb_s::Tuning& t) : kb(k), saved(k.tune) { kb.tune = t; }
  ~TuneScope() { kb.tune = saved; }
};
}  // namespace hth

extern "C" hth_status hth_plan_create(hth_kb kb, const hth_node* nodes, const uint32_t* hyp_node_offsets,
                                      uint32_t n_hyps, const uint32_t* children, uint32_t n_children,
                                      hth_plan* out, size_t* ws_bytes) {
  if (!kb || !nodes || !hyp_node_offsets || !out || !ws_bytes) return fail(HTH_E_INVALID, "NULL argument");
  if (n_children && !children) return fail(HTH_E_INVALID, "children is NULL");
  if (n_hyps == 0) return fail(HTH_E_RANGE, "a plan needs at least one hypothesis");
  if (hyp_node_offsets[0] != 0) return fail(HTH_E_INVALID, "hyp_node_offsets[0] must be 0");
  PlanOptions opt;
  opt.group_min = kb->tune.group_min ? kb->tune.group_min : 0xFFFFFFFFu;
  opt.group_k = kb->tune.group_k;
  opt.examples = opt.view = batch_view(*kb, opt);
  Plan P;
  std::function<hth_status(Plan&)> later;
  hth_status s = compile_plan(*kb, nodes, hyp_node_offsets, n_hyps, children, n_children, opt, P, nullptr,
                              opt.view ? &later : nullptr);
  if (s) return s;
  std::unique_ptr<hth_plan_s> pl(new (std::nothrow) hth_plan_s());
  if (!pl) return fail(HTH_E_NOMEM, "host allocation failed");
  pl->kb = kb;
  pl->tune = kb->tune;
  prepare(*kb, std::move(P), n_hyps, pl->X);
  if (pl->X.V.too_large(*kb, pl->X.need)) {
    s = later(P);
    if (s) return s;
    pl->X = Prepared();
    prepare(*kb, std::move(P), n_hyps, pl->X);
  } else if (pl->X.V.on) {
    pl->without_view = std::move(later);
  }
  *ws_bytes = pl->X.need;
  *out = pl.release();
  return HTH_OK;
}

extern "C" hth_status hth_plan_upload(hth_plan plan, void* ws, size_t ws_bytes, void* stream) {
  if (!plan || !ws) return fail(HTH_E_INVALID, "NULL argument");
  std::lock_guard<std::mutex> g(plan->kb->mu);
  const bool general = plan->X.need > ws_bytes && plan->without_view;
  if (general && !plan->G) {
    TuneScope ts(*plan->kb, plan->tune);
    Plan P;
    hth_status s = plan->without_view(P);
    if (s) return s;
    auto G = std::make_unique<Prepared>();
    prepare(*plan->kb, std::move(P), plan->X.n_hyps, *G);
    plan->G = std::move(G);
  }
  const Prepared& X = general ? *plan->G : plan->X;
  hth_status s = check_ws(X, static_cast<char*>(ws), ws_bytes);
  if (s) return s;
  HTH_HIP(hipMemcpyAsync(ws, X.blob.bytes.data(), X.blob.bytes.size(), hipMemcpyHostToDevice,
                         static_cast<hipStream_t>(stream)));
  if (general) plan->general.insert(ws);
  else plan->general.erase(ws);
  return HTH_OK;
}

extern "C" hth_status hth_plan_launch(hth_plan plan, void* ws, size_t ws_bytes, uint32_t* d_counts,
                                      void* stream) {
  if (!plan || !ws || !d_counts) return fail(HTH_E_INVALID, "NULL argument");
  std::lock_guard<std::mutex> g(plan->kb->mu);
  const Prepared& X = plan->general.count(ws) ? *plan->G : plan->X;   // as uploaded there
  hth_status s = check_ws(X, static_cast<char*>(ws), ws_bytes);
  if (s) return s;
  TuneScope ts(*plan->kb, plan->tune);
  return launch_prepared(*plan->kb, X, static_cast<char*>(ws), d_counts, nullptr, static_cast<hipStream_t>(stream));
}

extern "C" hth_status hth_plan_destroy(hth_plan plan) {
  delete plan;
  return HTH_OK;
}

extern "C" hth_status hth_batch_workspace_bytes(hth_kb kb, const hth_node* nodes,
                                                 const uint32_t* hyp_node_offsets, uint32_t n_hyps,
                                                 const uint32_t* children, uint32_t n_children,
                                                 size_t* bytes) {
  if (!kb || !nodes || !hyp_node_offsets || !bytes) return fail(HTH_E_INVALID, "NULL argument");
  if (n_children && !children) return fail(HTH_E_INVALID, "children is NULL");
  if (n_hyps == 0) {
    *bytes = 0;
    return HTH_OK;
  }
  PlanOptions opt;
  opt.group_min = kb->tune.group_min ? kb->tune.group_min : 0xFFFFFFFFu;
  opt.group_k = kb->tune.group_k;
  opt.examples = opt.view = batch_view(*kb, opt);
  Plan P, general;
  hth_status s = compile_plan(*kb, nodes, hyp_node_offsets, n_hyps, children, n_children, opt, P,
                              opt.view ? &general : nullptr);
  if (s) return s;
  *bytes = plan_workspace_bytes(*kb, opt.view ? general : P) + 4096;
  if (opt.view) {
    Prepared X;
    prepare(*kb, std::move(P), n_hyps, X);
    if (!X.V.too_large(*kb, X.need)) *bytes = std::max(*bytes, X.need);
  }
  return HTH_OK;
}

extern "C" hth_status hth_profile_begin(hth_kb kb) {
  if (!kb) return fail(HTH_E_INVALID, "kb is NULL");
  std::lock_guard<std::mutex> g(kb->mu);
  if (kb->prof) return fail(HTH_E_STATE, "profiling already active");
  kb->prof = true;
  kb->prof_recs.clear();
  return HTH_OK;
}

extern "C" hth_status hth_profile_end(hth_kb kb, hth_prof_entry* out) {
  if (!kb || !out) return fail(HTH_E_INVALID, "NULL argument");
  std::lock_guard<std::mutex> g(kb->mu);
  if (!kb->prof) return fail(HTH_E_STATE, "profiling not active");
  kb->prof = false;
  for (int k = 0; k < HTH_K_NUM; ++k) out[k] = hth_prof_entry{0, 0.0, 0.0};
  hth_status st = HTH_OK;
  for (auto& r : kb->prof_recs) {
    float ms = 0;
    hipError_t e = hipEventSynchronize(r.b);
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, r.a, r.b);
    if (e != hipSuccess && st == HTH_OK) st = hip_fail(e, "hipEventElapsedTime");
    out[r.kind].launches += 1;
    out[r.kind].ms += ms;
    out[r.kind].bytes += r.bytes;
    kb->event_pool.push_back(r.a);
    kb->event_pool.push_back(r.b);
  }
  kb->prof_recs.clear();
  return st;
}

#include "devplan.h"
