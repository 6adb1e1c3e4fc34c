// Knowledge-base loading: validation on the device and the derived layouts
// (32-bit per-role row offsets in both directions and the inverse-role CSR).
//
// The paper keeps role assertions as (subject, object) rows grouped per role
// with an offset table (Section 3.1) and obtains inverse restrictions by
// swapping subjects and objects (end of Section 3.2.2).  Here the forward
// assertions arrive as a CSR per role and the inverse is its exact transpose,
// built once at load time so that both directions are scanned row-parallel.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>

#include "kb_handle.h"

namespace hth {

static thread_local std::string g_err;

void set_error(const std::string& msg) { g_err = msg; }
hth_status fail(hth_status code, const std::string& msg) {
  g_err = msg;
  return code;
}
hth_status hip_fail(hipError_t e, const char* what) {
  g_err = std::string(what) + ": " + hipGetErrorString(e);
  return HTH_E_DEVICE;
}

enum : uint32_t {
  F_NONMONO = 1,   // offsets decrease or leave the role's range
  F_TARGET = 2,    // target outside [0, N)
  F_ORDER = 4,     // targets not strictly increasing inside a row
  F_PAD = 8,       // a padding bit is set
};

constexpr int kScanThreads = 1024;

__global__ void k_gather_bases(const int64_t* __restrict__ off, uint32_t R, uint32_t N,
                               uint64_t* __restrict__ base) {
  uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < R) base[r] = (uint64_t)off[(size_t)r * (N + 1)];
  if (r == R - 1) base[R] = (uint64_t)off[(size_t)r * (N + 1) + N];
}

// Members of each row (one block per row): the plan's push/pull choice.
__global__ void __launch_bounds__(256)
k_row_pop(const uint64_t* __restrict__ rows, uint32_t W, uint32_t S, uint32_t* __restrict__ out) {
  __shared__ uint32_t part[4];
  const uint64_t* p = rows + (size_t)blockIdx.x * S;
  uint32_t c = 0;
  for (uint32_t w = threadIdx.x; w < W; w += 256) c += (uint32_t)__popcll(p[w]);
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) c += __shfl_xor(c, d, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) out[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

// The number of examples, positive or negative.
__global__ void __launch_bounds__(256)
k_count_examples(const uint64_t* __restrict__ pos, const uint64_t* __restrict__ neg, uint32_t W,
                 uint32_t* __restrict__ out) {
  uint32_t c = 0;
  for (uint32_t w = blockIdx.x * 256 + threadIdx.x; w < W; w += gridDim.x * 256) c += (uint32_t)__popcll(pos[w] | neg[w]);
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) c += __shfl_xor(c, d, 64);
  if ((threadIdx.x & 63) == 0 && c) atomicAdd(out, c);
}

// Bits past N in word W-1 and words W..S-1 of every bit row must be zero.
__global__ void k_check_padding(const uint64_t* __restrict__ rows, uint32_t n_rows, uint32_t W,
                                uint32_t S, uint64_t tail, uint32_t* __restrict__ flags) {
  uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_rows) return;
  const uint64_t* p = rows + (size_t)i * S;
  uint64_t bad = p[W - 1] & ~tail;
  for (uint32_t w = W; w < S; ++w) bad |= p[w];
  if (bad) atomicOr(flags, F_PAD);
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, size_t n, uint32_t v) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t step = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += step) p[i] = v;
}

// Inclusive wave scan of one value per lane.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    uint32_t u = __shfl_up(v, d, 64);
    if (lane >= d) v += u;
  }
  return v;
}

// Block-wide exclusive scan of one value per thread (blockDim = 1024); returns
// the exclusive prefix and writes the block total to *total.
__device__ uint32_t block_excl_scan(uint32_t v, uint32_t* total) {
  __shared__ uint32_t wsum[kScanThreads / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint32_t inc = wave_incl_scan(v);
  if (lane == 63) wsum[wid] = inc;
  __syncthreads();
  if (wid == 0) {
    uint32_t s = lane < kScanThreads / 64 ? wsum[lane] : 0;
    uint32_t si = wave_incl_scan(s);
    if (lane < kScanThreads / 64) wsum[lane] = si - s;
    if (lane == kScanThreads / 64 - 1) *total = si;
  }
  __syncthreads();
  uint32_t r = inc - v + wsum[wid];
  __syncthreads();
  return r;
}

// In place exclusive scan of each row of p[gridDim.x][nb] (one block per row).
__global__ void __launch_bounds__(kScanThreads)
k_scan_block_sums(uint32_t* __restrict__ bsum, uint32_t nb) {
  uint32_t* p = bsum + (size_t)blockIdx.x * nb;
  __shared__ uint32_t carry_s;
  __shared__ uint32_t tot;
  if (threadIdx.x == 0) carry_s = 0;
  __syncthreads();
  for (uint32_t c = 0; c < nb; c += kScanThreads) {
    uint32_t i = c + threadIdx.x;
    uint32_t v = i < nb ? p[i] : 0;
    uint32_t ex = block_excl_scan(v, &tot);
    uint32_t carry = carry_s;
    if (i < nb) p[i] = ex + carry;
    __syncthreads();
    if (threadIdx.x == 0) carry_s = carry + tot;
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// building the derived layouts
//
// The inverse of a role is its exact transpose: a counting sort of the
// assertions by object.  Counting and placing them with one global atomic per
// assertion (two passes over random 4-byte addresses) took 16 of the 18 ms of
// a load of 133M assertions.  Here the objects are cut into buckets of
// 2^shift, and no pass touches random memory beyond an LDS area:
//   k_load_rows    offsets checked, 32-bit offsets, subjects' bit rows;
//   k_load_check   targets checked, assertions counted per bucket (LDS);
//   k_load_part    each assertion's subject found from the offsets, the pairs
//                  (subject, object) written bucket by bucket, in runs;
//   k_load_bucket  one block per bucket: counts, scan and placement of its
//                  pairs in LDS, the inverse rows written as one run.
// The pairs lie in the object-rank area (8 bytes per assertion), which is
// filled later.  Bound by HBM: about 30 bytes per assertion over the passes.
// 133M assertions of 16 roles over 1M individuals: rows 99 us, check 197,
// partition 805, buckets 676; a load 1.9 ms where it was 17.2.
// An invalid knowledge base sets *flags; every kernel that would index with
// unchecked data returns when it is set.  A role's assertions are those of its
// rows (fwd_off[r][N] of them): what may lie between its last row's end and the
// next role's first offset belongs to no subject and is not looked at.
// ---------------------------------------------------------------------------
constexpr uint32_t kPartEdges = 8192;       // assertions of one chunk
constexpr int kPartThreads = 512;
constexpr uint32_t kRowTiles = 8;           // 256-subject tiles of a block of k_load_rows
constexpr uint32_t kBucketMost = 8192;      // objects whose counters fit a block's LDS
constexpr uint32_t kBucketStage = 16384;    // inverse targets staged in LDS by one block
constexpr uint32_t kBucketsMost = 8192;     // buckets a role (LDS counters of k_load_part)
constexpr uint32_t kWordTile = 2048;        // words of a bit row per block
constexpr uint64_t kLoadFill = 2048;        // bucket blocks that fill the chip

struct HeavyOut {
  uint32_t hmin, cap;
  uint32_t* count;
  uint32_t* out;        // (direction 2r + dir, subject, degree), any order
};
__device__ __forceinline__ void heavy_append(const HeavyOut& H, uint32_t rd, uint32_t x, uint32_t deg) {
  const uint32_t slot = atomicAdd(H.count, 1u);
  if (slot < H.cap) {
    H.out[3 * (size_t)slot] = rd;
    H.out[3 * (size_t)slot + 1] = x;
    H.out[3 * (size_t)slot + 2] = deg;
  }
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, d, 64));
  return v;
}

// One thread per (role, subject): the offsets' check, the 32-bit offset, the
// subject's bit (the objects of the inverse direction), heavy rows, the
// role's largest degree.
__global__ void __launch_bounds__(256)
k_load_rows(const int64_t* __restrict__ off, const uint64_t* __restrict__ base, uint32_t N, uint32_t W,
            uint32_t* __restrict__ fwd_off, uint64_t* __restrict__ mask, uint32_t* __restrict__ maxdeg, HeavyOut H,
            uint32_t* __restrict__ flags) {
  __shared__ uint32_t s_most[4];
  const uint32_t r = blockIdx.y, lane = threadIdx.x & 63;
  const int64_t* o = off + (size_t)r * (N + 1);
  const int64_t b0 = (int64_t)base[r], b1 = (int64_t)base[r + 1];
  uint32_t* fo = fwd_off + (size_t)r * (N + 1);
  uint32_t most = 0;
  bool any_bad = false;
#pragma unroll 4
  for (uint32_t i = 0; i < kRowTiles; ++i) {
    const uint64_t x = ((uint64_t)blockIdx.x * kRowTiles + i) * 256 + threadIdx.x;
    uint32_t deg = 0;
    if (x < N) {
      const int64_t o0 = o[x], o1 = o[x + 1];
      if (o0 < b0 || o1 < o0 || o1 > b1) {
        any_bad = true;
      } else {
        fo[x] = (uint32_t)(o0 - b0);
        if (x == N - 1) fo[N] = (uint32_t)(o1 - b0);
        deg = (uint32_t)(o1 - o0);
        if (deg > H.hmin) heavy_append(H, 2 * r, (uint32_t)x, deg);
      }
    }
    most = max(most, deg);
    const uint64_t m = __ballot(deg > 0);
    if (lane == 0 && x < N) mask[((size_t)2 * r + 1) * W + (x >> 6)] = m;
  }
  if (any_bad) atomicOr(flags, F_NONMONO);
  most = wave_max(most);
  if (lane == 0) s_most[threadIdx.x >> 6] = most;
  __syncthreads();
  if (threadIdx.x == 0) {
    most = max(max(s_most[0], s_most[1]), max(s_most[2], s_most[3]));
    if (most > __hip_atomic_load(maxdeg + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(maxdeg + r, most);
  }
}

// The last x with off[x] <= v, for off[0] <= v < off[N]: a whole wave, 64
// probes a step.
__device__ __forceinline__ uint32_t wave_row_of(const uint32_t* __restrict__ off, uint32_t N, uint32_t v) {
  const uint32_t lane = threadIdx.x & 63;
  uint32_t lo = 0, hi = N;
  while (hi - lo > 1) {
    const uint32_t step = (hi - lo + 63) / 64;
    const uint64_t at = (uint64_t)lo + (uint64_t)(lane + 1) * step;
    const uint32_t c = (uint32_t)__popcll(__ballot(at < hi && off[min(at, (uint64_t)N)] <= v));
    lo += c * step;
    hi = min(hi, lo + step);
  }
  return lo;
}

// Targets in [0, N) and rising inside a row, chunk by chunk (a bit per
// assertion marks the rows' starts); the assertions of each bucket of objects.
__global__ void __launch_bounds__(kPartThreads)
k_load_check(const uint32_t* __restrict__ fwd_off, const int32_t* __restrict__ tg, const uint64_t* __restrict__ base,
             uint32_t N, uint32_t nb, uint32_t shift, uint32_t* __restrict__ bcount, uint32_t* __restrict__ flags) {
  constexpr uint32_t kOwn = kPartEdges / kPartThreads;
  extern __shared__ uint32_t s_hist[];
  __shared__ uint32_t s_start[kPartEdges / 32], s_range[2];
  const uint32_t r = blockIdx.y, tid = threadIdx.x;
  // (only what earlier kernels set: this one's own blocks add other reasons)
  if (*flags & (F_NONMONO | F_PAD)) return;
  const uint32_t* fo = fwd_off + (size_t)r * (N + 1);
  const uint32_t n = fo[N];
  const uint32_t chunks = (uint32_t)(((uint64_t)n + kPartEdges - 1) / kPartEdges);
  if (blockIdx.x >= chunks) return;
  const int32_t* t = tg + base[r];
  for (uint32_t i = tid; i < nb; i += kPartThreads) s_hist[i] = 0;
  uint32_t bad = 0;
  for (uint32_t c = blockIdx.x; c < chunks; c += gridDim.x) {
    const uint32_t c0 = c * kPartEdges, cn = min(kPartEdges, n - c0);
    int32_t y[kOwn], prev[kOwn];       // (a wave's first lane also loads the target before its own)
#pragma unroll
    for (uint32_t i = 0; i < kOwn; ++i) {
      const uint32_t e = min(tid + i * kPartThreads, cn - 1);
      y[i] = t[c0 + e];
      prev[i] = (tid & 63) == 0 ? t[c0 + e - (c0 + e > 0)] : 0;
    }
    __syncthreads();
    for (uint32_t i = tid; i < kPartEdges / 32; i += kPartThreads) s_start[i] = 0;
    if (tid < 128) {
      const uint32_t x = wave_row_of(fo, N, tid < 64 ? c0 : c0 + cn - 1);
      if ((tid & 63) == 0) s_range[tid >> 6] = x;
    }
    __syncthreads();
    const uint32_t lo = s_range[0], hi = s_range[1];
    if (tid == 0 && fo[lo] == c0) atomicOr(&s_start[0], 1u);
    for (uint32_t x = lo + 1 + tid; x <= hi; x += kPartThreads) {
      const uint32_t e = fo[x] - c0;
      if (e < cn) atomicOr(&s_start[e >> 5], 1u << (e & 31));
    }
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < kOwn; ++i) {
      const uint32_t e = tid + i * kPartThreads;
      const int32_t up = __shfl_up(y[i], 1, 64);
      const int32_t p = (tid & 63) == 0 ? prev[i] : up;
      if (e >= cn) continue;
      if (y[i] < 0 || (uint32_t)y[i] >= N) {
        bad |= F_TARGET;
        continue;
      }
      if (!((s_start[e >> 5] >> (e & 31)) & 1) && y[i] <= p) bad |= F_ORDER;
      atomicAdd(&s_hist[(uint32_t)y[i] >> shift], 1u);
    }
  }
  if (bad) atomicOr(flags, bad);
  __syncthreads();
  for (uint32_t i = tid; i < nb; i += kPartThreads)
    if (s_hist[i]) atomicAdd(bcount + (size_t)r * nb + i, s_hist[i]);
}

// A bucket that most of a role points into is counted and placed by slices of
// its pairs, a block each: k_load_big<false> adds a slice's counts to the
// objects' inverse offsets (cleared by k_load_part, which sets flags[3]), k_load_bucket turns them
// into each object's end, and k_load_big<true> takes a slice's places off them,
// which leaves the starts.  32M assertions to 5,000 objects: a load of 1.7 ms,
// 17.5 with one block for the bucket; to 64 objects 1.2 and 63.  The line: a
// bucket of that size takes its one block 0.14 ms, the two launches 5 us where
// none is that large.
constexpr uint32_t kBigSlice = 65536, kBigBucket = 4 * kBigSlice;
__device__ __forceinline__ bool big_bucket(const uint32_t* __restrict__ bb, uint32_t nb, uint32_t n, uint32_t b,
                                           uint32_t& i0, uint32_t& i1) {
  i0 = bb[b];
  i1 = b + 1 < nb ? bb[b + 1] : n;
  return i1 - i0 >= kBigBucket;
}

// The pairs of one chunk to their buckets: a thread takes 16 consecutive
// assertions, their subjects from the marked row starts by a running maximum.
// The pairs are put in bucket order in LDS, the chunk's share of each bucket is
// reserved with one global atomic, and consecutive threads write consecutive
// pairs of a bucket (a store per pair at its own address: 936 us for 133M
// pairs, 805 us with the runs).  s_hist: for each bucket its count, then its
// first place in the chunk; s_to: its first place in the bucket less that.
__global__ void __launch_bounds__(kPartThreads)
k_load_part(const uint32_t* __restrict__ fwd_off, const int32_t* __restrict__ tg, const uint64_t* __restrict__ base,
            uint32_t N, uint32_t nb, uint32_t shift, const uint32_t* __restrict__ bbase, uint32_t* __restrict__ bcur,
            uint2* __restrict__ pairs, uint32_t* __restrict__ inv_off, uint32_t* __restrict__ flags) {
  constexpr uint32_t kOwn = kPartEdges / kPartThreads;
  extern __shared__ uint2 s_pair[];                       // [kPartEdges]
  uint32_t* s_row = reinterpret_cast<uint32_t*>(s_pair);  // before the pairs: [kPartEdges] row marks
  uint32_t* s_hist = reinterpret_cast<uint32_t*>(s_pair + kPartEdges);   // [nb]
  uint32_t* s_to = s_hist + nb;                                          // [nb]
  __shared__ uint32_t s_range[2], s_last[kPartThreads / 64];
  const uint32_t r = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if (*flags) return;
  const uint32_t* fo = fwd_off + (size_t)r * (N + 1);
  const uint32_t n = fo[N];
  const uint64_t c0l = (uint64_t)blockIdx.x * kPartEdges;
  if (c0l >= n) return;
  const uint32_t c0 = (uint32_t)c0l, cn = min(kPartEdges, n - c0);
  const int32_t* t = tg + base[r] + c0;
  uint32_t y[kOwn], row[kOwn], rank[kOwn];
#pragma unroll
  for (uint32_t i = 0; i < kOwn; ++i) y[i] = (uint32_t)t[min(tid * kOwn + i, cn - 1)];
  for (uint32_t i = tid; i < nb; i += kPartThreads) s_hist[i] = 0;
  for (uint32_t i = tid; i < kPartEdges; i += kPartThreads) s_row[i] = 0;
  if (tid < 128) {
    const uint32_t x = wave_row_of(fo, N, tid < 64 ? c0 : c0 + cn - 1);
    if (lane == 0) s_range[wv] = x;
  }
  __syncthreads();
  const uint32_t lo = s_range[0], hi = s_range[1];
  // several rows may share a start: all but the last of them are empty
  for (uint32_t x = lo + tid; x <= hi; x += kPartThreads) {
    const uint32_t e = x == lo ? 0u : fo[x] - c0;
    if (e < cn) atomicMax(&s_row[e], x);
  }
  __syncthreads();
  uint32_t m = 0;
#pragma unroll
  for (uint32_t i = 0; i < kOwn; ++i) row[i] = m = max(m, s_row[tid * kOwn + i]);
  uint32_t inc = m;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t u = (uint32_t)__shfl_up((int)inc, d, 64);
    if (lane >= (uint32_t)d) inc = max(inc, u);
  }
  if (lane == 63) s_last[wv] = inc;
  uint32_t before = (uint32_t)__shfl_up((int)inc, 1, 64);
  if (lane == 0) before = 0;
  __syncthreads();
  for (uint32_t w = 0; w < wv; ++w) before = max(before, s_last[w]);
#pragma unroll
  for (uint32_t i = 0; i < kOwn; ++i) {
    row[i] = max(row[i], before);
    if (tid * kOwn + i < cn) rank[i] = atomicAdd(&s_hist[y[i] >> shift], 1u);
  }
  __syncthreads();
  // counts -> first places, and the chunk's share of each bucket
  const uint32_t per = (nb + kPartThreads - 1) / kPartThreads;
  const uint32_t k0 = min(tid * per, nb), k1 = min(k0 + per, nb);
  uint32_t sum = 0;
  for (uint32_t k = k0; k < k1; ++k) sum += s_hist[k];
  inc = wave_incl_scan(sum);
  if (lane == 63) s_last[wv] = inc;
  __syncthreads();
  uint32_t at = inc - sum;
  for (uint32_t w = 0; w < wv; ++w) at += s_last[w];
  for (uint32_t k = k0; k < k1; ++k) {
    const uint32_t c = s_hist[k];
    s_hist[k] = at;
    if (c) s_to[k] = atomicAdd(bcur + (size_t)r * nb + k, c) - at;
    at += c;
  }
  __syncthreads();
#pragma unroll
  for (uint32_t i = 0; i < kOwn; ++i)
    if (tid * kOwn + i < cn) s_pair[s_hist[y[i] >> shift] + rank[i]] = make_uint2(row[i], y[i]);
  __syncthreads();
  uint2* out = pairs + base[r];
  for (uint32_t i = tid; i < cn; i += kPartThreads) {
    const uint2 q = s_pair[i];
    out[s_to[q.y >> shift] + i] = q;
  }
  if (c0) return;
  uint32_t* io = inv_off + (size_t)r * (N + 1);
  for (uint32_t b = tid; b < nb; b += kPartThreads) {
    uint32_t i0, i1;
    if (!big_bucket(bbase + (size_t)r * nb, nb, n, b, i0, i1)) continue;
    flags[3] = 1;
    const uint64_t yend = min((uint64_t)(b + 1) << shift, (uint64_t)N);
    for (uint64_t y = (uint64_t)b << shift; y < yend; ++y) io[y] = 0;
  }
}

template <bool PLACE>
__global__ void __launch_bounds__(kPartThreads)
k_load_big(const uint2* __restrict__ pairs, const uint64_t* __restrict__ base, uint32_t N, uint32_t nb, uint32_t shift,
           uint32_t range, const uint32_t* __restrict__ bbase, const uint32_t* __restrict__ fwd_off,
           uint32_t* __restrict__ inv_off, int32_t* __restrict__ inv_tg, const uint32_t* __restrict__ flags) {
  extern __shared__ uint32_t s_dyn[];      // [range]
  __shared__ uint32_t s_end[2];
  if (flags[0] || !flags[3]) return;
  const uint32_t r = blockIdx.y, tid = threadIdx.x, n = fwd_off[(size_t)r * (N + 1) + N];
  const uint64_t s0l = (uint64_t)blockIdx.x * kBigSlice;
  if (s0l >= n) return;
  const uint32_t s0 = (uint32_t)s0l, s1 = (uint32_t)min(s0l + kBigSlice, (uint64_t)n);
  const uint32_t* bb = bbase + (size_t)r * nb;
  const uint2* p = pairs + base[r];
  uint32_t* io = inv_off + (size_t)r * (N + 1);
  int32_t* it = inv_tg + base[r];
  // a bucket this large reaches over one end of the slice at least
  if (tid < 128) {
    const uint32_t b = wave_row_of(bb, nb, tid < 64 ? s0 : s1 - 1);
    if ((tid & 63) == 0) s_end[tid >> 6] = b;
  }
  __syncthreads();
  for (uint32_t e = 0; e < 2; ++e) {
    const uint32_t b = s_end[e];
    uint32_t i0, i1;
    if ((e && b == s_end[0]) || !big_bucket(bb, nb, n, b, i0, i1)) continue;
    const uint32_t a = max(i0, s0), z = min(i1, s1);
    const uint64_t yend = min((uint64_t)(b + 1) << shift, (uint64_t)N);
    for (uint64_t y0 = (uint64_t)b << shift; y0 < yend; y0 += range) {
      for (uint32_t k = tid; k < range; k += kPartThreads) s_dyn[k] = 0;
      __syncthreads();
      for (uint64_t i = (uint64_t)a + tid; i < z; i += kPartThreads) {
        const uint32_t d = p[i].y - (uint32_t)y0;
        if (d < range) atomicAdd(&s_dyn[d], 1u);
      }
      __syncthreads();
      for (uint32_t k = tid; k < range; k += kPartThreads) {
        const uint32_t c = s_dyn[k];       // (none past N: every pair's object is below)
        if (!c) continue;
        if (PLACE) s_dyn[k] = atomicSub(io + y0 + k, c) - c;
        else atomicAdd(io + y0 + k, c);
      }
      __syncthreads();
      if (PLACE) {
        for (uint64_t i = (uint64_t)a + tid; i < z; i += kPartThreads) {
          const uint2 q = p[i];
          const uint32_t d = q.y - (uint32_t)y0;
          if (d < range) it[atomicAdd(&s_dyn[d], 1u)] = (int32_t)q.x;
        }
        __syncthreads();
      }
    }
  }
}

// One bucket of objects: the inverse offsets, rows, objects' bits, heavy rows
// and largest degree.  Order inside an inverse row follows the atomics and is
// not fixed; evaluation results do not depend on it.  A bucket wider than the
// LDS counters goes by sub-ranges, reading its pairs once for each.
__global__ void __launch_bounds__(kPartThreads)
k_load_bucket(const uint2* __restrict__ pairs, const uint64_t* __restrict__ base, uint32_t N, uint32_t W, uint32_t nb,
              uint32_t shift, uint32_t range, const uint32_t* __restrict__ bbase, const uint32_t* __restrict__ fwd_off,
              uint32_t* __restrict__ inv_off, int32_t* __restrict__ inv_tg, uint64_t* __restrict__ mask, uint32_t* __restrict__ maxdeg, HeavyOut H,
              const uint32_t* __restrict__ flags) {
  extern __shared__ uint32_t s_dyn[];
  __shared__ uint32_t s_wsum[kPartThreads / 64];
  uint32_t* s_cnt = s_dyn;                 // [range]
  uint32_t* s_out = s_dyn + range;         // [kBucketStage]
  if (*flags) return;
  const uint32_t r = blockIdx.y, b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const uint32_t n = fwd_off[(size_t)r * (N + 1) + N];
  uint32_t i0, i1;
  const bool big = big_bucket(bbase + (size_t)r * nb, nb, n, b, i0, i1);   // counted and placed by k_load_big
  const uint2* p = pairs + base[r];
  uint32_t* io = inv_off + (size_t)r * (N + 1);
  int32_t* it = inv_tg + base[r];
  const uint64_t yend = min((uint64_t)(b + 1) << shift, (uint64_t)N);
  uint32_t run = i0, most = 0;
  for (uint64_t y0 = (uint64_t)b << shift; y0 < yend; y0 += range) {
    for (uint32_t i = tid; i < range; i += kPartThreads) s_cnt[i] = big && y0 + i < N ? io[y0 + i] : 0u;
    __syncthreads();
    if (!big)
      for (uint64_t i = (uint64_t)i0 + tid; i < i1; i += kPartThreads) {
        const uint32_t d = p[i].y - (uint32_t)y0;
        if (d < range) atomicAdd(&s_cnt[d], 1u);
      }
    __syncthreads();
    for (uint32_t k = tid; k < range; k += kPartThreads) {
      const uint64_t m = __ballot(s_cnt[k] > 0);
      const uint64_t w = (y0 + k) >> 6;
      if (lane == 0 && w < W) mask[(size_t)2 * r * W + w] = m;
    }
    __syncthreads();
    const uint32_t per = (range + kPartThreads - 1) / kPartThreads;
    const uint32_t k0 = min(tid * per, range), k1 = min(k0 + per, range);
    uint32_t sum = 0;
    for (uint32_t k = k0; k < k1; ++k) sum += s_cnt[k];
    const uint32_t inc = wave_incl_scan(sum);
    if (lane == 63) s_wsum[wv] = inc;
    __syncthreads();
    uint32_t ex = inc - sum, total = 0;
    for (uint32_t w = 0; w < kPartThreads / 64; ++w) {
      if (w < wv) ex += s_wsum[w];
      total += s_wsum[w];
    }
    for (uint32_t k = k0; k < k1; ++k) {
      const uint32_t c = s_cnt[k];
      const uint64_t yy = y0 + k;
      if (yy < N) {
        io[yy] = run + ex + (big ? c : 0u);
        if (c > H.hmin) heavy_append(H, 2 * r + 1, (uint32_t)yy, c);
      }
      most = max(most, c);
      s_cnt[k] = ex;
      ex += c;
    }
    __syncthreads();
    const bool staged = total <= kBucketStage;
    for (uint64_t i = (uint64_t)i0 + tid; !big && i < i1; i += kPartThreads) {
      const uint2 q = p[i];
      const uint32_t d = q.y - (uint32_t)y0;
      if (d >= range) continue;
      const uint32_t pos = atomicAdd(&s_cnt[d], 1u);
      if (staged) s_out[pos] = q.x;
      else it[run + pos] = (int32_t)q.x;
    }
    __syncthreads();
    if (staged && !big)
      for (uint32_t i = tid; i < total; i += kPartThreads) it[run + i] = (int32_t)s_out[i];
    run += total;
    __syncthreads();
  }
  if (b + 1 == nb && tid == 0) io[N] = n;
  most = wave_max(most);
  if (lane == 0 && most > __hip_atomic_load(maxdeg + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMax(maxdeg + r, most);
}

// Objects of a role direction: the individuals that occur as targets in it
// (for the forward direction the subjects of non-empty inverse rows, and the
// other way round).  mask row 2r + dir holds one bit per individual; base row
// 2r + dir the number of objects in the words before each word (entry W =
// their total); ctg maps each assertion's target to its rank among the
// objects, so that a shared pass can index transposed child rows that hold
// the objects only.
// The words of 64 consecutive subjects with at least one assertion, in
// increasing order (the role passes visit only these, and a pass may take
// several consecutive entries at once), are the non-zero words of the other
// direction's objects.  Both lists of all directions in two kernels with a
// scan of the tiles' sums between them.
__device__ __forceinline__ void word_tile(const uint64_t* __restrict__ m, uint32_t W, uint64_t (&v)[8], uint32_t& pop,
                                          uint32_t& full) {
  const uint32_t w0 = blockIdx.x * kWordTile + threadIdx.x * 8;
  pop = full = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    v[i] = w0 + i < W ? m[w0 + i] : 0;
    pop += (uint32_t)__popcll(v[i]);
    full += v[i] != 0;
  }
}
__global__ void __launch_bounds__(256)
k_words_sum(const uint64_t* __restrict__ mask, uint32_t W, uint32_t tiles, uint32_t* __restrict__ tsum) {
  __shared__ uint32_t s[2][4];
  const uint32_t rd = 2 * blockIdx.y + blockIdx.z, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint64_t v[8];
  uint32_t pop, full;
  word_tile(mask + (size_t)rd * W, W, v, pop, full);
  pop = wave_incl_scan(pop), full = wave_incl_scan(full);
  if (lane == 63) s[0][wv] = pop, s[1][wv] = full;
  __syncthreads();
  if (threadIdx.x < 2)
    tsum[((size_t)threadIdx.x * 2 * gridDim.y + rd) * tiles + blockIdx.x] =
        s[threadIdx.x][0] + s[threadIdx.x][1] + s[threadIdx.x][2] + s[threadIdx.x][3];
}
__global__ void __launch_bounds__(256)
k_words_write(const uint64_t* __restrict__ mask, uint32_t W, uint32_t tiles, const uint32_t* __restrict__ tsum,
              uint32_t* __restrict__ objbase, uint32_t* __restrict__ words, uint32_t* __restrict__ nobj,
              uint32_t* __restrict__ nwords) {
  __shared__ uint32_t s[2][4];
  const uint32_t rd = 2 * blockIdx.y + blockIdx.z, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint64_t v[8];
  uint32_t pop, full;
  word_tile(mask + (size_t)rd * W, W, v, pop, full);
  const uint32_t ip = wave_incl_scan(pop), fi = wave_incl_scan(full);
  if (lane == 63) s[0][wv] = ip, s[1][wv] = fi;
  __syncthreads();
  uint32_t p = tsum[(size_t)rd * tiles + blockIdx.x] + ip - pop;
  uint32_t f = tsum[((size_t)2 * gridDim.y + rd) * tiles + blockIdx.x] + fi - full;
  for (uint32_t w = 0; w < wv; ++w) p += s[0][w], f += s[1][w];
  uint32_t* ob = objbase + (size_t)rd * (W + 1);
  uint32_t* list = words + (size_t)(rd ^ 1) * W;
  const uint32_t w0 = blockIdx.x * kWordTile + threadIdx.x * 8;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    if (w0 + i >= W) break;
    ob[w0 + i] = p;
    p += (uint32_t)__popcll(v[i]);
    if (v[i]) list[f++] = w0 + i;
  }
  if (blockIdx.x + 1 == tiles && threadIdx.x == 255) {   // the row's totals
    ob[W] = p;
    nobj[rd] = p;
    nwords[rd ^ 1] = f;
  }
}

// Object ranks of the directions whose objects are at most half of the
// individuals.
__global__ void __launch_bounds__(256)
k_object_rank(const int32_t* __restrict__ fwd_tg, const int32_t* __restrict__ inv_tg, const uint64_t* __restrict__ base,
              const uint32_t* __restrict__ fwd_off, uint32_t N, uint32_t W, const uint64_t* __restrict__ mask, const uint32_t* __restrict__ objbase,
              const uint32_t* __restrict__ nobj, int32_t* __restrict__ ctg_fwd, int32_t* __restrict__ ctg_inv,
              const uint32_t* __restrict__ flags) {
  const uint32_t rd = 2 * blockIdx.y + blockIdx.z, r = rd >> 1, dir = rd & 1;
  if ((uint64_t)nobj[rd] * 2 > N || *flags) return;
  const int32_t* tg = (dir ? inv_tg : fwd_tg) + base[r];
  int32_t* ctg = (dir ? ctg_inv : ctg_fwd) + base[r];
  const uint64_t* m = mask + (size_t)rd * W;
  const uint32_t* ob = objbase + (size_t)rd * (W + 1);
  const uint64_t n = fwd_off[(size_t)r * (N + 1) + N];
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256) {
    const uint32_t y = (uint32_t)tg[i];
    ctg[i] = (int32_t)(ob[y >> 6] + (uint32_t)__popcll(m[y >> 6] & ((1ull << (y & 63)) - 1ull)));
  }
}

struct DerivedLayout {
  size_t fwd_off, inv_off, inv_tg, cursor, tsum, base, meta, words, objmask, objbase, ctg;
  size_t heavy, hchunk, hchunk0, cpop, dir, total;
  uint32_t tiles;                // word tiles of a bit row
  size_t heavy_cap, chunk_cap;   // entries
};

static DerivedLayout layout_for(const hth_kb_desc& d) {
  DerivedLayout L{};
  size_t R = d.n_roles, N = d.n_individuals;
  size_t offs = align_up(R * (N + 1) * 4, 256);
  L.tiles = (uint32_t)(((N + 63) / 64 + kWordTile - 1) / kWordTile);
  size_t at = 0;
  L.fwd_off = at; at += offs;
  L.inv_off = at; at += offs;
  L.inv_tg = at; at += align_up((size_t)d.n_edges * 4, 256);
  L.cursor = at; at += offs;
  L.tsum = at; at += align_up(4 * R * L.tiles * 4 + 4, 256);
  L.base = at; at += align_up((R + 1) * 8, 256);
  L.meta = at; at += align_up((4 + 6 * R) * 4, 256);
  L.words = at; at += align_up(2 * R * ((N + 63) / 64) * 4, 256);
  L.objmask = at; at += align_up(2 * R * ((N + 63) / 64) * 8, 256);
  L.objbase = at; at += align_up(2 * R * ((N + 63) / 64 + 1) * 4, 256);
  L.ctg = at; at += align_up((size_t)d.n_edges * 8, 256);     // both directions
  // a direction holds at most E_dir / (heavy_min + 1) heavy rows, so the table
  // (by the floor of heavy_min) is never full; appends are checked regardless
  L.heavy_cap = 2 * (d.n_edges / (kHeavyMinFloor + 1)) + 2;
  L.chunk_cap = 2 * (d.n_edges / kHeavyChunk) + L.heavy_cap + 2;
  L.heavy = at; at += align_up(L.heavy_cap * 12, 256);
  L.hchunk = at; at += align_up(L.chunk_cap * sizeof(HeavyChunk), 256);
  L.hchunk0 = at; at += align_up((L.heavy_cap + 1) * 4, 256);
  L.cpop = at; at += align_up((size_t)d.n_concepts * 4 + 4, 256);
  L.dir = at; at += align_up(3 * (2 * R + 1) * 4, 256);
  L.total = at;
  return L;
}

static hth_status check_desc(const hth_kb_desc* d) {
  if (!d) return fail(HTH_E_INVALID, "desc is NULL");
  if (d->n_individuals == 0 || d->n_individuals >= (1u << 31))
    return fail(HTH_E_RANGE, "n_individuals must be in [1, 2^31)");
  uint32_t W = (d->n_individuals + 63) / 64;
  if (d->stride_words < W || d->stride_words % 8)
    return fail(HTH_E_INVALID, "stride_words must be >= ceil(N/64) and a multiple of 8");
  if (d->n_concepts && !d->concept_bits) return fail(HTH_E_INVALID, "concept_bits is NULL");
  if ((reinterpret_cast<uintptr_t>(d->concept_bits) | reinterpret_cast<uintptr_t>(d->pos_bits) |
       reinterpret_cast<uintptr_t>(d->neg_bits)) % 16)
    return fail(HTH_E_INVALID, "bit rows must be 16-byte aligned");
  if (d->n_roles && (!d->role_offsets || (d->n_edges && !d->role_targets)))
    return fail(HTH_E_INVALID, "role arrays are NULL");
  if (d->n_roles > 65535) return fail(HTH_E_RANGE, "at most 65535 roles");
  if (d->n_edges >= (1ull << 40)) return fail(HTH_E_RANGE, "too many assertions");
  if (d->n_data && !d->data) return fail(HTH_E_INVALID, "data is NULL");
  if (!d->pos_bits || !d->neg_bits) return fail(HTH_E_INVALID, "example rows are NULL");
  if (d->n_concepts >= (1u << 26)) return fail(HTH_E_RANGE, "too many concepts");
  return HTH_OK;
}

}  // namespace hth

using namespace hth;

extern "C" hth_status hth_kb_derived_bytes(const hth_kb_desc* desc, size_t* bytes) {
  hth_status s = check_desc(desc);
  if (s) return s;
  if (!bytes) return fail(HTH_E_INVALID, "bytes is NULL");
  *bytes = layout_for(*desc).total;
  return HTH_OK;
}

// A device error flag word -> HTH_E_INVALID with the reasons.
static hth_status check_flags(uint32_t flags) {
  if (!flags) return HTH_OK;
  std::string m = "invalid knowledge base:";
  if (flags & F_NONMONO) m += " role offsets not monotone;";
  if (flags & F_TARGET) m += " role target outside [0, N);";
  if (flags & F_ORDER) m += " role targets not strictly increasing in a row;";
  if (flags & F_PAD) m += " padding bits set in a bit row;";
  return fail(HTH_E_INVALID, m);
}

struct HeavyTables {
  std::vector<uint32_t> heavy_first, chunk_first;   // [2R+1]
  uint32_t heavy_most = 0, chunk_most = 0;
};

// Sorts the heavy rows by (direction, subject) and writes the heavy-row,
// chunk and first-chunk tables to the device.
static hth_status upload_heavy(hth_kb_s* kb, const DerivedLayout& L, const std::vector<uint32_t>& trip,
                               HeavyTables& T, hipStream_t st) {
  const uint32_t R = kb->d.n_roles;
  const uint32_t nh = (uint32_t)(trip.size() / 3);
  T.heavy_first.assign(2 * R + 1, 0);
  T.chunk_first.assign(2 * R + 1, 0);
  if (!nh) return HTH_OK;
  std::vector<uint32_t> ord(nh);
  for (uint32_t i = 0; i < nh; ++i) ord[i] = i;
  std::sort(ord.begin(), ord.end(), [&](uint32_t a, uint32_t b) {
    return trip[3 * a] != trip[3 * b] ? trip[3 * a] < trip[3 * b] : trip[3 * a + 1] < trip[3 * b + 1];
  });
  std::vector<uint32_t> rows(nh), chunk0(nh + 1);
  std::vector<HeavyChunk> chunks;
  std::vector<uint32_t> per(2 * R, 0), cper(2 * R, 0);
  for (uint32_t i = 0; i < nh; ++i) {
    const uint32_t* t = &trip[3 * (size_t)ord[i]];
    rows[i] = t[1];
    per[t[0]]++;
    const uint32_t nc = (t[2] + kHeavyChunk - 1) / kHeavyChunk;
    cper[t[0]] += nc;
    chunk0[i] = (uint32_t)chunks.size();
    for (uint32_t k = 0; k < nc; ++k) chunks.push_back(HeavyChunk{i, k});
  }
  chunk0[nh] = (uint32_t)chunks.size();
  if (chunks.size() > L.chunk_cap) return fail(HTH_E_RANGE, "heavy chunk table overflow");
  for (uint32_t rd = 0; rd < 2 * R; ++rd) {
    T.heavy_first[rd + 1] = T.heavy_first[rd] + per[rd];
    T.chunk_first[rd + 1] = T.chunk_first[rd] + cper[rd];
    T.heavy_most = std::max(T.heavy_most, per[rd]);
    T.chunk_most = std::max(T.chunk_most, cper[rd]);
  }
  HTH_HIP(hipMemcpyAsync(kb->heavy_rows, rows.data(), rows.size() * 4, hipMemcpyHostToDevice, st));
  HTH_HIP(hipMemcpyAsync(kb->heavy_chunks, chunks.data(), chunks.size() * sizeof(HeavyChunk),
                         hipMemcpyHostToDevice, st));
  HTH_HIP(hipMemcpyAsync(kb->heavy_chunk0, chunk0.data(), chunk0.size() * 4, hipMemcpyHostToDevice, st));
  HTH_HIP(hipStreamSynchronize(st));
  return HTH_OK;
}

static hth_status kb_build(hth_kb_s* kb, char* derived, hipStream_t st) {
  const hth_kb_desc& d = kb->d;
  const uint32_t R = d.n_roles, N = kb->N;
  DerivedLayout L = layout_for(d);
  kb->fwd_off = reinterpret_cast<uint32_t*>(derived + L.fwd_off);
  kb->inv_off = reinterpret_cast<uint32_t*>(derived + L.inv_off);
  kb->inv_tg = reinterpret_cast<int32_t*>(derived + L.inv_tg);
  uint32_t* tsum = reinterpret_cast<uint32_t*>(derived + L.tsum);
  uint64_t* base = reinterpret_cast<uint64_t*>(derived + L.base);
  uint32_t* meta = reinterpret_cast<uint32_t*>(derived + L.meta);
  uint32_t* flags = meta;              // meta: flags, heavy rows, examples, whether a bucket is big, then
  uint32_t* maxdeg = meta + 4;         // [2][R] largest degrees
  uint32_t* nwords = meta + 4 + 2 * R; // [R][2] non-empty words
  uint32_t* nobj = meta + 4 + 4 * R;   // [R][2] objects
  kb->role_base_dev = base;

  auto fill = [&](uint32_t* p, size_t n, uint32_t v) {
    if (!n) return;
    unsigned g = (unsigned)std::min<size_t>((n + 255) / 256, 65536);
    hipLaunchKernelGGL(k_fill_u32, dim3(g), dim3(256), 0, st, p, n, v);
  };
  fill(meta, 4 + 6 * (size_t)R, 0);
  const uint32_t tb = 256;
  // padding of concept rows and example rows
  if (d.n_concepts)
    hipLaunchKernelGGL(k_check_padding, dim3((d.n_concepts + tb - 1) / tb), dim3(tb), 0, st,
                       d.concept_bits, d.n_concepts, kb->W, kb->S, kb->tail, flags);
  hipLaunchKernelGGL(k_check_padding, dim3(1), dim3(1), 0, st, d.pos_bits, 1u, kb->W, kb->S,
                     kb->tail, flags);
  hipLaunchKernelGGL(k_check_padding, dim3(1), dim3(1), 0, st, d.neg_bits, 1u, kb->W, kb->S,
                     kb->tail, flags);
  hipLaunchKernelGGL(k_count_examples, dim3(std::min(256u, (kb->W + 255) / 256)), dim3(256), 0, st, d.pos_bits,
                     d.neg_bits, kb->W, meta + 2);
  kb->concept_pop.assign(d.n_concepts, 0);
  if (d.n_concepts) {
    uint32_t* cpop = reinterpret_cast<uint32_t*>(derived + L.cpop);
    hipLaunchKernelGGL(k_row_pop, dim3(d.n_concepts), dim3(256), 0, st, d.concept_bits, kb->W, kb->S, cpop);
    HTH_HIP(hipGetLastError());
    HTH_HIP(hipMemcpyAsync(kb->concept_pop.data(), cpop, (size_t)d.n_concepts * 4, hipMemcpyDeviceToHost, st));
  }
  kb->role_base.assign(R + 1, 0);
  kb->max_deg[0].assign(R, 0);
  kb->max_deg[1].assign(R, 0);
  std::vector<uint32_t> got(4 + 6 * (size_t)R);
  if (R) {
    hipLaunchKernelGGL(k_gather_bases, dim3((R + 255) / 256), dim3(256), 0, st, d.role_offsets,
                       R, N, base);
    HTH_HIP(hipGetLastError());
    HTH_HIP(hipMemcpyAsync(kb->role_base.data(), base, (R + 1) * 8, hipMemcpyDeviceToHost, st));
    HTH_HIP(hipStreamSynchronize(st));
    if (kb->role_base[0] != 0) return fail(HTH_E_INVALID, "role_offsets[0][0] must be 0");
    if (kb->role_base[R] != d.n_edges)
      return fail(HTH_E_INVALID, "role_offsets[R-1][N] must equal n_edges");
    uint64_t most = 0;      // assertions of the largest role
    for (uint32_t r = 0; r < R; ++r) {
      if (kb->role_base[r + 1] < kb->role_base[r])
        return fail(HTH_E_INVALID, "role offsets decrease between roles");
      if (kb->role_base[r + 1] - kb->role_base[r] >= (1ull << 32))
        return fail(HTH_E_RANGE, "a role has 2^32 or more assertions");
      most = std::max(most, kb->role_base[r + 1] - kb->role_base[r]);
    }
    kb->heavy_rows = reinterpret_cast<uint32_t*>(derived + L.heavy);
    kb->heavy_chunks = reinterpret_cast<HeavyChunk*>(derived + L.hchunk);
    kb->heavy_chunk0 = reinterpret_cast<uint32_t*>(derived + L.hchunk0);
    kb->words = reinterpret_cast<uint32_t*>(derived + L.words);
    kb->objmask = reinterpret_cast<uint64_t*>(derived + L.objmask);
    kb->objbase = reinterpret_cast<uint32_t*>(derived + L.objbase);
    kb->ctg_fwd = reinterpret_cast<int32_t*>(derived + L.ctg);
    kb->ctg_inv = kb->ctg_fwd + d.n_edges;
    const HeavyOut H{kb->heavy_min, (uint32_t)std::min<size_t>(L.heavy_cap, 0xFFFFFFFFu), meta + 1, kb->heavy_rows};
    // buckets of objects: a power of two so that an average bucket of the
    // largest role has its inverse targets staged in LDS (three quarters of the
    // stage, for the spread), at least one word of 64, and within the counters;
    // as wide as that allows (k_load_part's runs) while the blocks fill the chip
    uint32_t shift = 6;
    while (shift < 31 && ((uint64_t)N >> shift) > 0 &&
           ((((uint64_t)N + (1ull << shift) - 1) >> shift) > kBucketsMost ||
            ((1u << shift) < kBucketMost && (most << (shift + 1)) / N <= kBucketStage * 3 / 4 &&
             ((uint64_t)N >> (shift + 1)) * R >= kLoadFill)))
      ++shift;
    const uint32_t nb = (uint32_t)(((uint64_t)N + (1ull << shift) - 1) >> shift);
    const uint32_t range = (uint32_t)std::min<uint64_t>(1ull << shift, kBucketMost);
    uint32_t* bbase = reinterpret_cast<uint32_t*>(derived + L.cursor);   // [R][nb] twice, in [R][N+1]
    uint32_t* bcur = bbase + (size_t)R * nb;
    uint2* pairs = reinterpret_cast<uint2*>(derived + L.ctg);
    auto part_lds = [](size_t buckets) { return sizeof(uint2) * kPartEdges + 8 * buckets; };
    HTH_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_load_part),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)part_lds(kBucketsMost)));
    HTH_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_load_bucket),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)(4 * (kBucketMost + kBucketStage))));
    fill(bbase, (size_t)R * nb, 0);
    hipLaunchKernelGGL(k_load_rows, dim3((N - 1) / (256 * kRowTiles) + 1, R), dim3(256), 0, st, d.role_offsets, base, N, kb->W,
                       kb->fwd_off, kb->objmask, maxdeg, H, flags);
    const uint32_t chunks = (uint32_t)((most + kPartEdges - 1) / kPartEdges);
    if (chunks) {
      const unsigned per = std::max(1u, std::min(8u, (unsigned)((uint64_t)chunks * R / 2048)));
      hipLaunchKernelGGL(k_load_check, dim3((chunks + per - 1) / per, R), dim3(kPartThreads), nb * 4, st, kb->fwd_off,
                         d.role_targets, base, N, nb, shift, bbase, flags);
    }
    hipLaunchKernelGGL(k_scan_block_sums, dim3(R), dim3(kScanThreads), 0, st, bbase, nb);
    HTH_HIP(hipMemcpyAsync(bcur, bbase, (size_t)R * nb * 4, hipMemcpyDeviceToDevice, st));
    if (chunks)
      hipLaunchKernelGGL(k_load_part, dim3(chunks, R), dim3(kPartThreads), part_lds(nb), st, kb->fwd_off, d.role_targets,
                         base, N, nb, shift, bbase, bcur, pairs, kb->inv_off, flags);
    const dim3 slices((unsigned)((most + kBigSlice - 1) / kBigSlice), R);
    if (most >= kBigBucket)
      hipLaunchKernelGGL(k_load_big<false>, slices, dim3(kPartThreads), 4 * range, st, pairs, base, N, nb, shift, range,
                         bbase, kb->fwd_off, kb->inv_off, kb->inv_tg, flags);
    const size_t lds = 4 * ((size_t)range + kBucketStage);
    hipLaunchKernelGGL(k_load_bucket, dim3(nb, R), dim3(kPartThreads), lds, st, pairs, base, N, kb->W, nb, shift, range,
                       bbase, kb->fwd_off, kb->inv_off, kb->inv_tg, kb->objmask, maxdeg + R, H, flags);
    if (most >= kBigBucket)
      hipLaunchKernelGGL(k_load_big<true>, slices, dim3(kPartThreads), 4 * range, st, pairs, base, N, nb, shift, range,
                         bbase, kb->fwd_off, kb->inv_off, kb->inv_tg, flags);
    hipLaunchKernelGGL(k_words_sum, dim3(L.tiles, R, 2), dim3(256), 0, st, kb->objmask, kb->W, L.tiles, tsum);
    hipLaunchKernelGGL(k_scan_block_sums, dim3(4 * R), dim3(kScanThreads), 0, st, tsum, L.tiles);
    hipLaunchKernelGGL(k_words_write, dim3(L.tiles, R, 2), dim3(256), 0, st, kb->objmask, kb->W, L.tiles, tsum,
                       kb->objbase, kb->words, nobj, nwords);
    if (most) {
      const unsigned g = (unsigned)std::min<uint64_t>((most + 2047) / 2048, 65536);
      hipLaunchKernelGGL(k_object_rank, dim3(g, R, 2), dim3(256), 0, st, d.role_targets, kb->inv_tg, base, kb->fwd_off, N, kb->W,
                         kb->objmask, kb->objbase, nobj, kb->ctg_fwd, kb->ctg_inv, flags);
    }
    HTH_HIP(hipGetLastError());
  }
  HTH_HIP(hipMemcpyAsync(got.data(), meta, got.size() * 4, hipMemcpyDeviceToHost, st));
  HTH_HIP(hipStreamSynchronize(st));
  if (hth_status fs = check_flags(got[0])) return fs;
  kb->ex_hint = got[2];
  if (!R) return HTH_OK;
  const uint32_t* g = got.data() + 4;
  kb->max_deg[0].assign(g, g + R);
  kb->max_deg[1].assign(g + R, g + 2 * R);
  kb->n_words.assign(g + 2 * R, g + 4 * R);
  kb->n_obj.assign(g + 4 * R, g + 6 * R);
  // the heavy-row tables of both directions
  const uint32_t nh = got[1];
  if (nh > L.heavy_cap) return fail(HTH_E_RANGE, "heavy-row table overflow");
  std::vector<uint32_t> trip(3 * (size_t)nh);
  if (nh) {
    HTH_HIP(hipMemcpyAsync(trip.data(), kb->heavy_rows, trip.size() * 4, hipMemcpyDeviceToHost, st));
    HTH_HIP(hipStreamSynchronize(st));
  }
  HeavyTables all;
  hth_status fs = upload_heavy(kb, L, trip, all, st);
  if (fs) return fs;
  kb->heavy_first = all.heavy_first;
  kb->chunk_first = all.chunk_first;
  kb->heavy_most = all.heavy_most;
  kb->chunk_most = all.chunk_most;
  // each direction's non-empty words, first heavy chunk and first heavy row
  // (device plans read them)
  std::vector<uint32_t> dir(3 * (2 * (size_t)R + 1), 0);
  std::copy(kb->n_words.begin(), kb->n_words.end(), dir.begin());
  std::copy(kb->chunk_first.begin(), kb->chunk_first.end(), dir.begin() + 2 * R + 1);
  std::copy(kb->heavy_first.begin(), kb->heavy_first.end(), dir.begin() + 2 * (2 * R + 1));
  kb->dir_dev = reinterpret_cast<uint32_t*>(derived + L.dir);
  HTH_HIP(hipMemcpyAsync(kb->dir_dev, dir.data(), dir.size() * 4, hipMemcpyHostToDevice, st));
  HTH_HIP(hipStreamSynchronize(st));
  return HTH_OK;
}

extern "C" hth_status hth_kb_create(const hth_kb_desc* desc, void* derived, size_t derived_bytes,
                                    void* stream, hth_kb* out) {
  hth_status s = check_desc(desc);
  if (s) return s;
  if (!out) return fail(HTH_E_INVALID, "out is NULL");
  DerivedLayout L = layout_for(*desc);
  if (!derived || derived_bytes < L.total)
    return fail(HTH_E_NOMEM, "derived buffer smaller than hth_kb_derived_bytes");
  if (reinterpret_cast<uintptr_t>(derived) % 256)
    return fail(HTH_E_INVALID, "derived buffer must be 256-byte aligned");
  hth_kb_s* kb = new (std::nothrow) hth_kb_s();
  if (!kb) return fail(HTH_E_NOMEM, "host allocation failed");
  kb->d = *desc;
  kb->N = desc->n_individuals;
  kb->W = (kb->N + 63) / 64;
  kb->S = desc->stride_words;
  kb->tail = (kb->N & 63) ? ((1ull << (kb->N & 63)) - 1) : ~0ull;
  kb->pos = desc->pos_bits;
  kb->neg = desc->neg_bits;
  hipError_t e = hipGetDevice(&kb->device);
  int n_cu = 0, lds = 0;
  if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, kb->device);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, kb->device);
  if (e != hipSuccess) {
    delete kb;
    return hip_fail(e, "hipDeviceGetAttribute");
  }
  kb->n_cu = n_cu;
  auto env_u = [](const char* n, uint64_t dflt) {
    const char* e = std::getenv(n);
    return e ? (uint64_t)std::strtoull(e, nullptr, 10) : dflt;
  };
  kb->tune.group_min = (uint32_t)env_u("HTHEDL_GROUP_MIN", kb->tune.group_min);
  kb->tune.group_k = (uint32_t)std::min<uint64_t>(64, std::max<uint64_t>(1, env_u("HTHEDL_GROUP_K", kb->tune.group_k)));
  kb->tune.xcd_local = (uint32_t)env_u("HTHEDL_XCD", kb->tune.xcd_local);
  kb->tune.t_budget = env_u("HTHEDL_TBUDGET_MB", kb->tune.t_budget >> 20) << 20;
  kb->tune.group_unroll = (uint32_t)env_u("HTHEDL_GROUP_UNROLL", kb->tune.group_unroll);
  kb->tune.region_reg = (uint32_t)env_u("HTHEDL_REGION_REG", kb->tune.region_reg);
  kb->tune.t_compact = (uint32_t)env_u("HTHEDL_T_COMPACT", kb->tune.t_compact);
  kb->tune.t_segment_kb = (uint32_t)std::min<uint64_t>(1u << 22, env_u("HTHEDL_TSEG_KB", kb->tune.t_segment_kb));
  kb->tune.push_pct = (uint32_t)std::min<uint64_t>(100, env_u("HTHEDL_PUSH_PCT", kb->tune.push_pct));
  kb->tune.short_rows = (uint32_t)std::min<uint64_t>(64, env_u("HTHEDL_SHORT_ROWS", kb->tune.short_rows));
  kb->view_min = (uint32_t)std::min<uint64_t>(0xFFFFFFFFu, env_u("HTHEDL_VIEW_MIN", kb->view_min));
  kb->heavy_min = (uint32_t)std::min<uint64_t>(
      1u << 30, std::max<uint64_t>(kHeavyMinFloor, env_u("HTHEDL_HEAVY_MIN", kb->heavy_min)));
  kb->lds_per_block = (size_t)lds;
  s = kb_build(kb, static_cast<char*>(derived), static_cast<hipStream_t>(stream));
  if (s) {
    delete kb;
    return s;
  }
  *out = kb;
  return HTH_OK;
}

// ---------------------------------------------------------------------------
// multi-valued numeric concrete roles
// ---------------------------------------------------------------------------
namespace hth {

struct NumLayout {
  size_t heavy, hchunk, hchunk0, meta, roff, total;
  size_t heavy_cap, chunk_cap;
};
static NumLayout num_layout(uint32_t N, uint32_t n_roles, uint64_t n_values) {
  NumLayout L{};
  L.heavy_cap = n_values / (kHeavyMinFloor + 1) + 2;
  L.chunk_cap = n_values / kHeavyChunk + L.heavy_cap + 2;
  size_t at = 0;
  L.heavy = at; at += align_up(L.heavy_cap * 12, 256);
  L.hchunk = at; at += align_up(L.chunk_cap * sizeof(HeavyChunk), 256);
  L.hchunk0 = at; at += align_up((L.heavy_cap + 1) * 4, 256);
  L.meta = at; at += align_up((4 + (size_t)n_roles) * 4, 256);
  L.roff = at; at += align_up((size_t)n_roles * (N + 1) * 4, 256);
  L.total = at;
  return L;
}

// One thread per (role, subject): offsets within [lo, hi] and non-decreasing;
// the role's largest degree.
__global__ void k_validate_num_rows(const int64_t* __restrict__ off, uint32_t N, uint64_t n_values,
                                    uint32_t* __restrict__ maxdeg, uint32_t* __restrict__ flags) {
  const uint32_t x = blockIdx.x * blockDim.x + threadIdx.x, r = blockIdx.y;
  if (x >= N) return;
  const int64_t* o = off + (size_t)r * (N + 1);
  const int64_t a = o[x], b = o[x + 1];
  if (a < 0 || b < a || (uint64_t)b > n_values) {
    atomicOr(flags, F_NONMONO);
    return;
  }
  if (b - a >= (1ll << 32)) {
    atomicOr(flags, F_NONMONO);
    return;
  }
  atomicMax(maxdeg + r, (uint32_t)(b - a));
}

__global__ void k_check_values(const float* __restrict__ v, uint64_t n, uint32_t* __restrict__ flags) {
  bool bad = false;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256)
    bad |= v[i] != v[i];
  if (bad) atomicOr(flags, F_TARGET);
}

// 32-bit offsets relative to each role's first value (one thread per entry).
__global__ void k_rel_offsets(const int64_t* __restrict__ off, uint32_t N, uint32_t* __restrict__ rel) {
  const uint32_t x = blockIdx.x * blockDim.x + threadIdx.x, r = blockIdx.y;
  if (x > N) return;
  const int64_t* o = off + (size_t)r * (N + 1);
  rel[(size_t)r * (N + 1) + x] = (uint32_t)(o[x] - o[0]);
}

// Heavy rows of numeric role r (more than hmin values) as (r, subject, degree).
__global__ void __launch_bounds__(256)
k_heavy_rows64(const int64_t* __restrict__ o, uint32_t N, uint32_t hmin, uint32_t r, uint32_t cap,
               uint32_t* __restrict__ count, uint32_t* __restrict__ out) {
  const uint32_t x = blockIdx.x * 256 + threadIdx.x;
  if (x >= N) return;
  const uint64_t deg = (uint64_t)(o[x + 1] - o[x]);
  if (deg <= hmin) return;
  const uint32_t slot = atomicAdd(count, 1u);
  if (slot < cap) {
    out[3 * (size_t)slot] = r;
    out[3 * (size_t)slot + 1] = x;
    out[3 * (size_t)slot + 2] = (uint32_t)deg;
  }
}

}  // namespace hth

extern "C" hth_status hth_numeric_derived_bytes(hth_kb kb, uint32_t n_roles, uint64_t n_values, size_t* bytes) {
  if (!kb || !bytes) return fail(HTH_E_INVALID, "NULL argument");
  if (n_roles >= (1u << 16) || n_values >= (1ull << 40)) return fail(HTH_E_RANGE, "too many numeric roles or values");
  *bytes = num_layout(kb->N, n_roles, n_values).total;
  return HTH_OK;
}

namespace hth {

// Ids in [0, n) and non-decreasing offsets from 0 (string dictionary, patterns).
__global__ void k_check_ids(const int32_t* __restrict__ ids, uint64_t n, uint32_t n_strings,
                            uint32_t* __restrict__ flags) {
  bool bad = false;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256)
    bad |= ids[i] < 0 || (uint32_t)ids[i] >= n_strings;
  if (bad) atomicOr(flags, F_TARGET);
}
__global__ void k_check_monotone64(const int64_t* __restrict__ o, uint64_t n, uint32_t* __restrict__ flags) {
  bool bad = false;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256)
    bad |= (i == 0 && o[0] != 0) || (i > 0 && o[i] < o[i - 1]);
  if (bad) atomicOr(flags, F_ORDER);
}

// The tables of a registration of value roles (numeric or string): heavy rows
// and their chunks in the caller's derived buffer, per-role first chunk and
// first value on the host.
struct ValueRoles {
  uint32_t* roff = nullptr;   // [n_roles][N+1] relative offsets
  uint32_t* rows = nullptr;
  HeavyChunk* chunks = nullptr;
  std::vector<uint32_t> chunk_first;
  std::vector<uint64_t> bounds;
};

// Validates the chain and monotonicity of offsets [n_roles][N+1] against
// n_values; `extra` (run on the stream before the check) adds the kind's own
// value checks into flags.  Then builds the heavy-row tables.
template <class Extra>
static hth_status value_roles(hth_kb_s* kb, uint32_t n_roles, const int64_t* offsets, uint64_t n_values,
                              char* dv, const NumLayout& L, hipStream_t st, Extra&& extra, ValueRoles& out) {
  const uint32_t N = kb->N;
  uint32_t* meta = reinterpret_cast<uint32_t*>(dv + L.meta);
  uint32_t* flags = meta;
  uint32_t* count = meta + 1;
  uint32_t* maxdeg = meta + 4;
  hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(256), 0, st, meta, (size_t)4 + n_roles, 0u);
  std::vector<int64_t> ends(2 * (size_t)n_roles);
  for (uint32_t r = 0; r < n_roles; ++r) {
    HTH_HIP(hipMemcpyAsync(&ends[2 * r], offsets + (size_t)r * (N + 1), 8, hipMemcpyDeviceToHost, st));
    HTH_HIP(hipMemcpyAsync(&ends[2 * r + 1], offsets + (size_t)r * (N + 1) + N, 8, hipMemcpyDeviceToHost, st));
  }
  HTH_HIP(hipStreamSynchronize(st));
  if (ends[0] != 0) return fail(HTH_E_INVALID, "value role offsets[0][0] must be 0");
  for (uint32_t r = 1; r < n_roles; ++r)
    if (ends[2 * r] != ends[2 * r - 1]) return fail(HTH_E_INVALID, "value role ranges must follow one another");
  if ((uint64_t)ends[2 * (size_t)n_roles - 1] != n_values)
    return fail(HTH_E_INVALID, "value role offsets[n_roles-1][N] must equal n_values");
  hipLaunchKernelGGL(k_validate_num_rows, dim3((N + 255) / 256, n_roles), dim3(256), 0, st, offsets, N, n_values,
                     maxdeg, flags);
  extra(flags);
  HTH_HIP(hipGetLastError());
  uint32_t hflags = 0;
  std::vector<uint32_t> md(n_roles);
  HTH_HIP(hipMemcpyAsync(&hflags, flags, 4, hipMemcpyDeviceToHost, st));
  HTH_HIP(hipMemcpyAsync(md.data(), maxdeg, (size_t)n_roles * 4, hipMemcpyDeviceToHost, st));
  HTH_HIP(hipStreamSynchronize(st));
  if (hflags & F_NONMONO) return fail(HTH_E_INVALID, "value role offsets not monotone or out of range");
  if (hflags & F_TARGET) return fail(HTH_E_INVALID, "a value is NaN or a string id is out of range");
  if (hflags & F_ORDER) return fail(HTH_E_INVALID, "string or pattern offsets not non-decreasing from 0");
  // heavy rows, sorted by (role, subject), and their chunk tables
  out.rows = reinterpret_cast<uint32_t*>(dv + L.heavy);
  out.chunks = reinterpret_cast<HeavyChunk*>(dv + L.hchunk);
  out.chunk_first.assign(n_roles + 1, 0);
  bool any = false;
  for (uint32_t r = 0; r < n_roles; ++r)
    if (md[r] > kb->heavy_min) {
      any = true;
      hipLaunchKernelGGL(k_heavy_rows64, dim3((N + 255) / 256), dim3(256), 0, st, offsets + (size_t)r * (N + 1), N,
                         kb->heavy_min, r, (uint32_t)L.heavy_cap, count, out.rows);
    }
  HTH_HIP(hipGetLastError());
  if (any) {
    uint32_t nh = 0;
    HTH_HIP(hipMemcpyAsync(&nh, count, 4, hipMemcpyDeviceToHost, st));
    HTH_HIP(hipStreamSynchronize(st));
    if (nh > L.heavy_cap) return fail(HTH_E_RANGE, "heavy-row table overflow");
    std::vector<uint32_t> trip(3 * (size_t)nh);
    HTH_HIP(hipMemcpyAsync(trip.data(), out.rows, trip.size() * 4, hipMemcpyDeviceToHost, st));
    HTH_HIP(hipStreamSynchronize(st));
    std::vector<uint32_t> ord(nh);
    for (uint32_t i = 0; i < nh; ++i) ord[i] = i;
    std::sort(ord.begin(), ord.end(), [&](uint32_t a, uint32_t b) {
      return trip[3 * a] != trip[3 * b] ? trip[3 * a] < trip[3 * b] : trip[3 * a + 1] < trip[3 * b + 1];
    });
    std::vector<uint32_t> hrows(nh);
    std::vector<HeavyChunk> chunks;
    std::vector<uint32_t> cper(n_roles, 0);
    for (uint32_t i = 0; i < nh; ++i) {
      const uint32_t* t = &trip[3 * (size_t)ord[i]];
      hrows[i] = t[1];
      const uint32_t nc = (t[2] + kHeavyChunk - 1) / kHeavyChunk;
      cper[t[0]] += nc;
      for (uint32_t k = 0; k < nc; ++k) chunks.push_back(HeavyChunk{i, k});
    }
    if (chunks.size() > L.chunk_cap) return fail(HTH_E_RANGE, "heavy chunk table overflow");
    for (uint32_t r = 0; r < n_roles; ++r) out.chunk_first[r + 1] = out.chunk_first[r] + cper[r];
    HTH_HIP(hipMemcpyAsync(out.rows, hrows.data(), hrows.size() * 4, hipMemcpyHostToDevice, st));
    HTH_HIP(hipMemcpyAsync(out.chunks, chunks.data(), chunks.size() * sizeof(HeavyChunk), hipMemcpyHostToDevice, st));
    HTH_HIP(hipStreamSynchronize(st));
  }
  out.bounds.assign(n_roles + 1, 0);
  for (uint32_t r = 0; r < n_roles; ++r) out.bounds[r + 1] = (uint64_t)ends[2 * r + 1];
  out.roff = reinterpret_cast<uint32_t*>(dv + L.roff);
  hipLaunchKernelGGL(k_rel_offsets, dim3((N + 256) / 256, n_roles), dim3(256), 0, st, offsets, N, out.roff);
  HTH_HIP(hipGetLastError());
  HTH_HIP(hipStreamSynchronize(st));
  return HTH_OK;
}

static unsigned grid_for(uint64_t n) { return (unsigned)std::max<uint64_t>(1, std::min<uint64_t>((n + 255) / 256, 65536)); }

}  // namespace hth

extern "C" hth_status hth_kb_set_numeric(hth_kb kb, uint32_t n_roles, const int64_t* offsets, const float* values,
                                         uint64_t n_values, void* derived, size_t derived_bytes, void* stream) {
  if (!kb) return fail(HTH_E_INVALID, "kb is NULL");
  std::lock_guard<std::mutex> g(kb->mu);
  if (n_roles == 0) {
    kb->n_num = 0;
    kb->num_off = nullptr;
    kb->num_val = nullptr;
    kb->num_chunk_first.assign(1, 0);
    kb->num_bounds.assign(1, 0);
    return HTH_OK;
  }
  if (!offsets || (n_values && !values) || !derived) return fail(HTH_E_INVALID, "NULL argument");
  if (n_roles >= (1u << 16) || n_values >= (1ull << 40)) return fail(HTH_E_RANGE, "too many numeric roles or values");
  const NumLayout L = num_layout(kb->N, n_roles, n_values);
  if (derived_bytes < L.total) return fail(HTH_E_NOMEM, "numeric derived buffer smaller than hth_numeric_derived_bytes");
  if (reinterpret_cast<uintptr_t>(derived) % 256) return fail(HTH_E_INVALID, "derived buffer must be 256-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  ValueRoles V;
  hth_status s = value_roles(kb, n_roles, offsets, n_values, static_cast<char*>(derived), L, st, [&](uint32_t* flags) {
    if (n_values) hipLaunchKernelGGL(k_check_values, dim3(grid_for(n_values)), dim3(256), 0, st, values, n_values, flags);
  }, V);
  if (s) return s;
  kb->n_num = n_roles;
  kb->num_off = offsets;
  kb->num_val = values;
  kb->num_roff = V.roff;
  kb->num_heavy_rows = V.rows;
  kb->num_heavy_chunks = V.chunks;
  kb->num_chunk_first = V.chunk_first;
  kb->num_bounds = V.bounds;
  return HTH_OK;
}

extern "C" hth_status hth_string_derived_bytes(hth_kb kb, uint32_t n_roles, uint64_t n_values, size_t* bytes) {
  return hth_numeric_derived_bytes(kb, n_roles, n_values, bytes);
}

extern "C" hth_status hth_kb_set_strings(hth_kb kb, uint32_t n_roles, const int64_t* offsets, const int32_t* ids,
                                         uint64_t n_values, uint32_t n_strings, const int64_t* str_offsets,
                                         const uint8_t* chars, void* derived, size_t derived_bytes, void* stream) {
  if (!kb) return fail(HTH_E_INVALID, "kb is NULL");
  std::lock_guard<std::mutex> g(kb->mu);
  if (n_roles == 0) {
    kb->n_str = 0;
    kb->str_off = nullptr;
    kb->str_ids = nullptr;
    kb->str_chunk_first.assign(1, 0);
    kb->str_bounds.assign(1, 0);
    return HTH_OK;
  }
  if (!offsets || (n_values && !ids) || !derived || !str_offsets) return fail(HTH_E_INVALID, "NULL argument");
  if (n_roles >= (1u << 16) || n_values >= (1ull << 40)) return fail(HTH_E_RANGE, "too many string roles or values");
  if (n_strings >= (1u << 31)) return fail(HTH_E_RANGE, "n_strings >= 2^31");
  const NumLayout L = num_layout(kb->N, n_roles, n_values);
  if (derived_bytes < L.total) return fail(HTH_E_NOMEM, "string derived buffer smaller than hth_string_derived_bytes");
  if (reinterpret_cast<uintptr_t>(derived) % 256) return fail(HTH_E_INVALID, "derived buffer must be 256-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  ValueRoles V;
  hth_status s = value_roles(kb, n_roles, offsets, n_values, static_cast<char*>(derived), L, st, [&](uint32_t* flags) {
    if (n_values) hipLaunchKernelGGL(k_check_ids, dim3(grid_for(n_values)), dim3(256), 0, st, ids, n_values, n_strings, flags);
    hipLaunchKernelGGL(k_check_monotone64, dim3(grid_for((uint64_t)n_strings + 1)), dim3(256), 0, st, str_offsets,
                       (uint64_t)n_strings + 1, flags);
  }, V);
  if (s) return s;
  kb->n_str = n_roles;
  kb->n_strings = n_strings;
  kb->str_off = offsets;
  kb->str_ids = ids;
  kb->dict_off = str_offsets;
  kb->dict_chars = chars;
  kb->str_roff = V.roff;
  kb->str_heavy_rows = V.rows;
  kb->str_heavy_chunks = V.chunks;
  kb->str_chunk_first = V.chunk_first;
  kb->str_bounds = V.bounds;
  return HTH_OK;
}

extern "C" hth_status hth_kb_set_patterns(hth_kb kb, uint32_t n_patterns, const int64_t* offsets, const uint8_t* chars,
                                          void* stream) {
  if (!kb) return fail(HTH_E_INVALID, "kb is NULL");
  if (n_patterns && !offsets) return fail(HTH_E_INVALID, "NULL argument");
  std::lock_guard<std::mutex> g(kb->mu);
  if (n_patterns) {   // a short table: its offsets are checked on the host
    std::vector<int64_t> o((size_t)n_patterns + 1);
    hipStream_t st = static_cast<hipStream_t>(stream);
    HTH_HIP(hipMemcpyAsync(o.data(), offsets, o.size() * 8, hipMemcpyDeviceToHost, st));
    HTH_HIP(hipStreamSynchronize(st));
    if (o[0] != 0) return fail(HTH_E_INVALID, "pattern offsets[0] must be 0");
    for (size_t i = 1; i < o.size(); ++i)
      if (o[i] < o[i - 1]) return fail(HTH_E_INVALID, "pattern offsets must be non-decreasing");
    if (o.back() > 0 && !chars) return fail(HTH_E_INVALID, "pattern chars are NULL");
  }
  kb->n_patterns = n_patterns;
  kb->pat_off = n_patterns ? offsets : nullptr;
  kb->pat_chars = n_patterns ? chars : nullptr;
  return HTH_OK;
}

extern "C" hth_status hth_kb_set_examples(hth_kb kb, const uint64_t* pos, const uint64_t* neg) {
  if (!kb) return fail(HTH_E_INVALID, "kb is NULL");
  if (!pos || !neg) return fail(HTH_E_INVALID, "example rows are NULL");
  if ((reinterpret_cast<uintptr_t>(pos) | reinterpret_cast<uintptr_t>(neg)) % 16)
    return fail(HTH_E_INVALID, "example rows must be 16-byte aligned");
  std::lock_guard<std::mutex> g(kb->mu);
  kb->pos = pos;
  kb->neg = neg;
  return HTH_OK;
}

extern "C" hth_status hth_kb_set_sets(hth_kb kb, const uint64_t* rows, uint32_t n_rows) {
  if (!kb) return fail(HTH_E_INVALID, "kb is NULL");
  if (n_rows && !rows) return fail(HTH_E_INVALID, "set rows are NULL");
  if (n_rows >= (1u << 24)) return fail(HTH_E_RANGE, "set table holds at most 2^24 - 1 rows");
  if (reinterpret_cast<uintptr_t>(rows) % 16) return fail(HTH_E_INVALID, "set rows must be 16-byte aligned");
  std::lock_guard<std::mutex> g(kb->mu);
  kb->sets = n_rows ? rows : nullptr;
  kb->n_sets = n_rows;
  return HTH_OK;
}

extern "C" hth_status hth_kb_max_degree(hth_kb kb, uint32_t role, uint32_t inv, uint32_t* out) {
  if (!kb || !out) return fail(HTH_E_INVALID, "NULL argument");
  if (role >= kb->d.n_roles || inv > 1) return fail(HTH_E_RANGE, "role or direction out of range");
  *out = kb->max_deg[inv][role];
  return HTH_OK;
}

extern "C" hth_status hth_kb_get_tuning(hth_kb kb, hth_tuning* out) {
  if (!kb || !out) return fail(HTH_E_INVALID, "NULL argument");
  std::lock_guard<std::mutex> g(kb->mu);
  out->group_min = kb->tune.group_min;
  out->group_k = kb->tune.group_k;
  out->xcd_local = kb->tune.xcd_local;
  out->t_budget_mb = (uint32_t)(kb->tune.t_budget >> 20);
  out->unroll = kb->tune.group_unroll;
  out->region_reg = kb->tune.region_reg;
  out->t_compact = kb->tune.t_compact;
  out->t_segment_kb = kb->tune.t_segment_kb;
  out->push_pct = kb->tune.push_pct;
  out->short_rows = kb->tune.short_rows;
  return HTH_OK;
}

extern "C" hth_status hth_kb_set_tuning(hth_kb kb, const hth_tuning* t) {
  if (!kb || !t) return fail(HTH_E_INVALID, "NULL argument");
  if (t->group_k < 1 || t->group_k > 64 || t->xcd_local > 1 || t->t_budget_mb < 1 ||
      t->t_budget_mb > (1u << 20) || (t->unroll != 8 && t->unroll != 16) ||
      (t->region_reg != 0 && t->region_reg != 1 && t->region_reg != 2 && t->region_reg != 4) ||
      t->t_compact > 1 || t->t_segment_kb > (1u << 22) || t->push_pct > 100 || t->short_rows > 64)
    return fail(HTH_E_RANGE, "tuning value out of range");
  std::lock_guard<std::mutex> g(kb->mu);
  kb->tune.group_min = t->group_min;
  kb->tune.group_k = t->group_k;
  kb->tune.xcd_local = t->xcd_local;
  kb->tune.t_budget = (size_t)t->t_budget_mb << 20;
  kb->tune.group_unroll = t->unroll;
  kb->tune.region_reg = t->region_reg;
  kb->tune.t_compact = t->t_compact;
  kb->tune.t_segment_kb = t->t_segment_kb;
  kb->tune.push_pct = t->push_pct;
  kb->tune.short_rows = t->short_rows;
  return HTH_OK;
}

extern "C" hth_status hth_kb_destroy(hth_kb kb) {
  delete kb;
  return HTH_OK;
}

extern "C" hth_status hth_sync(void* stream) {
  HTH_HIP(hipStreamSynchronize(static_cast<hipStream_t>(stream)));
  HTH_HIP(hipGetLastError());
  return HTH_OK;
}

extern "C" const char* hth_status_str(hth_status s) {
  switch (s) {
    case HTH_OK: return "HTH_OK";
    case HTH_E_INVALID: return "HTH_E_INVALID";
    case HTH_E_RANGE: return "HTH_E_RANGE";
    case HTH_E_NOMEM: return "HTH_E_NOMEM";
    case HTH_E_DEVICE: return "HTH_E_DEVICE";
    case HTH_E_PLAN: return "HTH_E_PLAN";
    case HTH_E_STATE: return "HTH_E_STATE";
    case HTH_E_UNSUPPORTED: return "HTH_E_UNSUPPORTED";
    default: return "HTH_E_UNKNOWN";
  }
}

extern "C" size_t hth_last_error(char* buf, size_t n) {
  const std::string& m = g_err;
  if (buf && n) {
    size_t k = std::min(n - 1, m.size());
    std::memcpy(buf, m.data(), k);
    buf[k] = 0;
  }
  return m.size();
}
