// Learned screener kernels: hashed subtree features, a bf16 MLP whose products
// run on MFMA (v_mfma_f32_32x32x16_bf16, fp32 accumulation), its backward pass,
// BCE-with-logits on the two coverage fractions, AdamW, and top-k selection.
//
// The screener ranks refinement candidates so that only the best fraction is
// evaluated exactly; the exact engine stays the judge of every count.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "kb_handle.h"

namespace hth {

// ---------------------------------------------------------------------------
// features: Merkle FNV-1a over the postfix nodes of each hypothesis
// ---------------------------------------------------------------------------
constexpr uint64_t kFnvOffset = 0xCBF29CE484222325ull;
constexpr uint32_t kFeatDim = 4096;

__device__ __forceinline__ uint64_t fnv_bytes(uint64_t h, uint64_t v, int n) {
#pragma unroll
  for (int i = 0; i < n; ++i) {
    h ^= (v >> (8 * i)) & 0xFFu;
    // times the FNV prime, 2^40 + 0x1B3
    const uint32_t lo = (uint32_t)h, hi = (uint32_t)(h >> 32);
    h = (uint64_t)lo * 0x1B3u + ((uint64_t)(hi * 0x1B3u + (lo << 8)) << 32);
  }
  return h;
}

__device__ __forceinline__ uint64_t mix64(uint64_t x) {   // splitmix64 finaliser
  uint64_t z = x + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// header bytes of a node: op, inv, arity (2 LE), arg (4 LE), q (4 LE), with the
// fields a construct does not use set to zero
__device__ __forceinline__ uint64_t node_header_hash(const hth_node& n) {
  const uint32_t op = n.op;
  const bool value_op = op >= HTH_DATA_EQ && op <= HTH_NUM_EQ;   // EXACT and numeric concrete roles
  const bool uses_arg = op == HTH_ATOM || (op >= HTH_EXISTS && op <= HTH_DATA_LE) || value_op;
  const bool uses_q = (op >= HTH_ATLEAST && op <= HTH_EXACTLY) || op == HTH_DATA_GE || op == HTH_DATA_LE ||
                      value_op;
  const bool uses_inv = op >= HTH_EXISTS && op <= HTH_EXACTLY;
  const uint32_t arity = (op == HTH_AND || op == HTH_OR) ? n.arity : 0;
  uint32_t q;
  memcpy(&q, &n.q, 4);
  uint64_t h = kFnvOffset;
  h = fnv_bytes(h, op, 1);
  h = fnv_bytes(h, uses_inv ? n.inv : 0, 1);
  h = fnv_bytes(h, arity, 2);
  h = fnv_bytes(h, uses_arg ? n.arg : 0, 4);
  h = fnv_bytes(h, uses_q ? q : 0, 4);
  return h;
}

// Node i's subtree hash from its header's hash v: the child's hash for NOT and
// role constructs, the sum of the children's mixed hashes for AND / OR, read
// through at(local index).  A malformed child sets *bad and gives 0.
template <class At>
__device__ __forceinline__ uint64_t subtree_hash(uint64_t v, uint32_t op, uint32_t arity, uint32_t child, uint32_t li,
                                                 const uint32_t* __restrict__ children, uint32_t n_children, At at,
                                                 uint32_t* __restrict__ bad) {
  // the DL constructs; set-table leaves carry no syntax
  bool ok = op <= HTH_DATA_LE || (op >= HTH_DATA_EQ && op <= HTH_NUM_EQ);
  if (op == HTH_NOT || (op >= HTH_EXISTS && op <= HTH_EXACTLY)) {
    ok = ok && child < li;
    v = fnv_bytes(v, ok ? at(child) : 0ull, 8);
  } else if (op == HTH_AND || op == HTH_OR) {
    uint64_t s = 0;
    ok = ok && (uint64_t)child + arity <= n_children;
    for (uint32_t j = 0; ok && j < arity; ++j) {
      const uint32_t c = children[child + j];
      ok = c < li;
      if (ok) s += mix64(at(c));
    }
    v = fnv_bytes(v, s, 8);
  }
  if (!ok) {
    atomicOr(bad, 1u);
    v = 0;
  }
  return v;
}

// hash[i] holds node i's subtree hash, feat[i] its feature index (hash mod
// 4096).  A block takes 128 hypotheses.  Their nodes lie in one range: the
// header hashes (12 of a leaf's 12 bytes, 12 of an operator's 20) are computed
// a node per thread from coalesced loads, then each hypothesis's thread walks
// its nodes in LDS and hashes children into parents, and the results go out
// coalesced.  A range beyond the LDS area is walked in global memory.  One
// thread per hypothesis in global memory took 94 us for 262,157 hypotheses
// (2.6M nodes), bound by its uncoalesced 16-byte reads; this takes 61 us.
constexpr uint32_t kFeatHyps = 128, kFeatNodes = 2048;
__global__ void __launch_bounds__(256)
k_features(const hth_node* __restrict__ nodes, const uint32_t* __restrict__ offs,
           const uint32_t* __restrict__ children, uint32_t n_children,
           uint32_t n_hyps, uint64_t* __restrict__ hash, uint16_t* __restrict__ feat,
           uint32_t* __restrict__ bad) {
  __shared__ uint64_t s_hash[kFeatNodes];
  __shared__ uint2 s_node[kFeatNodes];   // op and arity; child
  const uint32_t h0 = blockIdx.x * kFeatHyps, h1 = min(h0 + kFeatHyps, n_hyps), h = h0 + threadIdx.x;
  const uint32_t first = offs[h0], last = offs[h1];
  // offsets rise; a range that does not is left to the walk below
  const bool staged = last - first <= kFeatNodes;
  if (!staged) {
    if (threadIdx.x >= kFeatHyps || h >= n_hyps) return;
    const uint32_t b = offs[h], e = offs[h + 1];
    for (uint32_t i = b; i < e; ++i) {
      const hth_node n = nodes[i];
      const uint64_t v = subtree_hash(node_header_hash(n), n.op, n.arity, n.child, i - b, children, n_children,
                                      [&](uint32_t c) { return hash[b + c]; }, bad);
      hash[i] = v;
      feat[i] = (uint16_t)(v & (kFeatDim - 1));
    }
    return;
  }
  for (uint32_t i = threadIdx.x; i < last - first; i += 256) {
    const hth_node n = nodes[first + i];
    s_hash[i] = node_header_hash(n);
    s_node[i] = make_uint2(n.op | (uint32_t)n.arity << 16, n.child);
  }
  __syncthreads();
  if (threadIdx.x < kFeatHyps && h < n_hyps) {
    const uint32_t b = offs[h] - first, e = offs[h + 1] - first;
    for (uint32_t i = b; i < e && i < kFeatNodes; ++i) {
      const uint2 q = s_node[i];
      s_hash[i] = subtree_hash(s_hash[i], q.x & 255u, q.x >> 16, q.y, i - b, children, n_children,
                               [&](uint32_t c) { return s_hash[b + c]; }, bad);
    }
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < last - first; i += 256) {
    const uint64_t v = s_hash[i];
    hash[first + i] = v;
    feat[first + i] = (uint16_t)(v & (kFeatDim - 1));
  }
}

// dense bf16 feature rows: x[r][f] = number of subtrees of hypothesis row0 + r
// whose feature index is f (small integers, exact in bf16)
__global__ void __launch_bounds__(256)
k_densify(const uint16_t* __restrict__ feat, const uint32_t* __restrict__ offs, uint32_t row0,
          uint32_t n_rows, const uint16_t* __restrict__ pfeat, const uint32_t* __restrict__ poffs,
          const uint32_t* __restrict__ pidx, uint32_t context, __bf16* __restrict__ x) {
  __shared__ int32_t cnt[kFeatDim];
  const uint32_t r = blockIdx.x;
  if (r >= n_rows) return;
  for (uint32_t i = threadIdx.x; i < kFeatDim; i += 256) cnt[i] = 0;
  __syncthreads();
  const uint32_t b = offs[row0 + r], e = offs[row0 + r + 1];
  for (uint32_t i = b + threadIdx.x; i < e; i += 256) atomicAdd(&cnt[feat[i] & (kFeatDim - 1)], 1);
  if (pidx) {   // minus the parent's subtrees: what the refinement added or changed
    const uint32_t p = pidx[row0 + r];
    const uint32_t pb = poffs[p], pe = poffs[p + 1];
    for (uint32_t i = pb + threadIdx.x; i < pe; i += 256) atomicSub(&cnt[pfeat[i] & (kFeatDim - 1)], 1);
    // the parent itself, in the other half of the index space (top bit flipped)
    if (context)
      for (uint32_t i = pb + threadIdx.x; i < pe; i += 256)
        atomicAdd(&cnt[(pfeat[i] & (kFeatDim - 1)) ^ (kFeatDim / 2)], 1);
  }
  __syncthreads();
  __bf16* row = x + (size_t)r * kFeatDim;
  for (uint32_t i = threadIdx.x; i < kFeatDim; i += 256) row[i] = (__bf16)(float)cnt[i];
}

// ---------------------------------------------------------------------------
// bf16 GEMM on MFMA: C[M][N] = sum_k A[m][k] B[k][n], fp32 accumulation
//   TA = 0: A stored [M][K] (lda >= K);  TA = 1: A stored [K][M] (A^T given)
//   TB = 0: B stored [K][N] (ldb >= N);  TB = 1: B stored [N][K]
// Epilogue: + bias[n]; ReLU; * (mask[m][n] > 0); outputs fp32 and/or bf16.
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

struct GemmEpi {
  const float* bias;     // [N] or null
  int relu;              // 1: max(x, 0)
  const __bf16* mask;    // [M][ldm] or null: zero where mask <= 0
  int ldm;
  float* c32;            // [M][ldc] or null
  int ldc;
  __bf16* cbf;           // [M][ldcb] or null
  int ldcb;
};

// One operand's share of a k-tile, T rows (m or n) by BK k's, staged by 128
// threads: 8 chunks of 8 values each.  TR = 0, the matrix is [row][k]: a chunk
// is 8 k's of one row and goes to LDS as it is.  TR = 1, the matrix is
// [k][row]: a thread holds 8 k's by 8 rows, transposed in registers (pairs of
// values, one byte permute each) on the way to LDS, so both layouts use 16-byte
// global loads and 16-byte LDS stores.  Addresses are clamped into the matrix
// (no branch around a load); k's past K are zeroed on the way to LDS, rows past
// the edge only reach outputs that are not stored.  LDS rows are padded by 16
// bytes: an odd number of 16-byte units, so neither the stores nor the
// fragments' loads meet in a bank.
template <int TR, int T, int BK>
struct Stage {
  static constexpr int KC = BK / 8;
  static_assert(T * BK == 128 * 64, "128 threads x 8 chunks of 8");
  __device__ static __forceinline__ void load(const __bf16* __restrict__ P, int ld, int row0, int rows, int K,
                                              int k0, int t, bf16x8 (&r)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if constexpr (TR == 0) {
        const int c = t + 128 * i, row = min(row0 + c / KC, rows - 1), k = k0 + (c % KC) * 8;
        r[i] = *reinterpret_cast<const bf16x8*>(P + (size_t)row * ld + (k < K ? k : 0));
      } else {
        const int k = k0 + (t % KC) * 8 + i, row = min(row0 + (t / KC) * 8, rows - 8);
        r[i] = *reinterpret_cast<const bf16x8*>(P + (size_t)(k < K ? k : 0) * ld + row);
      }
    }
  }
  __device__ static __forceinline__ void store(__bf16 (*L)[BK + 8], int K, int k0, int t, bf16x8 (&r)[8]) {
    bf16x8 z;
#pragma unroll
    for (int i = 0; i < 8; ++i) z[i] = (__bf16)0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if constexpr (TR == 0) {
        const int c = t + 128 * i, kk = (c % KC) * 8;
        *reinterpret_cast<bf16x8*>(&L[c / KC][kk]) = k0 + kk < K ? r[i] : z;
      } else {
        if (k0 + (t % KC) * 8 + i >= K) r[i] = z;
      }
    }
    if constexpr (TR == 1) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        bf16x8 v;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = r[i][j];
        *reinterpret_cast<bf16x8*>(&L[(t / KC) * 8 + j][(t % KC) * 8]) = v;
      }
    }
  }
};

// One T x T tile of C per block, 4 waves, each a quarter as products of 32 x 32
// on v_mfma_f32_32x32x16_bf16; k in rising steps of 16 into one accumulator, so
// every tile size gives the same bits.  Two k-tiles of global loads are in
// flight in registers while the MFMAs work on a third in LDS (two buffers, one
// barrier a k-tile): a 1,024-row batch has few blocks a CU, so the loads'
// latency is what has to be covered.  Waves 0 and 1 stage A, 2 and 3 stage B.
// Bound by the LDS reads and the barrier of a k-tile.  Against one 128 x 128 x 64
// tile per block with one k-tile of loads ahead (forward) and 128 x 128 x 32
// with the transpose as 2-byte LDS stores (weight gradients): 1024 x 1024 x 4096
// forward 24.9 us (was 54), 4096 x 1024 x 1024 gradient 25.6 us (was 82),
// 1024 x 256 x 1024 gradient 12.3 us (was 77).
//
// DEEP = 0, for short k: one k-tile of loads ahead and one LDS buffer, so that
// three blocks fit a CU and the stores of C, which bound it there, run beside
// other blocks' products.  With DEEP = 1 the registers are held to two blocks a
// CU; left to the compiler they were more than 256, one block a CU (65,536 x
// 1024 x 64: 121 us; two deep blocks a CU 78, three flat ones 55).
template <int T, int BK, int DEEP>
struct GemmLds {
  __bf16 a[1 + DEEP][T][BK + 8], b[1 + DEEP][T][BK + 8];
};

template <int TA, int TB, int T, int BK, int DEEP>
__device__ __forceinline__ void gemm_tile(GemmLds<T, BK, DEEP>& L, int bx, int by, int M, int N, int K,
                                          const __bf16* __restrict__ A, int lda, const __bf16* __restrict__ B,
                                          int ldb, const GemmEpi& ep) {
  auto& As = L.a;
  auto& Bs = L.b;
  constexpr int F = T / 64;                       // 32 x 32 products per wave and side
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int wm = wv >> 1, wn = wv & 1, t = tid & 127;
  const int m0 = by * T, n0 = bx * T;
  using SA = Stage<TA, T, BK>;
  using SB = Stage<1 - TB, T, BK>;
  f32x16 acc[F][F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  auto load = [&](int k0, bf16x8 (&r)[8]) {
    if (tid < 128) SA::load(A, lda, m0, M, K, k0, t, r);
    else SB::load(B, ldb, n0, N, K, k0, t, r);
  };
  auto store = [&](int buf, int k0, bf16x8 (&r)[8]) {
    if (tid < 128) SA::store(As[buf], K, k0, t, r);
    else SB::store(Bs[buf], K, k0, t, r);
  };
  auto multiply = [&](int buf) {
#pragma unroll
    for (int ks = 0; ks < BK; ks += 16) {
      bf16x8 a[F], b[F];
#pragma unroll
      for (int i = 0; i < F; ++i)
        a[i] = *reinterpret_cast<const bf16x8*>(&As[buf][wm * (T / 2) + i * 32 + (lane & 31)][ks + 8 * (lane >> 5)]);
#pragma unroll
      for (int j = 0; j < F; ++j)
        b[j] = *reinterpret_cast<const bf16x8*>(&Bs[buf][wn * (T / 2) + j * 32 + (lane & 31)][ks + 8 * (lane >> 5)]);
#pragma unroll
      for (int i = 0; i < F; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  };
  bf16x8 r0[8];
  load(0, r0);
  if constexpr (!DEEP) {
    store(0, 0, r0);
    __syncthreads();
    for (int k0 = 0; k0 < K; k0 += BK) {
      const bool more = k0 + BK < K;
      if (more) load(k0 + BK, r0);
      __builtin_amdgcn_sched_barrier(0);
      multiply(0);
      __syncthreads();
      if (more) {
        store(0, k0 + BK, r0);
        __syncthreads();
      }
    }
  } else {
    bf16x8 r1[8];
    load(BK, r1);
    store(0, 0, r0);
    __syncthreads();
    // two k-tiles a turn, the second one all zeros where their number is odd;
    // the scheduling barriers keep the loads above the products
    for (int k0 = 0; k0 < K; k0 += 2 * BK) {
      load(k0 + 2 * BK, r0);
      __builtin_amdgcn_sched_barrier(0);
      multiply(0);
      store(1, k0 + BK, r1);
      __syncthreads();
      load(k0 + 3 * BK, r1);
      __builtin_amdgcn_sched_barrier(0);
      multiply(1);
      store(0, k0 + 2 * BK, r0);
      __syncthreads();
    }
  }
  // epilogue: register r of lane l holds row 8(r/4) + 4(l/32) + r%4, column l%32;
  // the bias and the mask values are loaded before the first store
  float bias[F];
#pragma unroll
  for (int j = 0; j < F; ++j)
    bias[j] = ep.bias ? ep.bias[min(n0 + wn * (T / 2) + j * 32 + (lane & 31), N - 1)] : 0.f;
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j) {
      const int gm0 = m0 + wm * (T / 2) + i * 32 + 4 * (lane >> 5), gn = n0 + wn * (T / 2) + j * 32 + (lane & 31);
      __bf16 mk[16];
      if (ep.mask) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          mk[r] = ep.mask[(size_t)min(gm0 + 8 * (r >> 2) + (r & 3), M - 1) * ep.ldm + min(gn, N - 1)];
      }
      if (gn < N) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int gm = gm0 + 8 * (r >> 2) + (r & 3);
          float v = acc[i][j][r];
          if (ep.bias) v += bias[j];
          if (ep.relu) v = fmaxf(v, 0.f);
          if (ep.mask && !((float)mk[r] > 0.f)) v = 0.f;
          if (gm < M && ep.c32) ep.c32[(size_t)gm * ep.ldc + gn] = v;
          if (gm < M && ep.cbf) ep.cbf[(size_t)gm * ep.ldcb + gn] = (__bf16)v;
        }
      }
    }
}

template <int TA, int TB, int T, int BK, int DEEP>
__global__ void __launch_bounds__(256, DEEP ? 2 : 3)
k_gemm(int M, int N, int K, const __bf16* __restrict__ A, int lda, const __bf16* __restrict__ B, int ldb,
       GemmEpi ep) {
  __shared__ GemmLds<T, BK, DEEP> L;
  gemm_tile<TA, TB, T, BK, DEEP>(L, blockIdx.x, blockIdx.y, M, N, K, A, lda, B, ldb, ep);
}

// Two products that do not depend on each other in one launch: the first n1
// blocks compute A^T B, the rest A B^T.  A training step's second-layer weight
// gradient has 64 tiles, which would leave three CUs of four idle on its own.
struct GemmArgs {
  int M, N, K;
  const __bf16* A;
  int lda;
  const __bf16* B;
  int ldb;
  GemmEpi ep;
};
__global__ void __launch_bounds__(256) k_gemm_pair(GemmArgs tn, GemmArgs nt, int n1) {
  __shared__ GemmLds<64, 128, 1> L;
  const int b = blockIdx.x;
  if (b < n1) {
    const int w = (tn.N + 63) / 64;
    gemm_tile<1, 0, 64, 128, 1>(L, b % w, b / w, tn.M, tn.N, tn.K, tn.A, tn.lda, tn.B, tn.ldb, tn.ep);
  } else {
    const int w = (nt.N + 63) / 64;
    gemm_tile<0, 1, 64, 128, 1>(L, (b - n1) % w, (b - n1) / w, nt.M, nt.N, nt.K, nt.A, nt.lda, nt.B, nt.ldb, nt.ep);
  }
}

constexpr size_t kGemmFill = 256;   // blocks: one a CU

// The tile: 128 x 128 (a fragment feeds two MFMAs, half the LDS reads a flop)
// where those tiles give every CU a block, 64 x 64 below that.  Its flat form
// up to 512 k's (A B^T, 65,536 x 256: 512 k's 37.2 us against 40.2, 2,048 k's
// 118 against 109; A B at 512 and 1,024 k's 45.2 against 50.0 and 72.0 against
// 70.9), up to 128 where A is transposed and staging costs more (27.1 against
// 27.0 at 128, 36.7 against 33.9 at 256).
template <int TA, int TB>
static void launch_gemm(int M, int N, int K, const __bf16* a, int lda, const __bf16* b, int ldb, const GemmEpi& ep,
                        hipStream_t st) {
  auto tiles = [&](int t) { return dim3((N + t - 1) / t, (M + t - 1) / t); };
  const dim3 big = tiles(128);
  if ((size_t)big.x * big.y < kGemmFill)
    hipLaunchKernelGGL((k_gemm<TA, TB, 64, 128, 1>), tiles(64), dim3(256), 0, st, M, N, K, a, lda, b, ldb, ep);
  else if (K <= (TA ? 128 : 512))
    hipLaunchKernelGGL((k_gemm<TA, TB, 128, 64, 0>), big, dim3(256), 0, st, M, N, K, a, lda, b, ldb, ep);
  else
    hipLaunchKernelGGL((k_gemm<TA, TB, 128, 64, 1>), big, dim3(256), 0, st, M, N, K, a, lda, b, ldb, ep);
}

// dst[c][r] = src[r][c] for a rows x cols bf16 matrix (32 x 32 tiles through LDS)
__global__ void __launch_bounds__(256)
k_transpose_bf16(const __bf16* __restrict__ src, int rows, int cols, __bf16* __restrict__ dst) {
  __shared__ __bf16 t[32][33];
  const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8 threads
  for (int i = ty; i < 32; i += 8)
    if (r0 + i < rows && c0 + tx < cols) t[i][tx] = src[(size_t)(r0 + i) * cols + c0 + tx];
  __syncthreads();
  for (int i = ty; i < 32; i += 8)
    if (c0 + i < cols && r0 + tx < rows) dst[(size_t)(c0 + i) * rows + r0 + tx] = t[tx][i];
}

// ---------------------------------------------------------------------------
// the 2-wide output layer, loss and its gradient
// ---------------------------------------------------------------------------
// z[b][o] = sum_k h[b][k] w[k][o] + bias[o]; with targets y: per element
// either BCE-with-logits, dz = (sigmoid(z) - y) * scale (kind 0), or the
// squared error (z - y)^2 / 2, dz = (z - y) * scale (kind 1); loss summed
// into *loss.
//
// 64 rows a block, wave o on output o with a row per lane.  Each sum is one
// chain over k, so it is bound by the chain's latency; the rows and the weights
// are brought to LDS 256 k's at a time with every load in flight (a row per
// thread read two bytes at a time from HBM took 36 us for 1,024 rows, this
// takes 8.6 us with dh).  With dh (VEC, Kd <= 256) the block also writes
// dh[b][k] = (dz[b] . w[k]) where h[b][k] > 0, else 0, from the rows in LDS.
// VEC: rows are 16-byte aligned and Kd is a multiple of 8.
constexpr int kHeadRows = 64, kHeadK = 256;
template <bool VEC>
__global__ void __launch_bounds__(128)
k_head_forward(const __bf16* __restrict__ h, int Bn, int Kd, const float* __restrict__ w,
               const float* __restrict__ bias, float* __restrict__ z, const float* __restrict__ y,
               float* __restrict__ dz, float scale, float* __restrict__ loss, int kind, __bf16* __restrict__ dh) {
  __shared__ __bf16 t[kHeadRows][kHeadK + 8];
  __shared__ float sw[2][kHeadK];
  __shared__ float sd[2][kHeadRows];
  const int lane = threadIdx.x & 63, o = threadIdx.x >> 6;
  const int b0 = blockIdx.x * kHeadRows, b = b0 + lane, rows = min(kHeadRows, Bn - b0);
  float v = bias[o];
  for (int k0 = 0; k0 < Kd; k0 += kHeadK) {
    const int kn = min(kHeadK, Kd - k0);
    if (k0) __syncthreads();
    for (int i = threadIdx.x; i < 2 * kn; i += 128) sw[i & 1][i >> 1] = w[2 * (size_t)k0 + i];
    if constexpr (VEC) {
      bf16x8 r[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int c = threadIdx.x + 128 * i, row = min(c >> 5, rows - 1), kk = min((c & 31) * 8, kn - 8);
        r[i] = *reinterpret_cast<const bf16x8*>(h + (size_t)(b0 + row) * Kd + k0 + kk);
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int c = threadIdx.x + 128 * i;
        *reinterpret_cast<bf16x8*>(&t[c >> 5][(c & 31) * 8]) = r[i];
      }
    } else {
      for (int i = threadIdx.x; i < rows * kn; i += 128) t[i / kn][i % kn] = h[(size_t)(b0 + i / kn) * Kd + k0 + i % kn];
    }
    __syncthreads();
    int k = 0;
#pragma unroll 4
    for (; k + 8 <= kn; k += 8) {
      const bf16x8 hv = *reinterpret_cast<const bf16x8*>(&t[lane][k]);
#pragma unroll
      for (int i = 0; i < 8; ++i) v = fmaf((float)hv[i], sw[o][k + i], v);
    }
    for (; k < kn; ++k) v = fmaf((float)t[lane][k], sw[o][k], v);
  }
  float l = 0.f;
  if (b < Bn) {
    z[2 * b + o] = v;
    if (y) {
      const float q = y[2 * b + o];
      float d;
      if (kind == 0) {
        l = fmaxf(v, 0.f) - v * q + log1pf(expf(-fabsf(v)));
        d = (1.f / (1.f + expf(-v)) - q) * scale;
      } else {
        l = 0.5f * (v - q) * (v - q);
        d = (v - q) * scale;
      }
      dz[2 * b + o] = d;
      sd[o][lane] = d;
    } else if (dh) {
      sd[o][lane] = dz[2 * b + o];
    }
  }
  if (y && loss) {
    for (int d = 32; d >= 1; d >>= 1) l += __shfl_xor(l, d, 64);
    if (lane == 0) atomicAdd(loss, l);
  }
  if constexpr (VEC) {
    if (!dh) return;
    __syncthreads();
    const int k = (threadIdx.x & 31) * 8;   // eight columns of every fourth row
    if (k >= Kd) return;
    float w0[8], w1[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) w0[i] = sw[0][k + i], w1[i] = sw[1][k + i];
    for (int r = threadIdx.x >> 5; r < rows; r += 4) {
      const bf16x8 hv = *reinterpret_cast<const bf16x8*>(&t[r][k]);
      const float d0 = sd[0][r], d1 = sd[1][r];
      bf16x8 q;
#pragma unroll
      for (int i = 0; i < 8; ++i) q[i] = (__bf16)((float)hv[i] > 0.f ? fmaf(d0, w0[i], d1 * w1[i]) : 0.f);
      *reinterpret_cast<bf16x8*>(dh + (size_t)(b0 + r) * Kd + k) = q;
    }
  }
}

static void launch_head(const __bf16* h, int Bn, int Kd, const float* w, const float* bias, float* z, const float* y,
                        float* dz, float scale, float* loss, int kind, __bf16* dh, hipStream_t st) {
  const dim3 grid((Bn + kHeadRows - 1) / kHeadRows);
  if (Kd % 8 == 0 && reinterpret_cast<uintptr_t>(h) % 16 == 0)
    hipLaunchKernelGGL(k_head_forward<true>, grid, dim3(128), 0, st, h, Bn, Kd, w, bias, z, y, dz, scale, loss, kind, dh);
  else
    hipLaunchKernelGGL(k_head_forward<false>, grid, dim3(128), 0, st, h, Bn, Kd, w, bias, z, y, dz, scale, loss, kind, dh);
}

// predicted F1 of each candidate from its two outputs, F1 = 2p / (p + q + |P|),
// with (P_b, N_b) the candidate's base coverage (its parent's) or (|P|, |Ng|):
//   kind 0: the outputs are logits of the kept shares, p = sigmoid(z0) P_b,
//           q = sigmoid(z1) N_b;
//   kind 1: the outputs are log(1 + removed count), p = P_b - expm1(z0) and
//           q = N_b - expm1(z1), each clamped to [0, base].
__device__ __forceinline__ float predicted_f1(float z0, float z1, float bp, float bn, float n_pos, int kind) {
  float p, q;
  if (kind == 0) {
    p = bp / (1.f + expf(-z0));
    q = bn / (1.f + expf(-z1));
  } else {
    p = fminf(fmaxf(bp - expm1f(fmaxf(z0, 0.f)), 0.f), bp);
    q = fminf(fmaxf(bn - expm1f(fmaxf(z1, 0.f)), 0.f), bn);
  }
  const float den = p + q + n_pos;
  return den > 0.f ? 2.f * p / den : 0.f;
}
__global__ void k_head_score(const float* __restrict__ z, int Bn, float n_pos, float n_neg,
                             const uint32_t* __restrict__ base, int kind, float* __restrict__ score) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= Bn) return;
  const float bp = base ? (float)base[2 * b] : n_pos, bn = base ? (float)base[2 * b + 1] : n_neg;
  score[b] = predicted_f1(z[2 * b], z[2 * b + 1], bp, bn, n_pos, kind);
}

// ---------------------------------------------------------------------------
// scoring: from feature lists to predicted F1 in one kernel
// ---------------------------------------------------------------------------
// A row's features are a handful of the 4,096 (a refinement minus its parent:
// about five), so the first layer is a sum of that many rows of W1, not a
// dense product: k_densify and a 4096-wide GEMM wrote and read 8 KB a row for
// it and did 400 times the multiplications.  The products of a small integer
// and a bf16 weight are exact in fp32 and so few that their sum is too but for
// far apart exponents, so both forms agree.
//
// A block takes 32 rows in three steps, all in LDS: (1) each wave lists the
// net feature counts of four rows (equal features merged, as in the dense row;
// counts rounded to bf16 as there) and adds their W1 rows, 16 columns a lane,
// four rows of W1 in flight; bias, ReLU, bf16; (2) the waves multiply the 32
// rows by 32 columns of W2 each on MFMA, W2's fragments straight from L2, eight
// ahead; (3) the output layer and the F1.  Two blocks
// share a CU, so one's loads overlap the other's products.
// Bound by the latency of the lists and of the W1 rows (2 KB each, most from
// L2).  262,157 rows: 489 us, where features apart the chain of densify, GEMMs,
// head and score took 5.2 ms (33 batches of 8,192).
constexpr int kScoreRows = 32, kScoreWaves = 8, kScoreH1 = 1024, kScoreLd = kScoreH1 + 8;
struct ScoreArgs {
  const uint16_t *feat, *pfeat;
  const uint32_t *offs, *poffs, *pidx;   // pfeat, poffs, pidx null: features of the rows themselves
  uint32_t row0, n_rows, context;
  const __bf16* w1;                      // [4096][1024]
  const bf16x8* w2f;                     // W2's fragments (k_score_pack)
  const float *b1, *b2, *w3, *b3;
  float n_pos, n_neg;
  const uint32_t* base;
  int kind;
  float* score;
};
// W2^T [256][1024] as k_score_rows' MFMA operands: fragment (32 columns, 16 k's)
// after fragment, each 64 lanes x 16 bytes, so a wave reads whole lines (read
// from w2t directly, 32 bytes of each of 32 lines, the kernel took 822 us).
__global__ void __launch_bounds__(256) k_score_pack(const __bf16* __restrict__ w2t, bf16x8* __restrict__ out) {
  const int i = blockIdx.x * 256 + threadIdx.x, lane = i & 63, ks = (i >> 6) % (kScoreH1 / 16), cb = (i >> 6) / (kScoreH1 / 16);
  out[i] = *reinterpret_cast<const bf16x8*>(w2t + (size_t)(cb * 32 + (lane & 31)) * kScoreH1 + 16 * ks + 8 * (lane >> 5));
}

__global__ void __launch_bounds__(64 * kScoreWaves) k_score_rows(ScoreArgs S) {
  extern __shared__ __bf16 lds[];
  __bf16(*t)[kScoreLd] = reinterpret_cast<__bf16(*)[kScoreLd]>(lds);       // the rows' h1, then h2
  __shared__ uint32_t s_list[kScoreWaves][4][64];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t r0 = blockIdx.x * kScoreRows;
  // ---- 1: h1, four rows a wave
  uint32_t b[4], n1[4], pb[4], n2[4], total[4], most = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t row = S.row0 + min(r0 + 4 * wv + j, S.n_rows - 1);
    b[j] = S.offs[row], n1[j] = S.offs[row + 1] - b[j];
    pb[j] = n2[j] = 0;
    if (S.pidx) {
      const uint32_t p = S.pidx[row];
      pb[j] = S.poffs[p], n2[j] = S.poffs[p + 1] - pb[j];
    }
    total[j] = n1[j] + n2[j] + (S.context ? n2[j] : 0u);
    most = max(most, total[j]);
  }
  // a row's entry i: feature index in the low bits, bit 31 set where it counts -1
  auto entry = [&](int j, uint32_t i) -> uint32_t {
    if (i < n1[j]) return S.feat[b[j] + i] & (kFeatDim - 1);
    if (i < n1[j] + n2[j]) return (S.pfeat[pb[j] + i - n1[j]] & (kFeatDim - 1)) | 0x80000000u;
    return (S.pfeat[pb[j] + i - n1[j] - n2[j]] & (kFeatDim - 1)) ^ (kFeatDim / 2);
  };
  // the lanes' net counts of their features f as (feature, bf16 count) in the row's list; -> how many
  auto list = [&](int j, bool keep, uint32_t f, int net) -> int {
    keep = keep && net != 0;
    const uint64_t m = __ballot(keep);
    if (keep)
      s_list[wv][j][__popcll(m & ((1ull << lane) - 1))] =
          f | (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)(float)net) << 16;
    __builtin_amdgcn_wave_barrier();
    return __popcll(m);
  };
  // a row of at most 64 entries (mine: this lane's): each feature at its first entry
  auto merge = [&](int j, uint32_t mine) -> int {
    const uint32_t f = mine & 0xFFFFu;
    int net = 0;
    bool first = (uint32_t)lane < total[j];
    for (uint32_t i = 0; i < total[j]; ++i) {
      const uint32_t e = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)i);
      const bool same = (e & 0xFFFFu) == f;
      net += same ? (int)(1 - 2 * (e >> 31)) : 0;
      first = first && !(same && i < (uint32_t)lane);
    }
    return list(j, first, f, net);
  };
  auto add_rows = [&](int j, int n, float (&acc)[16]) {
    for (int i = 0; i < n; i += 4) {
      bf16x8 w[4][2];
      float c[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t e = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_list[wv][j][min(i + u, n - 1)]);
        c[u] = __builtin_bit_cast(float, e & 0xFFFF0000u);
        const __bf16* wr = S.w1 + (size_t)(e & 0xFFFFu) * kScoreH1 + 8 * lane;
        if (i + u < n) {
          w[u][0] = *reinterpret_cast<const bf16x8*>(wr);
          w[u][1] = *reinterpret_cast<const bf16x8*>(wr + kScoreH1 / 2);
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (i + u < n) {
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            acc[k] = fmaf(c[u], (float)w[u][0][k], acc[k]);
            acc[8 + k] = fmaf(c[u], (float)w[u][1][k], acc[8 + k]);
          }
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
  };
  // a longer row: counted feature range by range in the LDS that its h1 takes
  // afterwards, work per entry and not per pair of entries (65,536 rows of 256
  // features 1.7 ms, of 512 entries that mostly cancel 0.54; with every entry
  // compared with every other 5.6 and 11.9)
  auto add_long_row = [&](int j, float (&acc)[16]) {
    constexpr uint32_t kRange = kScoreH1 * sizeof(__bf16) / sizeof(int32_t);
    typedef int32_t __attribute__((may_alias)) Count;
    Count* cnt = reinterpret_cast<Count*>(&t[4 * wv + j][0]);
    auto sync = [] {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    for (uint32_t f0 = 0; f0 < kFeatDim; f0 += kRange) {
      for (uint32_t i = lane; i < kRange; i += 64) cnt[i] = 0;
      sync();
#pragma unroll 4
      for (uint32_t i = lane; i < total[j]; i += 64) {
        const uint32_t e = entry(j, i), d = (e & 0xFFFFu) - f0;
        if (d < kRange) __hip_atomic_fetch_add(cnt + d, (int32_t)(1 - 2 * (e >> 31)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
      }
      sync();
      for (uint32_t k = lane; k < kRange; k += 64) add_rows(j, list(j, true, f0 + k, cnt[k]), acc);
      sync();
    }
  };
  float b1[16];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    b1[i] = S.b1[8 * lane + i];
    b1[8 + i] = S.b1[kScoreH1 / 2 + 8 * lane + i];
  }
  int n[4] = {0, 0, 0, 0};
  if (most <= 64) {                       // the four lists first: their loads overlap
    uint32_t mine[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) mine[j] = (uint32_t)lane < total[j] ? entry(j, lane) : 0xFFFFu;
#pragma unroll
    for (int j = 0; j < 4; ++j) n[j] = merge(j, mine[j]);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float acc[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    if (total[j] > 64) {
      add_long_row(j, acc);
    } else {
      if (most > 64) n[j] = merge(j, (uint32_t)lane < total[j] ? entry(j, lane) : 0xFFFFu);
      add_rows(j, n[j], acc);
    }
    bf16x8 h[2];
#pragma unroll
    for (int i = 0; i < 16; ++i) h[i >> 3][i & 7] = (__bf16)fmaxf(acc[i] + b1[i], 0.f);
    *reinterpret_cast<bf16x8*>(&t[4 * wv + j][8 * lane]) = h[0];
    *reinterpret_cast<bf16x8*>(&t[4 * wv + j][kScoreH1 / 2 + 8 * lane]) = h[1];
  }
  __syncthreads();
  // ---- 2: h2 = relu(h1 W2 + b2), 32 columns a wave, k in rising steps of 16
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  const int col = wv * 32 + (lane & 31);
  {
    const bf16x8* wr = S.w2f + (size_t)wv * (kScoreH1 / 16) * 64 + lane;
    bf16x8 w[2][8];
#pragma unroll
    for (int u = 0; u < 8; ++u) w[0][u] = wr[64 * u];
#pragma unroll 2
    for (int g = 0; g < kScoreH1 / 128; ++g) {
#pragma unroll
      for (int u = 0; u < 8; ++u) w[(g + 1) & 1][u] = wr[64 * ((g + 1 < kScoreH1 / 128 ? 8 * (g + 1) : 0) + u)];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(&t[lane & 31][128 * g + 16 * u + 8 * (lane >> 5)]);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, w[g & 1][u], acc, 0, 0, 0);
      }
    }
  }
  __syncthreads();
  const float b2 = S.b2[col];
#pragma unroll
  for (int r = 0; r < 16; ++r) t[8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)][col] = (__bf16)fmaxf(acc[r] + b2, 0.f);
  __syncthreads();
  // ---- 3: a row per 16 lanes, 16 k's each
  const int j = threadIdx.x >> 4, part = threadIdx.x & 15;
  float z0 = 0.f, z1 = 0.f;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const bf16x8 h = *reinterpret_cast<const bf16x8*>(&t[j][16 * part + 8 * i]);
    const float* w3 = S.w3 + 2 * (16 * part + 8 * i);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      z0 = fmaf((float)h[k], w3[2 * k], z0);
      z1 = fmaf((float)h[k], w3[2 * k + 1], z1);
    }
  }
#pragma unroll
  for (int d = 8; d >= 1; d >>= 1) {
    z0 += __shfl_xor(z0, d, 64);
    z1 += __shfl_xor(z1, d, 64);
  }
  if (part == 0 && r0 + j < S.n_rows) {
    const uint32_t r = r0 + j;
    const float bp = S.base ? (float)S.base[2 * (size_t)r] : S.n_pos, bn = S.base ? (float)S.base[2 * (size_t)r + 1] : S.n_neg;
    S.score[r] = predicted_f1(z0 + S.b3[0], z1 + S.b3[1], bp, bn, S.n_pos, S.kind);
  }
}

// The output layer's weight gradient and dh for a caller's own chain: a block
// per k, dw[k] as 256 chains b, b + 256, ... added as a binary tree (the order
// of k_colred below), and dh[b][k] = (dz[b] . w[k]) * (h[b][k] > 0) in the same
// pass.  Bound by one column's strided loads; a block per k keeps every CU at
// it: 65,536 x 256 take 188 us, against 977 as k_colred and a pass for dh,
// whose four blocks leave the chip idle (64 x 256: 7.5 us against 9.6).
__global__ void __launch_bounds__(256)
k_head_backward(const __bf16* __restrict__ h, int Bn, int Kd, const float* __restrict__ w,
                const float* __restrict__ dz, float* __restrict__ dw, __bf16* __restrict__ dh) {
  const int k = blockIdx.x;
  float s0 = 0.f, s1 = 0.f;
  const float w0 = w[2 * k], w1 = w[2 * k + 1];
  for (int b = threadIdx.x; b < Bn; b += 256) {
    const float hv = (float)h[(size_t)b * Kd + k];
    const float d0 = dz[2 * (size_t)b], d1 = dz[2 * (size_t)b + 1];
    s0 = fmaf(hv, d0, s0);
    s1 = fmaf(hv, d1, s1);
    dh[(size_t)b * Kd + k] = (__bf16)(hv > 0.f ? fmaf(d0, w0, d1 * w1) : 0.f);
  }
  __shared__ float r0[256], r1[256];
  r0[threadIdx.x] = s0;
  r1[threadIdx.x] = s1;
  __syncthreads();
  for (int d = 128; d >= 1; d >>= 1) {
    if (threadIdx.x < d) {
      r0[threadIdx.x] += r0[threadIdx.x + d];
      r1[threadIdx.x] += r1[threadIdx.x + d];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    dw[2 * k] = r0[0];
    dw[2 * k + 1] = r1[0];
  }
}

// Sums over the rows of row-major [M][N] matrices, several in one launch, each
// in an order fixed by (M, N):
// - column sums (bias gradients) of bf16 or fp32 values: four chains a column,
//   rows c, c + 4, ...; ((0 + 1) + 2) + 3.  A wave holds 64 columns of one
//   chain, a block 64 columns for every four of its waves;
// - with dz, the output layer's weight gradient out[n][o] = sum_m a[m][n]
//   dz[m][o]: 256 chains a column, rows t, t + 256, ..., added as a binary tree
//   (t with t + 128, + 64, ...).  A wave holds chains w, w + 16, ... of 64
//   columns in registers, a block 64 columns.
// Bound by the chains' row loads, 32 in flight (16 us for a training step's
// four at M = 1,024; launches of their own took 25 us).
constexpr int kRedWaves = 16, kRedAhead = 32;
struct RedTask {
  const void* a;
  const float* dz;     // [M][2] or null
  float* out;
  int M, N, f32;       // f32: a holds fp32 values
  int block0;          // first block of the task
};
struct RedTasks {
  RedTask t[4];
  int n;
};
template <typename T>
__device__ __forceinline__ float red_chain(const T* __restrict__ a, int M, int N, int c) {
  float s = 0.f;
  int m = c;
  for (; m + 4 * (kRedAhead - 1) < M; m += 4 * kRedAhead) {
    T v[kRedAhead];
#pragma unroll
    for (int i = 0; i < kRedAhead; ++i) v[i] = a[(size_t)(m + 4 * i) * N];
#pragma unroll
    for (int i = 0; i < kRedAhead; ++i) s += (float)v[i];
  }
  for (; m < M; m += 4) s += (float)a[(size_t)m * N];
  return s;
}
__global__ void __launch_bounds__(64 * kRedWaves) k_colred(RedTasks ts) {
  __shared__ float part[2][kRedWaves][64];
  int i = 0;
  while (i + 1 < ts.n && (int)blockIdx.x >= ts.t[i + 1].block0) ++i;
  const RedTask T = ts.t[i];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), b = blockIdx.x - T.block0;
  if (!T.dz) {
    const int n = b * (blockDim.x >> 2) + (wv >> 2) * 64 + lane;
    float s = 0.f;
    if (n < T.N)
      s = T.f32 ? red_chain(static_cast<const float*>(T.a) + n, T.M, T.N, wv & 3)
                : red_chain(static_cast<const __bf16*>(T.a) + n, T.M, T.N, wv & 3);
    part[0][wv][lane] = s;
    __syncthreads();
    if ((wv & 3) == 0 && n < T.N)
      T.out[n] = ((part[0][wv][lane] + part[0][wv + 1][lane]) + part[0][wv + 2][lane]) + part[0][wv + 3][lane];
    return;
  }
  const int n = b * 64 + lane;
  float s[2][16];
#pragma unroll
  for (int j = 0; j < 16; ++j) s[0][j] = s[1][j] = 0.f;
  if (n < T.N) {
    const __bf16* a = static_cast<const __bf16*>(T.a) + n;
    for (int m0 = wv; m0 < T.M; m0 += 256) {
      float v[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) v[j] = (float)a[(size_t)min(m0 + 16 * j, T.M - 1) * T.N];
#pragma unroll
      for (int j = 0; j < 16; ++j)
        if (m0 + 16 * j < T.M) {
          s[0][j] = fmaf(v[j], T.dz[2 * (size_t)(m0 + 16 * j)], s[0][j]);
          s[1][j] = fmaf(v[j], T.dz[2 * (size_t)(m0 + 16 * j) + 1], s[1][j]);
        }
    }
  }
#pragma unroll
  for (int o = 0; o < 2; ++o) {
#pragma unroll
    for (int d = 8; d >= 1; d >>= 1)
#pragma unroll
      for (int j = 0; j < d; ++j) s[o][j] += s[o][j + d];
    part[o][wv][lane] = s[o][0];
  }
  __syncthreads();
  for (int d = 8; d >= 1; d >>= 1) {
    if (wv < d) {
      part[0][wv][lane] += part[0][wv + d][lane];
      part[1][wv][lane] += part[1][wv + d][lane];
    }
    __syncthreads();
  }
  if (wv < 2 && n < T.N) T.out[2 * n + wv] = part[wv][0][lane];
}
// waves a block: 16, which the weight gradient needs, or 4
static void launch_colred(RedTasks& ts, int waves, hipStream_t st) {
  int blocks = 0;
  for (int i = 0; i < ts.n; ++i) {
    const int cols = ts.t[i].dz ? 64 : 16 * waves;
    ts.t[i].block0 = blocks;
    blocks += (ts.t[i].N + cols - 1) / cols;
  }
  hipLaunchKernelGGL(k_colred, dim3(blocks), dim3(64 * waves), 0, st, ts);
}

// AdamW on fp32 master weights (decoupled weight decay), with a bf16 copy
struct AdamArgs {
  float lr, b1, b2, eps, c1, c2;   // c1, c2: 1 - b^step
};
__device__ __forceinline__ void adamw_update(float& p, float g, float& m, float& v, const AdamArgs& A, float wd) {
  m = A.b1 * m + (1.f - A.b1) * g;
  v = A.b2 * v + (1.f - A.b2) * g * g;
  const float mh = m / A.c1, vh = v / A.c2;
  p = p * (1.f - A.lr * wd);
  p -= A.lr * mh / (sqrtf(vh) + A.eps);
}
__global__ void k_adamw(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                        float* __restrict__ v, __bf16* __restrict__ pbf, size_t n, AdamArgs A, float wd) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t step = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += step) {
    adamw_update(p[i], g[i], m[i], v[i], A, wd);
    if (pbf) pbf[i] = (__bf16)p[i];
  }
}

// All tensors of a training step in one launch.  A weight matrix with a bf16
// copy goes by 64 x 64 tiles, a thread on four consecutive columns of four
// rows; the tile's bf16 values pass through LDS so that the transposed copy
// (pt, the layout that the forward products read) is written with it in
// 16-byte stores.  The small tensors take an element per thread.  Bound by HBM
// and the L3: 30 bytes a parameter (p, g, m, v read; p, m, v and two bf16
// copies written), 23.4 us for 4.5M parameters; six launches and two transposes
// took 45 us.
struct AdamTask {
  float *p, *m, *v;
  const float* g;
  __bf16 *pb, *pt;     // [rows][cols] and [cols][rows], or null
  int rows, cols;
  float wd;
  int block0;
};
struct AdamTasks {
  AdamTask t[6];
};
__global__ void __launch_bounds__(256) k_adamw_all(AdamTasks ts, AdamArgs A) {
  __shared__ __bf16 tile[64][64 + 2];
  int i = 0;
  while (i < 5 && (int)blockIdx.x >= ts.t[i + 1].block0) ++i;
  const AdamTask T = ts.t[i];
  const int b = blockIdx.x - T.block0;
  if (!T.pb) {
    const int e = b * 256 + threadIdx.x;
    if (e < T.rows * T.cols) adamw_update(T.p[e], T.g[e], T.m[e], T.v[e], A, T.wd);
    return;
  }
  const int r0 = b / (T.cols / 64) * 64, c0 = b % (T.cols / 64) * 64;
  const int cc = (threadIdx.x & 15) * 4;
  float4 p[4], g[4], m[4], v[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const size_t at = (size_t)(r0 + (threadIdx.x >> 4) + 16 * j) * T.cols + c0 + cc;
    p[j] = *reinterpret_cast<const float4*>(T.p + at);
    g[j] = *reinterpret_cast<const float4*>(T.g + at);
    m[j] = *reinterpret_cast<const float4*>(T.m + at);
    v[j] = *reinterpret_cast<const float4*>(T.v + at);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = (threadIdx.x >> 4) + 16 * j;
    const size_t at = (size_t)(r0 + r) * T.cols + c0 + cc;
    adamw_update(p[j].x, g[j].x, m[j].x, v[j].x, A, T.wd);
    adamw_update(p[j].y, g[j].y, m[j].y, v[j].y, A, T.wd);
    adamw_update(p[j].z, g[j].z, m[j].z, v[j].z, A, T.wd);
    adamw_update(p[j].w, g[j].w, m[j].w, v[j].w, A, T.wd);
    *reinterpret_cast<float4*>(T.p + at) = p[j];
    *reinterpret_cast<float4*>(T.m + at) = m[j];
    *reinterpret_cast<float4*>(T.v + at) = v[j];
    bf16x4 q;
    q[0] = (__bf16)p[j].x, q[1] = (__bf16)p[j].y, q[2] = (__bf16)p[j].z, q[3] = (__bf16)p[j].w;
    *reinterpret_cast<bf16x4*>(T.pb + at) = q;
#pragma unroll
    for (int e = 0; e < 4; ++e) tile[r][cc + e] = q[e];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int c = (threadIdx.x >> 3) + 32 * j, rr = (threadIdx.x & 7) * 8;
    bf16x8 q;
#pragma unroll
    for (int e = 0; e < 8; ++e) q[e] = tile[rr + e][c];
    *reinterpret_cast<bf16x8*>(T.pt + (size_t)(c0 + c) * T.rows + r0 + rr) = q;
  }
}

__global__ void k_to_bf16(const float* __restrict__ s, __bf16* __restrict__ d, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t step = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += step) d[i] = (__bf16)s[i];
}

// ---------------------------------------------------------------------------
// top-k by a float score: radix select on the order-preserving key (11, 11 and
// 10 bits), then a compaction
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t fkey(float f) {
  uint32_t u;
  memcpy(&u, &f, 4);
  if (f != f) return 0;                       // NaN ranks last
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// The work area: three histograms and two counters, in this order.  Digit d of
// a key covers bits [kTopShift[d], kTopShift[d] + 11) (the last one 10 bits).
constexpr int kTopBins = 2048, kTopWords = 3 * kTopBins + 2;
__device__ __forceinline__ int top_shift(int d) { return d == 0 ? 21 : d == 1 ? 10 : 0; }

// The first `digits` digits of the k-th largest key, from their histograms;
// need: how many keys are still to take among those that share them.  A whole
// block of 256 threads, every thread with the same answer.
__device__ uint32_t top_prefix(const uint32_t* __restrict__ work, int digits, uint32_t& need) {
  __shared__ uint32_t s_sum[256], s_pick[2];
  uint32_t prefix = 0;
  for (int d = 0; d < digits; ++d) {
    const uint32_t* h = work + d * kTopBins;
    // thread t holds bins 2047 - 8t down to 2040 - 8t
    uint32_t c[8], s = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) s += c[i] = h[kTopBins - 1 - (8 * threadIdx.x + i)];
    s_sum[threadIdx.x] = s;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
      const uint32_t v = threadIdx.x >= o ? s_sum[threadIdx.x - o] : 0;
      __syncthreads();
      s_sum[threadIdx.x] += v;
      __syncthreads();
    }
    uint32_t before = s_sum[threadIdx.x] - s;
    if (before < need && before + s >= need) {
      int i = 0;
      while (before + c[i] < need) before += c[i++];
      s_pick[0] = kTopBins - 1 - (8 * threadIdx.x + i);
      s_pick[1] = need - before;
    }
    __syncthreads();
    prefix |= s_pick[0] << top_shift(d);
    need = s_pick[1];
    __syncthreads();
  }
  return prefix;
}

// Histogram of digit d among the keys that share the k-th largest key's digits
// before it.  Counted in LDS and added once per block and bin: scores of one
// beam share their leading bits, and 65,536 global bins took 237 us a pass for
// 262,157 of them, all on a few counters (30 us for the whole selection now).
__global__ void __launch_bounds__(256)
k_topk_hist(const float* __restrict__ s, uint32_t n, uint32_t k, int d, uint32_t* __restrict__ work) {
  __shared__ uint32_t s_hist[kTopBins];
  for (int i = threadIdx.x; i < kTopBins; i += 256) s_hist[i] = 0;
  uint32_t need = k;
  const uint32_t prefix = top_prefix(work, d, need);
  __syncthreads();
  const int sh = top_shift(d), up = d == 0 ? 32 : top_shift(d - 1);
  const uint32_t mask = d == 2 ? 1023u : 2047u;
  for (size_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const uint32_t key = fkey(s[i]);
    if (d == 0 || (key >> up) == (prefix >> up)) atomicAdd(&s_hist[(key >> sh) & mask], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kTopBins; i += 256)
    if (s_hist[i]) atomicAdd(work + d * kTopBins + i, s_hist[i]);
}

// Keys above the k-th largest go out, and as many equal ones as are left to
// take (which ones is the counter's order).
__global__ void __launch_bounds__(256)
k_topk_collect(const float* __restrict__ s, uint32_t n, uint32_t k, uint32_t* __restrict__ work,
               uint32_t* __restrict__ out) {
  uint32_t take = k;
  const uint32_t thr = top_prefix(work, 3, take);
  uint32_t* cnt = work + 3 * kTopBins;
  for (size_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const uint32_t key = fkey(s[i]);
    bool go = key > thr;
    if (key == thr) go = atomicAdd(&cnt[1], 1u) < take;
    if (go) out[atomicAdd(&cnt[0], 1u)] = (uint32_t)i;
  }
}

__global__ void k_topk_clear(uint32_t* __restrict__ work) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < kTopWords) work[i] = 0;
}

}  // namespace hth

using namespace hth;

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
extern "C" hth_status hth_features(const hth_node* d_nodes, const uint32_t* d_hyp_node_offsets,
                                   uint32_t n_hyps, const uint32_t* d_children, uint32_t n_children,
                                   uint64_t* d_hash, uint16_t* d_feat, uint32_t* d_bad, void* stream) {
  if (!d_nodes || !d_hyp_node_offsets || !d_hash || !d_feat || !d_bad)
    return fail(HTH_E_INVALID, "NULL argument");
  if (n_children && !d_children) return fail(HTH_E_INVALID, "children is NULL");
  if (!n_hyps) return HTH_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  HTH_HIP(hipMemsetAsync(d_bad, 0, 4, st));
  hipLaunchKernelGGL(k_features, dim3((n_hyps + kFeatHyps - 1) / kFeatHyps), dim3(256), 0, st, d_nodes,
                     d_hyp_node_offsets, d_children, n_children, n_hyps, d_hash, d_feat, d_bad);
  HTH_HIP(hipGetLastError());
  return HTH_OK;
}

extern "C" hth_status hth_densify(const uint16_t* d_feat, const uint32_t* d_hyp_node_offsets,
                                  uint32_t row0, uint32_t n_rows, uint16_t* d_x, void* stream) {
  if (!d_feat || !d_hyp_node_offsets || !d_x) return fail(HTH_E_INVALID, "NULL argument");
  if (!n_rows) return HTH_OK;
  hipLaunchKernelGGL(k_densify, dim3(n_rows), dim3(256), 0, static_cast<hipStream_t>(stream), d_feat,
                     d_hyp_node_offsets, row0, n_rows, nullptr, nullptr, nullptr, 0u,
                     reinterpret_cast<__bf16*>(d_x));
  HTH_HIP(hipGetLastError());
  return HTH_OK;
}

extern "C" hth_status hth_densify_delta(const uint16_t* d_feat, const uint32_t* d_hyp_node_offsets,
                                        uint32_t row0, uint32_t n_rows, const uint16_t* d_parent_feat,
                                        const uint32_t* d_parent_offsets, const uint32_t* d_parent_index,
                                        uint32_t parent_context, uint16_t* d_x, void* stream) {
  if (!d_feat || !d_hyp_node_offsets || !d_parent_feat || !d_parent_offsets || !d_parent_index || !d_x)
    return fail(HTH_E_INVALID, "NULL argument");
  if (parent_context > 1) return fail(HTH_E_RANGE, "parent_context must be 0 or 1");
  if (!n_rows) return HTH_OK;
  hipLaunchKernelGGL(k_densify, dim3(n_rows), dim3(256), 0, static_cast<hipStream_t>(stream), d_feat,
                     d_hyp_node_offsets, row0, n_rows, d_parent_feat, d_parent_offsets, d_parent_index,
                     parent_context, reinterpret_cast<__bf16*>(d_x));
  HTH_HIP(hipGetLastError());
  return HTH_OK;
}

extern "C" hth_status hth_gemm_bf16(int trans_a, int trans_b, int M, int N, int K, const uint16_t* A,
                                    int lda, const uint16_t* B, int ldb, const float* bias, int relu,
                                    const uint16_t* mask, int ldm, float* c32, int ldc, uint16_t* cbf,
                                    int ldcb, void* stream) {
  if (!A || !B || (!c32 && !cbf)) return fail(HTH_E_INVALID, "NULL argument");
  if (M <= 0 || N <= 0 || K <= 0) return fail(HTH_E_RANGE, "M, N, K must be positive");
  if ((trans_a == 0 && (K % 8 || lda % 8)) || (trans_a == 1 && (M % 8 || lda % 8)) ||
      (trans_b == 0 && (N % 8 || ldb % 8)) || (trans_b == 1 && (K % 8 || ldb % 8)))
    return fail(HTH_E_INVALID, "the contiguous dimension and leading dimensions must be multiples of 8");
  if ((reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(B)) % 16)
    return fail(HTH_E_INVALID, "A and B must be 16-byte aligned");
  if (trans_a == 1 && trans_b == 1) return fail(HTH_E_UNSUPPORTED, "A^T B^T is not provided");
  GemmEpi ep{bias, relu, reinterpret_cast<const __bf16*>(mask), ldm, c32, ldc,
             reinterpret_cast<__bf16*>(cbf), ldcb};
  hipStream_t st = static_cast<hipStream_t>(stream);
  const __bf16* a = reinterpret_cast<const __bf16*>(A);
  const __bf16* b = reinterpret_cast<const __bf16*>(B);
  if (trans_a == 0 && trans_b == 0) launch_gemm<0, 0>(M, N, K, a, lda, b, ldb, ep, st);
  else if (trans_a == 0) launch_gemm<0, 1>(M, N, K, a, lda, b, ldb, ep, st);
  else launch_gemm<1, 0>(M, N, K, a, lda, b, ldb, ep, st);
  HTH_HIP(hipGetLastError());
  return HTH_OK;
}

extern "C" hth_status hth_head_forward(const uint16_t* h, int Bn, int Kd, const float* w, const float* bias,
                                       float* z, const float* y, float* dz, float scale, float* loss,
                                       int loss_kind, void* stream) {
  if (!h || !w || !bias || !z || (y && !dz)) return fail(HTH_E_INVALID, "NULL argument");
  if (loss_kind != 0 && loss_kind != 1) return fail(HTH_E_RANGE, "loss_kind must be 0 or 1");
  if (Bn <= 0) return HTH_OK;
  launch_head(reinterpret_cast<const __bf16*>(h), Bn, Kd, w, bias, z, y, dz, scale, loss, loss_kind, nullptr,
              static_cast<hipStream_t>(stream));
  HTH_HIP(hipGetLastError());
  return HTH_OK;
}

extern "C" hth_status hth_head_score(const float* z, int Bn, float n_pos, float n_neg, const uint32_t* base,
                                     int kind, float* score, void* stream) {
  if (!z || !score) return fail(HTH_E_INVALID, "NULL argument");
  if (kind != 0 && kind != 1) return fail(HTH_E_RANGE, "kind must be 0 or 1");
  if (kind == 1 && !base) return fail(HTH_E_INVALID, "kind 1 needs the base coverage");
  if (Bn <= 0) return HTH_OK;
  hipLaunchKernelGGL(k_head_score, dim3((Bn + 255) / 256), dim3(256), 0, static_cast<hipStream_t>(stream),
                     z, Bn, n_pos, n_neg, base, kind, score);
  HTH_HIP(hipGetLastError());
  return HTH_OK;
}

extern "C" hth_status hth_head_backward(const uint16_t* h, int Bn, int Kd, const float* w, const float* dz,
                                        float* dw, uint16_t* dh, void* stream) {
  if (!h || !w || !dz || !dw || !dh) return fail(HTH_E_INVALID, "NULL argument");
  hipLaunchKernelGGL(k_head_backward, dim3(Kd), dim3(256), 0, static_cast<hipStream_t>(stream),
                     reinterpret_cast<const __bf16*>(h), Bn, Kd, w, dz, dw, reinterpret_cast<__bf16*>(dh));
  HTH_HIP(hipGetLastError());
  return HTH_OK;
}

extern "C" hth_status hth_colsum(const void* d, int is_bf16, int M, int N, float* out, void* stream) {
  if (M < 0 || N < 0) return fail(HTH_E_RANGE, "negative matrix size");
  if (!N) return HTH_OK;
  if (!out || (M && !d)) return fail(HTH_E_INVALID, "NULL argument");
  hipStream_t st = static_cast<hipStream_t>(stream);
  RedTasks ts{{{d, nullptr, out, M, N, !is_bf16, 0}}, 1};
  // 256 columns a block where those blocks fill the chip, 64 below that
  // (1,024 x 100,000: 35.6 us, 44.0 in blocks of 64; 8,192 x 1,024: 63 and 27)
  launch_colred(ts, N >= 256 * 256 ? kRedWaves : 4, st);
  HTH_HIP(hipGetLastError());
  return HTH_OK;
}

static AdamArgs adam_args(float lr, float beta1, float beta2, float eps, int step) {
  return AdamArgs{lr, beta1, beta2, eps, 1.f - std::pow(beta1, (float)step), 1.f - std::pow(beta2, (float)step)};
}

extern "C" hth_status hth_adamw(float* p, const float* g, float* m, float* v, uint16_t* pbf, size_t n,
                                float lr, float beta1, float beta2, float eps, float wd, int step,
                                void* stream) {
  if (!p || !g || !m || !v) return fail(HTH_E_INVALID, "NULL argument");
  if (step < 1) return fail(HTH_E_RANGE, "step counts from 1");
  const AdamArgs A = adam_args(lr, beta1, beta2, eps, step);
  const unsigned g_ = (unsigned)std::min<size_t>((n + 255) / 256, 8192);
  hipLaunchKernelGGL(k_adamw, dim3(std::max(1u, g_)), dim3(256), 0, static_cast<hipStream_t>(stream), p, g,
                     m, v, reinterpret_cast<__bf16*>(pbf), n, A, wd);
  HTH_HIP(hipGetLastError());
  return HTH_OK;
}

extern "C" hth_status hth_train_step(const hth_train* t, void* stream) {
  if (!t) return fail(HTH_E_INVALID, "NULL argument");
  const uint16_t* bufs[] = {t->x, t->w1b, t->w2b, t->w1t, t->w2t, t->h1, t->h2, t->dh1, t->dh2};
  for (const uint16_t* b : bufs) {
    if (!b) return fail(HTH_E_INVALID, "NULL argument");
    if (reinterpret_cast<uintptr_t>(b) % 16) return fail(HTH_E_INVALID, "bf16 buffers must be 16-byte aligned");
  }
  for (int i = 0; i < 6; ++i) {
    if (!t->p[i] || !t->g[i] || !t->m[i] || !t->v[i]) return fail(HTH_E_INVALID, "NULL argument");
    if ((reinterpret_cast<uintptr_t>(t->p[i]) | reinterpret_cast<uintptr_t>(t->g[i]) |
         reinterpret_cast<uintptr_t>(t->m[i]) | reinterpret_cast<uintptr_t>(t->v[i])) % 16)
      return fail(HTH_E_INVALID, "parameters must be 16-byte aligned");
  }
  if (!t->z || !t->dz) return fail(HTH_E_INVALID, "NULL argument");
  if (t->n <= 0 || t->step < 1) return fail(HTH_E_RANGE, "n must be positive and step counts from 1");
  if (t->loss_kind != 0 && t->loss_kind != 1) return fail(HTH_E_RANGE, "loss_kind must be 0 or 1");
  const int n = t->n, D = t->d_in, H1 = t->d_h1, H2 = t->d_h2;
  if (D <= 0 || H1 <= 0 || H2 <= 0 || D % 64 || H1 % 64 || H2 % 64 || H2 > kHeadK)
    return fail(HTH_E_UNSUPPORTED, "layer widths must be multiples of 64, the last at most 256");
  hipStream_t st = static_cast<hipStream_t>(stream);
  auto bf = [](const uint16_t* q) { return reinterpret_cast<const __bf16*>(q); };
  auto wr = [](uint16_t* q) { return reinterpret_cast<__bf16*>(q); };
  enum { W1, B1, W2, B2, W3, B3 };
  // forward
  launch_gemm<0, 1>(n, H1, D, bf(t->x), D, bf(t->w1t), D, GemmEpi{t->p[B1], 1, nullptr, 0, nullptr, 0, wr(t->h1), H1}, st);
  launch_gemm<0, 1>(n, H2, H1, bf(t->h1), H1, bf(t->w2t), H1, GemmEpi{t->p[B2], 1, nullptr, 0, nullptr, 0, wr(t->h2), H2}, st);
  launch_head(bf(t->h2), n, H2, t->p[W3], t->p[B3], t->z, t->y, t->dz, (float)(1.0 / (2.0 * n)), t->loss, t->loss_kind,
              wr(t->dh2), st);
  // backward: dW2 = h1^T dh2 beside dh1 = (dh2 W2^T) (h1 > 0), then dW1 = x^T dh1
  const GemmArgs tn{H1, H2, n, bf(t->h1), H1, bf(t->dh2), H2, GemmEpi{nullptr, 0, nullptr, 0, t->g[W2], H2, nullptr, 0}};
  const GemmArgs nt{n, H1, H2, bf(t->dh2), H2, bf(t->w2b), H2, GemmEpi{nullptr, 0, bf(t->h1), H1, nullptr, 0, wr(t->dh1), H1}};
  const int n1 = H1 / 64 * (H2 / 64), n2 = (n + 63) / 64 * (H1 / 64);
  hipLaunchKernelGGL(k_gemm_pair, dim3(n1 + n2), dim3(256), 0, st, tn, nt, n1);
  launch_gemm<1, 0>(D, H1, n, bf(t->x), D, bf(t->dh1), H1, GemmEpi{nullptr, 0, nullptr, 0, t->g[W1], H1, nullptr, 0}, st);
  RedTasks red{{{t->h2, t->dz, t->g[W3], n, H2, 0, 0},
                {t->dh1, nullptr, t->g[B1], n, H1, 0, 0},
                {t->dh2, nullptr, t->g[B2], n, H2, 0, 0},
                {t->dz, nullptr, t->g[B3], n, 2, 1, 0}}, 4};
  launch_colred(red, kRedWaves, st);
  const int rows[6] = {D, 1, H1, 1, H2, 1}, cols[6] = {H1, H1, H2, H2, 2, 2};
  AdamTasks ts;
  int blocks = 0;
  for (int i = 0; i < 6; ++i) {
    const bool tiled = i == W1 || i == W2;
    ts.t[i] = AdamTask{t->p[i], t->m[i], t->v[i], t->g[i], i == W1 ? wr(t->w1b) : i == W2 ? wr(t->w2b) : nullptr,
                       i == W1 ? wr(t->w1t) : i == W2 ? wr(t->w2t) : nullptr, rows[i], cols[i],
                       i % 2 == 0 ? t->wd : 0.f, blocks};
    blocks += tiled ? rows[i] / 64 * (cols[i] / 64) : (rows[i] * cols[i] + 255) / 256;
  }
  hipLaunchKernelGGL(k_adamw_all, dim3(blocks), dim3(256), 0, st, ts,
                     adam_args(t->lr, t->beta1, t->beta2, t->eps, t->step));
  HTH_HIP(hipGetLastError());
  return HTH_OK;
}

extern "C" hth_status hth_transpose_bf16(const uint16_t* src, int rows, int cols, uint16_t* dst, void* stream) {
  if (!src || !dst) return fail(HTH_E_INVALID, "NULL argument");
  if (rows <= 0 || cols <= 0) return fail(HTH_E_RANGE, "rows and cols must be positive");
  if (src == dst) return fail(HTH_E_INVALID, "the transpose is not in place");
  const dim3 grid((cols + 31) / 32, (rows + 31) / 32), block(256);
  hipLaunchKernelGGL(k_transpose_bf16, grid, block, 0, static_cast<hipStream_t>(stream),
                     reinterpret_cast<const __bf16*>(src), rows, cols, reinterpret_cast<__bf16*>(dst));
  HTH_HIP(hipGetLastError());
  return HTH_OK;
}

extern "C" hth_status hth_to_bf16(const float* s, uint16_t* d, size_t n, void* stream) {
  if (!s || !d) return fail(HTH_E_INVALID, "NULL argument");
  const unsigned g_ = (unsigned)std::min<size_t>((n + 255) / 256, 8192);
  hipLaunchKernelGGL(k_to_bf16, dim3(std::max(1u, g_)), dim3(256), 0, static_cast<hipStream_t>(stream), s,
                     reinterpret_cast<__bf16*>(d), n);
  HTH_HIP(hipGetLastError());
  return HTH_OK;
}

// Indices of the k largest scores (NaN last): five launches, each finding what
// it needs from the histograms on the device, so nothing is read back.
extern "C" hth_status hth_topk(const float* d_scores, uint32_t n, uint32_t k, uint32_t* d_idx,
                               uint32_t* d_work, void* stream) {
  if (!d_scores || !d_idx || !d_work) return fail(HTH_E_INVALID, "NULL argument");
  if (k > n) return fail(HTH_E_RANGE, "k > n");
  if (k == 0) return HTH_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const unsigned grid = std::min<unsigned>((n - 1) / 256 + 1, 512);
  hipLaunchKernelGGL(k_topk_clear, dim3((kTopWords + 255) / 256), dim3(256), 0, st, d_work);
  for (int d = 0; d < 3; ++d)
    hipLaunchKernelGGL(k_topk_hist, dim3(grid), dim3(256), 0, st, d_scores, n, k, d, d_work);
  hipLaunchKernelGGL(k_topk_collect, dim3(grid), dim3(256), 0, st, d_scores, n, k, d_work, d_idx);
  HTH_HIP(hipGetLastError());
  return HTH_OK;
}

extern "C" hth_status hth_score_rows(const uint16_t* d_feat, const uint32_t* d_hyp_node_offsets, uint32_t row0,
                                     uint32_t n_rows, const uint16_t* d_parent_feat, const uint32_t* d_parent_offsets,
                                     const uint32_t* d_parent_index, uint32_t parent_context, const uint16_t* w1,
                                     const float* b1, const uint16_t* w2t, const float* b2, const float* w3,
                                     const float* b3, float n_pos, float n_neg, const uint32_t* base, int kind,
                                     float* score, void* scratch, size_t scratch_bytes, void* stream) {
  if (!d_feat || !d_hyp_node_offsets || !w1 || !b1 || !w2t || !b2 || !w3 || !b3 || !score || !scratch)
    return fail(HTH_E_INVALID, "NULL argument");
  if (scratch_bytes < HTH_SCORE_SCRATCH_BYTES) return fail(HTH_E_NOMEM, "scratch smaller than HTH_SCORE_SCRATCH_BYTES");
  if (!d_parent_index != !d_parent_feat || !d_parent_index != !d_parent_offsets)
    return fail(HTH_E_INVALID, "parent features, offsets and index go together");
  if ((reinterpret_cast<uintptr_t>(w1) | reinterpret_cast<uintptr_t>(w2t) | reinterpret_cast<uintptr_t>(scratch)) % 16)
    return fail(HTH_E_INVALID, "w1, w2t and scratch must be 16-byte aligned");
  if (parent_context > 1) return fail(HTH_E_RANGE, "parent_context must be 0 or 1");
  if (kind != 0 && kind != 1) return fail(HTH_E_RANGE, "kind must be 0 or 1");
  if (kind == 1 && !base) return fail(HTH_E_INVALID, "kind 1 needs the base coverage");
  if (!n_rows) return HTH_OK;
  ScoreArgs S{d_feat, d_parent_feat, d_hyp_node_offsets, d_parent_offsets, d_parent_index, row0, n_rows,
              parent_context, reinterpret_cast<const __bf16*>(w1), static_cast<const bf16x8*>(scratch), b1, b2, w3, b3,
              n_pos, n_neg, base, kind, score};
  const size_t lds = sizeof(__bf16) * kScoreRows * kScoreLd;
  HTH_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_score_rows), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL(k_score_pack, dim3(8 * (kScoreH1 / 16) * 64 / 256), dim3(256), 0, static_cast<hipStream_t>(stream),
                     reinterpret_cast<const __bf16*>(w2t), static_cast<bf16x8*>(scratch));
  hipLaunchKernelGGL(k_score_rows, dim3((n_rows - 1) / kScoreRows + 1), dim3(64 * kScoreWaves), lds, static_cast<hipStream_t>(stream), S);
  HTH_HIP(hipGetLastError());
  return HTH_OK;
}
