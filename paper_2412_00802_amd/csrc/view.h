// The example view: the part of an evaluation that only coverage needs, done
// over the examples alone.
//
// A hypothesis's result is its coverage of the positive and negative examples
// (Algorithm 15).  Only instance sets that fillers read are needed for every
// individual; a node above every role restriction matters at the examples
// only, which are a few percent of the individuals.  The view numbers the
// examples (the set bits of pos | neg, in order) and holds, over them:
//   - bit rows (64 examples a word): the examples' positive and negative bits,
//     thresholds, the restrictions that no filler reads, and copies of the
//     full rows that root programs read (atoms, set rows, shared restrictions);
//   - for each role direction used there, the examples' rows of its CSR.
// The shared passes and region programs run on it unchanged: DevKB::view
// points at {examples, words}, counted on the device, so nothing here depends
// on what the host believes about the example rows (they are read at each
// launch).  The host's count of the examples at load time (ex_hint) decides
// whether a plan uses the view; its grids have blocks for that many examples
// and for the whole chip, and every area has room for all individuals.
// Included by exec.hip only.
#pragma once

namespace hth {
namespace {

constexpr uint32_t kExTile = 2048;     // words per block of the example list
constexpr uint32_t kVDirTile = 1024;   // examples per tile of a direction's copy
constexpr uint32_t kVRows = 16;        // row copies per block

// One role direction of the view: its CSR copy starts at `base` in the view's
// target area; compact: its targets are object ranks.
struct ViewDir {
  uint32_t rd, compact;
  uint64_t base;
};
// Exclusive scan of p[0 .. n) in place by one block of 1024; -> the total.
__device__ uint32_t block_scan_row(uint32_t* __restrict__ p, uint32_t n) {
  __shared__ uint32_t s_w[16], s_carry;
  const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (threadIdx.x == 0) s_carry = 0;
  __syncthreads();
  for (uint32_t c = 0; c < n; c += 1024) {
    const uint32_t i = c + threadIdx.x, v = i < n ? p[i] : 0;
    uint32_t inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t u = (uint32_t)__shfl_up((int)inc, d, 64);
      if (lane >= (uint32_t)d) inc += u;
    }
    if (lane == 63) s_w[wv] = inc;
    __syncthreads();
    uint32_t before = s_carry;
    for (uint32_t w = 0; w < wv; ++w) before += s_w[w];
    if (i < n) p[i] = before + inc - v;
    __syncthreads();
    if (threadIdx.x == 1023) s_carry = before + inc;
    __syncthreads();
  }
  return s_carry;
}

__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {   // inclusive
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t u = (uint32_t)__shfl_up((int)v, d, 64);
    if (lane >= d) v += u;
  }
  return v;
}

// The example list in three steps: words' popcounts by tile, their scan (and
// the view's sizes), the list.  hdr: {examples, words of 64 examples}.  Bound
// by launch latency (a few microseconds each over 4M individuals).  Bits past
// the last individual are no examples: the rows are the caller's, read at each
// launch, and what they hold there must not become an index.
__device__ __forceinline__ uint32_t ex_words(const DevKB& kb, uint64_t (&v)[8]) {
  const uint32_t w0 = blockIdx.x * kExTile + threadIdx.x * 8;
  uint32_t n = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint64_t valid = w0 + i + 1 < kb.W ? ~0ull : w0 + i < kb.W ? kb.tail : 0ull;
    v[i] = valid ? (kb.pos[w0 + i] | kb.neg[w0 + i]) & valid : 0ull;
    n += (uint32_t)__popcll(v[i]);
  }
  return n;
}
__global__ void __launch_bounds__(256) k_ex_sum(DevKB kb, uint32_t* __restrict__ tsum) {
  __shared__ uint32_t s[4];
  uint64_t v[8];
  const uint32_t n = wave_sum(ex_words(kb, v));
  if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = n;
  __syncthreads();
  if (threadIdx.x == 0) tsum[blockIdx.x] = s[0] + s[1] + s[2] + s[3];
}
__global__ void __launch_bounds__(1024) k_ex_scan(uint32_t* __restrict__ tsum, uint32_t tiles, uint32_t* __restrict__ hdr) {
  const uint32_t m = block_scan_row(tsum, tiles);
  if (threadIdx.x == 0) {
    hdr[0] = m;
    hdr[1] = (m + 63) / 64;
  }
}
// list[i] = example i; words[w] = w (the view's passes visit every word)
__global__ void __launch_bounds__(256)
k_ex_list(DevKB kb, const uint32_t* __restrict__ tsum, uint32_t* __restrict__ list, uint32_t* __restrict__ words) {
  __shared__ uint32_t s[4];
  uint64_t v[8];
  const uint32_t n = ex_words(kb, v), inc = wave_scan(n), wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 63) s[wv] = inc;
  __syncthreads();
  uint32_t at = tsum[blockIdx.x] + inc - n;
  for (uint32_t w = 0; w < wv; ++w) at += s[w];
  const uint32_t w0 = blockIdx.x * kExTile + threadIdx.x * 8;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    if (w0 + i >= kb.W) break;
    words[w0 + i] = w0 + i;
    for (uint64_t m = v[i]; m; m &= m - 1) list[at++] = (w0 + i) * 64 + (uint32_t)__builtin_ctzll(m);
  }
}

// The examples' rows of each direction: degrees by tile, their scan, then the
// offsets and the targets (a wave copies 64 rows at a time as one run: each
// lane finds the row of its output position among the 64 in LDS).  Bound by
// the lines that scattered rows touch: 96 directions at 250,000 examples of 4M
// individuals 0.6 ms, where the passes over every individual's rows that the
// copies replace take 14.
__device__ __forceinline__ const uint32_t* dir_offsets(const DevKB& kb, uint32_t rd) {
  return (rd & 1 ? kb.inv_off : kb.fwd_off) + (size_t)(rd >> 1) * (kb.N + 1);
}
__global__ void __launch_bounds__(256)
k_vdir_sum(DevKB kb, const ViewDir* __restrict__ dirs, const uint32_t* __restrict__ hdr,
           const uint32_t* __restrict__ list, uint32_t per, uint32_t tcap, uint32_t* __restrict__ tsum) {
  __shared__ uint32_t s[4];
  const uint32_t m = hdr[0], tiles = (m + kVDirTile - 1) / kVDirTile;
  const ViewBlock B = view_block(blockIdx.x, gridDim.x / per, per, tiles);
  const uint32_t* off = dir_offsets(kb, dirs[B.item].rd);
  for (uint32_t t = B.b; t < tiles; t += per) {
    uint32_t n = 0;
#pragma unroll
    for (uint32_t i = 0; i < kVDirTile / 256; ++i) {
      const uint32_t e = t * kVDirTile + i * 256 + threadIdx.x;
      if (e < m) {
        const uint32_t x = list[e];
        n += off[x + 1] - off[x];
      }
    }
    n = wave_sum(n);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) tsum[(size_t)B.item * tcap + t] = s[0] + s[1] + s[2] + s[3];
  }
}
__global__ void __launch_bounds__(1024)
k_vdir_scan(const uint32_t* __restrict__ hdr, uint32_t tcap, uint32_t N, uint32_t* __restrict__ tsum,
            uint32_t* __restrict__ voff) {
  const uint32_t m = hdr[0];
  const uint32_t total = block_scan_row(tsum + (size_t)blockIdx.x * tcap, (m + kVDirTile - 1) / kVDirTile);
  if (threadIdx.x == 0) voff[(size_t)blockIdx.x * (N + 1) + m] = total;
}
__global__ void __launch_bounds__(256)
k_vdir_copy(DevKB kb, const ViewDir* __restrict__ dirs, const uint32_t* __restrict__ hdr,
            const uint32_t* __restrict__ list, uint32_t per, uint32_t tcap, const uint32_t* __restrict__ tsum,
            uint32_t* __restrict__ voff, int32_t* __restrict__ vtg) {
  constexpr uint32_t kSub = kVDirTile / 256;     // rounds of 64 rows a wave
  __shared__ uint32_t s[4], s_pre[4][64], s_lo[4][64];
  const uint32_t m = hdr[0], tiles = (m + kVDirTile - 1) / kVDirTile;
  const ViewBlock B = view_block(blockIdx.x, gridDim.x / per, per, tiles);
  const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const ViewDir D = dirs[B.item];
  const uint32_t* off = dir_offsets(kb, D.rd);
  const int32_t* tg = (D.compact ? (D.rd & 1 ? kb.ctg_inv : kb.ctg_fwd) : (D.rd & 1 ? kb.inv_tg : kb.fwd_tg)) +
                      kb.role_base[D.rd >> 1];
  uint32_t* vo = voff + (size_t)B.item * (kb.N + 1);
  int32_t* out = vtg + D.base;
  for (uint32_t t = B.b; t < tiles; t += per) {
    uint32_t lo[kSub], inc[kSub], tot[kSub], sum = 0;
#pragma unroll
    for (uint32_t i = 0; i < kSub; ++i) {
      const uint32_t e = t * kVDirTile + wv * 64 * kSub + i * 64 + lane;
      lo[i] = inc[i] = 0;
      if (e < m) {
        const uint32_t x = list[e];
        lo[i] = off[x];
        inc[i] = off[x + 1] - lo[i];
      }
    }
#pragma unroll
    for (uint32_t i = 0; i < kSub; ++i) {
      inc[i] = wave_scan(inc[i]);
      tot[i] = (uint32_t)__builtin_amdgcn_readlane((int)inc[i], 63);
      sum += tot[i];
    }
    __syncthreads();
    if (lane == 0) s[wv] = sum;
    __syncthreads();
    uint32_t at = tsum[(size_t)B.item * tcap + t];
    for (uint32_t w = 0; w < wv; ++w) at += s[w];
#pragma unroll
    for (uint32_t i = 0; i < kSub; ++i) {
      const uint32_t e = t * kVDirTile + wv * 64 * kSub + i * 64 + lane;
      const uint32_t up = (uint32_t)__shfl_up((int)inc[i], 1, 64), pre = lane ? up : 0u;
      if (e < m) vo[e] = at + pre;
      s_pre[wv][lane] = pre;
      s_lo[wv][lane] = lo[i];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 4
      for (uint32_t p = lane; p < tot[i]; p += 64) {
        uint32_t r = 0;                    // the last row that starts at or before p
#pragma unroll
        for (uint32_t d = 32; d; d >>= 1)
          if (s_pre[wv][r + d] <= p) r += d;
        out[at + p] = tg[s_lo[wv][r] + p - s_pre[wv][r]];
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      at += tot[i];
    }
  }
}

// Row copies: a wave takes 8 view words, a lane one example of each, and
// gathers the examples' bits of one full row after another; a ballot makes a
// word.  64 consecutive examples lie in a few lines of a row, so the loads
// read each row about once: bound by HBM and by the bit tests (0.42 ms for the
// rows that 65,536 root programs over 4M individuals read).
__global__ void __launch_bounds__(256)
k_view_rows(DevKB kb, uint64_t* __restrict__ vslots, const uint32_t* __restrict__ hdr,
            const uint32_t* __restrict__ list, const ViewCopy* __restrict__ copies, uint32_t n_copies,
            uint32_t slot0) {
  const uint32_t m = hdr[0], vw = hdr[1];
  const uint32_t per = gridDim.x;
  const ViewBlock B = view_block(blockIdx.y * per + blockIdx.x, gridDim.y, per, (vw + 31) / 32);
  const uint32_t lane = threadIdx.x & 63, c0 = B.item * kVRows, c1 = min(c0 + kVRows, n_copies);
  for (uint32_t b = B.b * 4 + (threadIdx.x >> 6); b * 8 < vw; b += per * 4) {
    uint32_t x[8];
    bool in[8];
#pragma unroll
    for (uint32_t j = 0; j < 8; ++j) {
      const uint32_t e = (b * 8 + j) * 64 + lane;
      in[j] = e < m;
      x[j] = list[in[j] ? e : 0u];
    }
    // (one copy's loads in flight at a time: with two, 16 of a lane's, 424 us for
    // 416, and 442 for 433 over 32M individuals)
    for (uint32_t c = c0; c < c1; ++c) {
      const ViewCopy C = copies[c];
      const uint64_t* row = C.src == kPosRow ? kb.pos : C.src == kNegRow ? kb.neg
                            : row_ptr(kb, C.src & kSlotRow ? slot0 + (C.src & ~kSlotRow) : C.src);
      const uint32_t* r32 = reinterpret_cast<const uint32_t*>(row);
      uint32_t v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = r32[x[j] >> 5];
      uint64_t mine = 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint64_t w = __ballot(in[j] && ((v[j] >> (x[j] & 31)) & 1u));
        if (lane == (uint32_t)j) mine = w;
      }
      if (lane < 8 && b * 8 + lane < vw) vslots[(size_t)C.dst * kb.S + b * 8 + lane] = mine;
    }
  }
}

// Whether a plan uses the view: the examples are few, and the individuals so
// many that its extra launches (about ten) are worth it.  Microseconds with
// the view / without, 6 % examples, 8 roles of 8 assertions a subject, 256
// hypotheses planned on the host: 16,000 individuals 346 / 283, 33,000 387 /
// 387, 65,536 441 / 474, 400,000 1,226 / 1,333; 2,048 planned on the device:
// 833 / 809, 926 / 980, 1,076 / 1,299, 3,023 / 3,787.  By the share of examples,
// 6 %, 25 % and 50 % with the view / without: 256 on the host over 400,000
// 832, 932, 1,106 / 1,069, over 1M 2,084, 2,472, 2,977 / 3,457; 2,048 on the
// device over 65,536 677, 702, 784 / 785, over 1M 6,677, 8,310, 10,481 / 12,985.
// A quarter is where the least of them (256 on the host, 400,000) still gains.
inline bool view_wanted(const hth_kb_s& kb) {
  return kb.N >= kb.view_min && kb.ex_hint && (uint64_t)kb.ex_hint * 4 <= kb.N;
}

// The view of one plan: its directions, shared passes and areas (offsets into
// the workspace, from `at`).
struct ViewPlan {
  bool on = false;
  std::vector<ViewDir> dirs;            // by view direction
  std::vector<GroupTask> groups;        // as built from: real role and direction
  std::vector<GroupTask> passes;        // as counted over: role = view direction, inv = 0
  std::vector<GroupChunk> chunks;
  uint32_t n_rows = kViewFixed, n_copies = 2, n_thg = 0;
  uint64_t targets = 0;
  size_t bytes = 0;                     // of its areas
  size_t o_hdr = 0, o_list = 0, o_words = 0, o_tsum = 0, o_dsum = 0, o_off = 0, o_tg = 0, o_base = 0, o_slot = 0;

  // the `count` role nodes of direction rd, each added once, as shared passes of
  // at most gk, their members from `first` on
  void add_passes(const hth_kb_s& kb, uint32_t rd, uint64_t count, uint32_t gk, uint32_t first, bool short_rows) {
    const uint32_t v = (uint32_t)dirs.size();
    dirs.push_back(ViewDir{rd, kb.tune.t_compact && 2ull * kb.n_obj[rd] <= kb.N ? 1u : 0u, targets});
    targets += kb.role_base[rd / 2 + 1] - kb.role_base[rd / 2];
    for (uint64_t i0 = 0; i0 < count; i0 += gk) {
      GroupTask g{};
      g.role = rd / 2;
      g.inv = rd & 1;
      g.k = (uint32_t)std::min<uint64_t>(gk, count - i0);
      g.first = (uint32_t)(first + i0);
      g.n_words = kb.n_words[rd];
      g.n_obj_words = kb.n_words[rd ^ 1u];
      g.compact = dirs[v].compact;
      g.short_rows = short_rows;
      groups.push_back(g);
      g.role = v;
      g.inv = 0;
      passes.push_back(g);
    }
  }
  // What it adds (its areas have room for every individual, since the examples
  // may be any by the time of a launch; less the rows that stand for full ones)
  // is out of proportion: over a gigabyte, and over 128 times the rest of the
  // workspace (need holds both).  Below that the caller chooses: a workspace
  // without the room is served without the view.  Half a round over 32M
  // individuals, 71 directions: 11.4 GB beside 0.4, rounds of 25.1, 24.3 and
  // 25.9 ms with it, 28.2, 27.3 and 30.9 without; 4,096 hypotheses over 1M
  // individuals, 266M assertions: 1.9 GB beside 2.6.
  bool too_large(const hth_kb_s& kb, size_t need) const {
    const size_t added = bytes - (size_t)(n_rows - n_copies) * kb.S * 8;
    return on && added > (1ull << 30) && added / 128 > need - added;
  }
  uint32_t tiles(const hth_kb_s& kb) const { return (kb.W + kExTile - 1) / kExTile; }
  uint32_t dir_tiles(const hth_kb_s& kb) const { return (kb.N + kVDirTile - 1) / kVDirTile; }
  template <class Area>
  void layout(const hth_kb_s& kb, Area&& area) {
    if (!on) return;
    o_hdr = area(256);
    o_list = area((size_t)kb.N * 4);
    o_words = area((size_t)kb.W * 4);
    o_tsum = area((size_t)tiles(kb) * 4);
    o_dsum = area(dirs.size() * dir_tiles(kb) * 4);
    o_off = area(dirs.size() * ((size_t)kb.N + 1) * 4);
    o_tg = area(targets * 4 + 4);
    o_slot = area((size_t)n_rows * kb.S * 8);
  }
};

// The DevKB that the view's passes and regions see.  bases: [dirs] device
// copy of the directions' first targets.
inline DevKB view_kb(const DevKB& d, const ViewPlan& V, char* ws, const uint64_t* bases) {
  DevKB x = d;
  x.view = reinterpret_cast<const uint32_t*>(ws + V.o_hdr);
  x.slots = reinterpret_cast<uint64_t*>(ws + V.o_slot);
  x.n_concepts = x.n_fixed = 0;
  x.fwd_off = reinterpret_cast<const uint32_t*>(ws + V.o_off);
  x.fwd_tg = x.ctg_fwd = reinterpret_cast<const int32_t*>(ws + V.o_tg);
  x.role_base = bases;
  x.words = reinterpret_cast<const uint32_t*>(ws + V.o_words);
  x.pos = x.slots;
  x.neg = x.slots + d.S;
  return x;
}

// Everything of the view before its thresholds, passes and regions.
hth_status launch_view_rows(Launcher& L, const DevKB& d, const ViewPlan& V, char* ws, const ViewDir* dirs,
                            const ViewCopy* copies, uint32_t slot0) {
  const hth_kb_s& kb = L.kb;
  uint32_t* hdr = reinterpret_cast<uint32_t*>(ws + V.o_hdr);
  uint32_t* list = reinterpret_cast<uint32_t*>(ws + V.o_list);
  uint32_t* words = reinterpret_cast<uint32_t*>(ws + V.o_words);
  uint32_t* tsum = reinterpret_cast<uint32_t*>(ws + V.o_tsum);
  uint32_t* dsum = reinterpret_cast<uint32_t*>(ws + V.o_dsum);
  uint32_t* voff = reinterpret_cast<uint32_t*>(ws + V.o_off);
  int32_t* vtg = reinterpret_cast<int32_t*>(ws + V.o_tg);
  uint64_t* slots = reinterpret_cast<uint64_t*>(ws + V.o_slot);
  const uint32_t tiles = V.tiles(kb), tcap = V.dir_tiles(kb), nd = (uint32_t)V.dirs.size();
  hth_status s = L.run(HTH_K_REGION, 2.0 * kb.W * 8, [&] {
    hipLaunchKernelGGL(k_ex_sum, dim3(tiles), dim3(256), 0, L.st, d, tsum);
    hipLaunchKernelGGL(k_ex_scan, dim3(1), dim3(1024), 0, L.st, tsum, tiles, hdr);
    hipLaunchKernelGGL(k_ex_list, dim3(tiles), dim3(256), 0, L.st, d, tsum, list, words);
  });
  if (s) return s;
  if (nd) {
    // blocks for the examples expected, and for the whole chip; more examples are taken in turns
    const uint32_t want = std::max(kb.ex_hint / kVDirTile + 1, std::min(tcap, view_fill(kb, nd)));
    const uint32_t gx = std::max(1u, std::min(want, 65536u / nd + 1));
    s = L.run(HTH_K_GROUP, 0.0, [&] {
      hipLaunchKernelGGL(k_vdir_sum, dim3(gx * nd), dim3(256), 0, L.st, d, dirs, hdr, list, gx, tcap, dsum);
      hipLaunchKernelGGL(k_vdir_scan, dim3(nd), dim3(1024), 0, L.st, hdr, tcap, kb.N, dsum, voff);
      hipLaunchKernelGGL(k_vdir_copy, dim3(gx * nd), dim3(256), 0, L.st, d, dirs, hdr, list, gx, tcap, dsum, voff, vtg);
    });
    if (s) return s;
  }
  for (uint32_t c = 0; c < V.n_copies; c += 65535 * kVRows) {
    const uint32_t n = std::min(V.n_copies - c, 65535 * kVRows), gy = (n + kVRows - 1) / kVRows;
    const uint32_t fill = std::min((kb.W + 31) / 32, view_fill(kb, gy));
    const uint32_t gx = std::max(fill, std::min((view_words_hint(kb) + 31) / 32, 16384u));
    s = L.run(HTH_K_REGION, (double)n * kb.W * 8, [&] {
      hipLaunchKernelGGL(k_view_rows, dim3(gx, gy), dim3(256), 0, L.st, d, slots, hdr, list,
                         copies + c, n, slot0);
    });
    if (s) return s;
  }
  return HTH_OK;
}

// The whole view, after every full row of the plan is complete: its lists, row
// copies, thresholds and shared passes.  *d becomes the view's DevKB for the
// root regions.
hth_status launch_view(Launcher& L, const DevKB& full, const ViewPlan& V, char* ws, const ViewDir* dirs,
                       const uint64_t* bases, const ViewCopy* copies, uint32_t slot0, const ThrGroup* thg,
                       const ThrTask* thr, const GroupTask* groups, const GroupTask* passes,
                       const GroupMember* members, const uint32_t* xslots, void* tarea, DevKB* d) {
  const hth_kb_s& kb = L.kb;
  const DevKB f = full;
  hth_status s = launch_view_rows(L, f, V, ws, dirs, copies, slot0);
  if (s) return s;
  const DevKB x = view_kb(f, V, ws, bases);
  if (V.n_thg) {
    const uint32_t* list = reinterpret_cast<const uint32_t*>(ws + V.o_list);
    const uint32_t bpt = std::max((view_words_hint(kb) + 31) / 32, std::min((kb.W + 31) / 32, view_fill(kb, V.n_thg)));
    s = split_launch(L, HTH_K_THRESHOLD, 4.0 * kb.ex_hint * V.n_thg, V.n_thg, bpt, 256,
                     [&](uint32_t i0, uint32_t, uint32_t blocks) {
                       hipLaunchKernelGGL(k_threshold<true>, dim3(blocks), dim3(256), 0, L.st, x, thg + i0, thr, bpt, list);
                     });
    if (s) return s;
  }
  if (!V.groups.empty()) {
    L.csr_seen.clear();
    s = launch_groups(L, f, groups, members, V.groups, V.chunks, xslots, tarea, nullptr, &x, passes);
    if (s) return s;
  }
  *d = x;
  return HTH_OK;
}

}  // namespace
}  // namespace hth
