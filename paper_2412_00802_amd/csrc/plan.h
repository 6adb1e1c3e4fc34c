// Host-side evaluation plans: a batch of postfix hypotheses becomes one
// canonical DAG (shared subexpressions evaluated once) scheduled by role
// nesting level.  The paper generates an evaluation plan per hypothesis on the
// CPU before running its DL operations (Section 4, "evaluation plan").
#pragma once

#include <cstdint>
#include <functional>
#include <string>
#include <vector>

#include "kb_handle.h"

namespace hth {

// A cross-batch cache of role-node rows (plan.cpp): canonical subexpressions
// of every batch compiled with it are interned in one persistent DAG, so that
// equal subexpressions of different batches get the same id; a role node whose
// id holds a row is read from that row, and a role node without one may be
// given the least recently used row to write its result into.
struct SubexprCache;
SubexprCache* cache_new(uint32_t n_rows);
void cache_delete(SubexprCache* c);
struct CacheCounters {
  uint64_t hits = 0, misses = 0, admitted = 0, evictions = 0, batches = 0;
  uint32_t entries = 0, rows = 0;
};
CacheCounters cache_counters(const SubexprCache* c);
// Undo the admissions of the last compiled batch (its launch did not happen).
void cache_rollback(SubexprCache* c);

struct PlanOptions {
  SubexprCache* cache = nullptr; // cross-batch cache of role-node rows (the set table)
  bool instances = false;        // write the (single) root's instance set
  uint32_t group_min = 0xFFFFFFFFu;  // (role, dir, level) buckets with at least this many
                                     // role nodes use a shared CSR pass; others run alone
  uint32_t group_k = 64;             // most role nodes per shared pass
  // counts only: restrictions that no filler reads are evaluated at the examples alone
  bool examples = false;
  // ... and, from view_nodes role nodes on, in shared passes over the example view
  bool view = false;
};
// Fewer cost less one by one than the view's launches and copies: what one node
// costs grows with the examples, the view's launches do not (16 + 2^20 / examples
// with the default view_min).  Microseconds one
// by one / in the view / over everyone, batches of hypotheses with one or two
// such nodes each: 6 % of 100,000 individuals, 48 hypotheses 197 / 279 / 253, 96
// 246 / 294 / 276; of 400,000, 32 454 / 479 / 588, 96 732 / 672 / 829; of 1M, 16
// 855 / 881 / 1,255, 64 1,631 / 1,400 / 2,012; 25 % of 1M, 16 1,115 / 1,109 /
// 1,253, 32 1,582 / 1,301 / 1,526.
inline uint64_t view_nodes(const hth_kb_s& kb) { return 16 + 16ull * kb.view_min / std::max(1u, kb.ex_hint); }

// Whether a batch takes its n value-role restrictions that no filler reads at
// the examples: an eighth of the individuals at most, and, below 2^19 of them,
// enough restrictions that one more launch beside the fillers' is worth it.
// Microseconds at the examples / over everyone: 6 % of 65,537, 4 numeric 21.3 /
// 15.3, 8 string 32.4 / 23.4, 40 numeric roots 15.0 / 20.1; of 131,073, 8 string
// 33.3 / 27.4, 8 numeric roots 12.3 / 13.4; of 262,145, 4 roots 12.8 / 13.1, 8 13.0 /
// 19.2; of 524,289, 4 13.2 / 19.0; of 1M, one 12.1 / 12.6; 24 %, 40 roots: of 65,537
// 23.9 / 20.0, of 1M 150.6 / 130.9.
inline bool values_at_examples(const hth_kb_s& kb, uint64_t n) {
  return (uint64_t)kb.ex_hint * 8 <= kb.N && (kb.N >= 1u << 19 || n * kb.N > 3ull << 19);
}

struct PlanLevel {
  std::vector<RegionTask> mat;      // children materialised before this level's role passes
  std::vector<RoleTask> roles;      // single role nodes (k = 1)
  std::vector<RoleTask> ex_roles;   // those needed at the examples only
  std::vector<GroupTask> groups;    // shared passes (k <= 64)
  std::vector<GroupMember> members;
};

struct ViewBucket {
  uint32_t rd, count, first;        // direction 2 role + inv; members [first, first + count)
};

// What the caller had registered when the plan was compiled.
struct Registered {
  const uint32_t* num_roff = nullptr;
  const float* num_val = nullptr;
  const uint32_t* num_heavy_rows = nullptr;
  const HeavyChunk* num_heavy_chunks = nullptr;
  std::vector<uint32_t> num_chunk_first;
  std::vector<uint64_t> num_bounds;        // [P+1] first value of each numeric role
  const uint32_t* str_roff = nullptr;
  const int32_t* str_ids = nullptr;
  const uint32_t* str_heavy_rows = nullptr;
  const HeavyChunk* str_heavy_chunks = nullptr;
  std::vector<uint32_t> str_chunk_first;
  std::vector<uint64_t> str_bounds;
  const int64_t* dict_off = nullptr;
  const uint8_t* dict_chars = nullptr;
  const int64_t* pat_off = nullptr;
  const uint8_t* pat_chars = nullptr;
  uint32_t n_strings = 0;
  const uint64_t* sets = nullptr;   // the set table the plan's HTH_SET rows refer to
  uint32_t n_sets = 0;
};

struct Plan : Registered {
  std::vector<ThrTask> thr;
  std::vector<NumTask> num;         // restrictions on numeric concrete roles
  std::vector<NumTask> ex_num;      // those needed at the examples only
  std::vector<StrTask> str;                // restrictions on string concrete roles
  std::vector<StrTask> ex_str;             // those needed at the examples only
  std::vector<uint32_t> code;
  std::vector<PlanLevel> levels;
  std::vector<RegionTask> roots;
  // the example view (view.h): root programs and these tasks read and write its rows
  bool view = false;
  std::vector<ThrTask> vthr;
  std::vector<ViewCopy> vcopies;    // full rows that root programs read
  std::vector<ViewBucket> vbuckets; // role nodes by direction ...
  std::vector<GroupMember> vmembers;   // ... and these, in the same order
  uint32_t n_vrows = kViewFixed;
  uint32_t n_slots = 0;
  // statistics
  uint32_t n_input_nodes = 0, n_canonical = 0, n_role_nodes = 0;
};

// Compile hypotheses nodes[hyp_off[h] .. hyp_off[h+1]) (local child indices).
// general: also the plan without options examples and view.  later: receives
// what compiles that plan when it is asked for, from what is kept of this call
// (by the knowledge base's schedule then).
hth_status compile_plan(const hth_kb_s& kb, const hth_node* nodes, const uint32_t* hyp_off,
                        uint32_t n_hyps, const uint32_t* children, uint32_t n_children,
                        const PlanOptions& opt, Plan& out, Plan* general = nullptr,
                        std::function<hth_status(Plan&)>* later = nullptr);

}  // namespace hth
