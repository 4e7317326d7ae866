// small.h -- planning, store update and pair list of small batches (small.hip).
#pragma once

#include "store.h"

// A batch that one workgroup plans (of one graph).
struct SmallPlan {
    StoreDev g;
    BatchIn b;
    PlanScratch w;
    uint64_t* acc;       // phase accumulators to clear
    uint32_t n_acc;
    uint32_t pad0;
    BatchSummary* out;   // pinned host memory: the summary for the host (pad0 = 1: too large after
                         // all, nothing planned)
};

// The limits are what fits the workgroup's LDS: keys of 8 bytes, and per row and per touched
// vertex 4 to 8 bytes.  At them a workgroup takes about as long as the kernels it replaces
// (100 changes of cardinality 2 to 8: 4.35 -> 3.94 ms for the whole batch); the update's
// list words, which it only passes through, are held to 32 passes of its threads.
constexpr uint64_t kSmallRows = 2048;    // deletions, and inserts
constexpr uint32_t kSmallPairs = 8192;   // (vertex, hyperedge) pairs, or touched vertex pairs
constexpr uint64_t kSmallIds = 1ull << 22;  // 16 rounds over the free-ID bitmap
constexpr uint64_t kSmallStage = 32768;  // old list words of the touched vertices

struct SmallCommit {
    StoreDev g;
    BatchIn b;
    PlanScratch w;
    uint64_t n_touched, h_bump, v_bump, next_seq;
    uint32_t* out_ids;   // may be NULL
};

// The touched vertex pairs of a batch with at most kSmallPairs pairs inside its rows.
struct SmallIv {
    const uint32_t* del;
    uint64_t n_del, n_ins;
    const uint64_t* h_off;
    const uint32_t* h_len;
    const uint32_t* h2v;
    const uint32_t* canon;
    const uint64_t* ins_rel;
    const uint32_t* v_len;
    const DevScalars* sc;
    uint64_t* t1;        // sums of C(d, 3): deleted rows, inserted rows
    uint64_t* own;       // owner << 32 | other, sorted
    uint64_t* n_uniq;
    uint64_t* tab;
    uint64_t tab_slots;
    uint64_t* owner_start;
    uint64_t* n_owners;
};

// Arguments travel in the kernel's argument block, several jobs a launch.
constexpr int kSmallPlanJobs = 5, kSmallCommitJobs = 5, kSmallIvJobs = 16;
void small_plan(const SmallPlan* jobs, uint32_t n, hipStream_t s);      // n <= kSmallPlanJobs
void small_commit(const SmallCommit* jobs, uint32_t n, hipStream_t s);  // n <= kSmallCommitJobs
void small_iv(const SmallIv* jobs, uint32_t n, hipStream_t s);          // n <= kSmallIvJobs
