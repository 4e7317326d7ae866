// small.h -- planning, store update and pair list of small batches (small.hip).
#pragma once

#include "internal.h"
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
// vertex 4 to 8 bytes.  A batch alone in its call is taken up to fewer rows, since sorting and
// scanning by one workgroup outgrows the launches that it saves: deleting and inserting n rows
// of two members among 1M hyperedges takes 0.34 ms so and 0.55 kernel by kernel at n = 100,
// 0.63 and 0.66 at 1,025, 0.77 and 0.72 at 1,500, 0.85 and 0.71 at 2,048 (among 4M: 0.71 both
// at 1,024, 0.98 and 0.81 at 2,048).  A round's graphs share the launch, so there the limit is
// the LDS's.  The update's list words, which it only passes through, are held to 32 passes of
// its threads.
constexpr uint64_t kSmallRows = 2048;    // deletions, and inserts
constexpr uint64_t kSmallRowsAlone = 1280;  // ... of the only batch of a call
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

// The jobs of a few graphs travel in the kernel's argument block; those of more are read
// by their workgroups from pinned memory, where every graph has a place for its own, so
// that all run at once (48 graphs: 8 launches of plans, 1.36 ms, and 7 of updates, 0.58 ms,
// are one each of 0.24 and 0.14 ms).
constexpr uint32_t kSmallByValue = 5, kSmallJobs = 256, kSmallIvJobs = 16;
struct SmallHost {  // pinned, one per graph
    BatchSummary sum;
    SmallPlan plan;      // written before the plan is launched, read until its wait
    SmallCommit commit;  // read until the batch's update has run, which the next plan waits for
    uint64_t counts[HGT_COUNT_WORDS];  // written with the device's at the end of every batch
};
void small_plan(SmallHost* const* jobs, uint32_t n, hipStream_t s);
void small_commit(SmallHost* const* jobs, uint32_t n, hipStream_t s);
void small_iv(const SmallIv* jobs, uint32_t n, hipStream_t s);  // n <= kSmallIvJobs
