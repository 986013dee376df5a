// Draw-ordered steps of the batched and the served paths: the samples of many
// graphs and requests, run graph by graph in the order of their draws.
#pragma once

#include <vector>

#include "backoff.hpp"
#include "batch.hpp"

namespace pm {

// The samples first, first + 1, ..., first + count - 1 of one sampler of one
// graph (weight R > 0), counted into tally slot `slot`.
struct StepItem {
    uint32_t graph;
    uint32_t tag;  // 0 3-path sampler, 1 centered sampler
    uint32_t slot;
    uint64_t first, count, seed, R;
};

// A step is run in parts of at most kSortedChunk samples, each a sequence of
// chunks laid end to end: positions [start, next chunk's start) are the
// samples first, first + 1, ... of one item.  The chunks of one graph and
// sampler follow each other and form a group.  Both tables end with a
// sentinel that holds the end positions.
struct StepChunk {
    uint64_t first, seed;
    uint32_t start;
    uint32_t slot;
    uint32_t group;
    uint32_t pad;
};

struct StepGroup {
    double scale;     // (samples of the group) / (total weight of its sampler)
    uint32_t begin;   // first position
    uint32_t chunk0;  // first chunk
    uint32_t graph;
    uint32_t tag;
};

constexpr uint32_t kStepChunks = 512;  // chunks of a part, at most (their counts live in LDS: 16 KiB)
constexpr unsigned kStepBlocks = 2048;  // blocks of a launch, at most (more would not be resident)
// Blocks per compute unit where the caller sets none: 64 graphs of up to 2e6
// edges at 2e5 + 2e5 samples each took 2.23, 2.10, 1.98 and 1.97 ms a run at
// 4, 5, 6 and 7 (in id order more blocks hold more graphs in flight and are
// slower: 13.8 ms at 4, 16.3 at 8, over the requests of step.hip).
constexpr int kStepBlocksPerCu = 6;

// Runs draw-ordered steps on one stream.  It keeps the tables' memory; a step's
// sort buffers (at most those of a part of kSortedChunk samples, 0.3 GB) are
// the library's cached memory and go back with the step, so that any number of
// batches and servers share them.  One step at a time: the caller has waited
// for the step before.
class StepRunner {
public:
    // Enqueue the items' samples: tallies[0, slots * 16) receive their counts
    // (slot * 16 + tag * 8 + c; zero elsewhere).  No two items share a slot
    // and a sampler.  *done is false, and nothing is enqueued, where the step
    // is left to the id order: fewer than draw_order_min() samples or more
    // than 2^40, draw order off, too many small items, or no memory (after
    // which up to Backoff::kMost steps are left out before the next try).
    pm_status run(const BatchGraph *graphs, std::vector<StepItem> &items, uint64_t *tallies, int64_t slots,
                  unsigned blocks, hipStream_t s, bool *done);
    void free(hipStream_t s);

private:
    bool grow(size_t table_bytes, hipStream_t s);

    char *d_tables = nullptr, *h_tables = nullptr;  // the parts' tables; h_ pinned
    size_t table_cap = 0;
    Backoff memory;  // after steps without memory for their buffers
};

}  // namespace pm
