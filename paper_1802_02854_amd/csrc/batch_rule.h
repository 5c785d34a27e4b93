// How the sequences of a Green's-function call share launches: the size, number and
// layout of its batches.  Plain C++, tested on the host.
#pragma once

#include <algorithm>
#include <cstddef>

namespace ftk {

constexpr int kMaxChains = 2;  // batches of Green's sequences in flight, a stream each
constexpr int kMaxBatch = 32;  // sequences per batch: 16 in block layout, 32 as a stack
constexpr int kMaxRows = 32768;  // rows of one launch (grid y, which ends at 65535)

// batches the block layout has kernels for, a wavefront's 512 entries at least; 1 is a
// sequence alone
inline bool block_batch(int B, int n_sites)
{
    return B == 1 || ((B == 2 || B == 4 || B == 8 || B == 16) && ((size_t)B << n_sites) >= 512);
}

struct Batches {
    int B;       // sequences of a batch
    int chains;  // batches in flight
    int stack;   // layout for B > 1: 1 a stack of multi-pass sequences, 0 block, -1 the default
};

// How `rows` sequences run where the batch asked for may be changed (run_green): batches
// of B in chains, each on its own stream.  A second chain fills the first one's launch
// gaps and overlaps its loads with the other's bonds (all workgroups of a small launch are
// in the same phase), and larger stacks share launches, so up to 64 sequences go in
// flight, those beyond the batch asked for with up to 256 MiB of vectors (spare, the
// last-level cache's size), in even batches.  us per sequence and step as asked, in chains of
// what was asked, so: 16 sites, 6 in batches of 1: 12 / 7.6 / 3.9; 24 of 8: 2.8 / 2.6 /
// 2.4; 72 of 32: 2.1 / 2.2 / 1.85; 110 of 32: 1.9 / 1.8 / 1.6; 18 sites, 4 of 1: 19 / 13.3
// / 10.6; 24 of 16: 6.4 / 6.6 / 6.3; 20 sites, 4 of 1: 41.6 / 38.9 / 35.4; 22 sites, 4 of
// 1: 137 / 118 as asked and so.  Three or four chains are no faster (16 sites, 110 in flight
// in four: 1.77).
// The batch asked for runs alone where its vectors (per bytes a sequence) are past spare
// (20 sites, two chains of 16: 35.4 us per sequence and step against 31.0; 24 sites, of
// 1: 557 against 510) and where the block layout was picked for it.  A layout recorded for
// single sequences says nothing about larger batches: those are stacks, the only
// layout that has a kernel for every size up to kMaxBatch.
inline Batches spread_rows(size_t rows, Batches asked, size_t per, size_t spare, bool streams)
{
    if (per * asked.B > spare || (asked.stack == 0 && asked.B > 1)) return asked;
    const size_t limit = streams ? kMaxChains : 1;
    const size_t most = std::max<size_t>(asked.B, std::min(limit * kMaxBatch, asked.B + spare / per));
    const size_t rounds = (rows + most - 1) / most, now = (rows + rounds - 1) / rounds;
    Batches r = asked;
    r.chains = (int)std::min(limit, now);
    r.B = (int)((now + r.chains - 1) / r.chains);
    if (r.B > 1) r.stack = 1;
    return r;
}

// The batch whose recorded pass grid and cache hints a run takes: the one asked for, whose
// stack the batches that run are even parts or multiples of; a record for single
// sequences holds for those alone (0: none).
inline int tuned_batch(const Batches &asked, const Batches &run) { return asked.B > 1 || run.B == 1 ? asked.B : 0; }

// Sequences of one resident launch (one workgroup each; their start vectors and shift
// updates are rows of a grid): what fits in spare bytes at per bytes a sequence.
inline size_t resident_rows(size_t rows, size_t per, size_t spare)
{
    return std::min({rows, std::max<size_t>(1, spare / per), (size_t)kMaxRows});
}

}  // namespace ftk
