// sca_internal.hpp -- declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sweep_args.hpp"

namespace sca {

// Launches one half-step; returns the launch status.
hipError_t launch_halfstep(const SweepArgs& a, XiMode mode, bool has_q, hipStream_t stream);

// `depth` MCS (2*depth half-steps from MCS a.t on) in one pass, reading src
// and writing dst (both S[2][2][Y][W]); one workgroup per band of `band` rows.
// The deepest pass depends on the kind of acceptance words: mode and, in
// mask mode, the number of draws (0: p and q in {0, 1}, which allows the
// deepest passes).
int max_fused_depth(int32_t W, XiMode mode, int32_t ndraw);
bool fused_supported(int32_t W, int64_t Y, int32_t band, int32_t depth, XiMode mode, int32_t ndraw);
hipError_t launch_mcs_fused(const SweepArgs& a, XiMode mode, bool has_q, const uint64_t* src, uint64_t* dst,
                            int32_t band, int32_t depth, hipStream_t stream);

// Name of the kernel (with its template arguments) that launch_mcs_fused and
// launch_halfstep run for these arguments; written next to their dispatch.
void fused_kernel_name(const SweepArgs& a, XiMode mode, bool has_q, int32_t depth, char* out, size_t n);
void halfstep_kernel_name(int32_t W, XiMode mode, bool has_q, char* out, size_t n);

// A tile of the on-chip sweep (tile.hpp): `rows` rows per workgroup, of which
// the `band` rows behind the first `halo` are written; halo = 0: the tile is
// the whole lattice (rows = band = Y), in place and for any number of MCS.
// Otherwise halo >= 2 n_mcs, src and dst are different states and the bands
// partition Y.  In mode Ahead, for tiles that tile_ahead allows, waves of their
// own form the words of mode Mask.
struct TileShape {
    int32_t rows_per_thread = 0;  // 0: no tile serves the lattice
    int32_t rows = 0, band = 0, halo = 0;
};
hipError_t launch_tile(const SweepArgs& a, XiMode mode, bool has_q, const uint64_t* src, uint64_t* dst,
                       const TileShape& s, int32_t n_mcs, hipStream_t stream);

inline bool tile_ahead(int32_t W, const TileShape& s)
{
    return s.rows_per_thread == 2 && W <= 64 && (s.rows / 2 * W + 63) / 64 * 64 + (s.rows * W + 63) / 64 * 64 <= 1024;
}

void tile_kernel_name(const SweepArgs& a, XiMode mode, bool has_q, int32_t rows_per_thread, char* out, size_t n);

// Flat initial surface into S and h0 = 0.
hipError_t launch_flat_init(uint64_t* S, int64_t Y, int32_t W, int32_t nb, int64_t* h0,
                            hipStream_t stream);

// The flat surface for a list of lattices in one launch (device table of
// items); meant for small states such as an ensemble's realizations.
struct FlatItem {
    uint64_t* S;
    int64_t* h0;
    int64_t plane;   // Y*W
    uint64_t valid;  // used bits of a word
};
FlatItem flat_item(uint64_t* S, int64_t Y, int32_t W, int32_t nb, int64_t* h0);
hipError_t launch_flat_init_many(const FlatItem* items_dev, int32_t n, hipStream_t stream);
constexpr int32_t kFlatFew = 32;  // at most 1 KiB of arguments
hipError_t launch_flat_init_few(const FlatItem* items_host, int32_t n, hipStream_t stream);

// Exact sums of the height field into res[7] (device memory or pinned host
// memory): {S1 lo,hi, S2 lo,hi, S3 lo,hi, *flag or 0}, 128 bits each, with
// S = {sum h, sum h^2, h(0,0)} or, with a snapshot, {sum h_t, sum h_t h_s, sum h_s}.
// partials: kMomentsPartial int64 per block of rows, at most 3 Y in all.
constexpr int kMomentsPartial = 5;
hipError_t launch_moments(const uint64_t* S, const int64_t* h0, const uint64_t* snap, const int64_t* snap_h0,
                          int64_t X, int64_t Y, int32_t W, int32_t nb, int64_t* partials, int64_t* res,
                          const int32_t* flag, hipStream_t stream);

// The sums of n lattices whose moments take one block each (res[7] of each as
// above); items in device memory or pinned host memory.
struct MomentsItem {
    const uint64_t* S;
    const int64_t* h0;
    int64_t* res;
    int32_t Y, W, nb;
};
bool moments_in_one_block(int64_t Y, int32_t W);
hipError_t launch_moments_many(const MomentsItem* items, int32_t n, const int32_t* flag, hipStream_t stream);

// Heights h(0,y) of column 0 into col[Y], h(0,0) into *h0_out.
hipError_t launch_column(const uint64_t* S, const int64_t* h0, int64_t Y, int32_t W, int64_t* col, int64_t* h0_out,
                         hipStream_t stream);

// Heights of rows [y0, y0+ny) into out (needs col[] from launch_column).
hipError_t launch_heights(const uint64_t* S, int64_t X, int64_t Y, int32_t W, const int64_t* col, int64_t y0,
                          int64_t ny, int32_t* out, hipStream_t stream);

// The temporally blocked passes (phase 1 of the persistent kernel) of one
// realization in an epoch, set by the host: depth > 0 runs passes of `depth` MCS on
// bands of one group of W lanes each, `bands` bands per workgroup; a realization
// split into parts > 1 runs on as many workgroups (part m owns bands m*bands ..
// (m+1)*bands-1) that meet at a barrier on counter sync[sync_idx] and keep their
// band save slots in `save` (contiguous for all parts); parts == 1 uses the
// workgroup's own save area.  (On chip: parts workgroups, bands rows per thread.)
struct BlockedGeometry {
    int32_t depth;
    int32_t bands;
    int32_t parts;
    int32_t sync_idx;
    uint64_t* save;
};

// One realization of an ensemble epoch (device table, one entry per slot).
struct BatchDesc {
    uint64_t* S;       // state S[2][2][Y][W] in the arena
    int64_t* h0;       // origin height in the arena
    int64_t plane;     // Y*W
    int32_t W, Y, nb;
    int32_t mode;      // 0 mask, 1 per-site
    uint32_t k0, k1;
    uint32_t dig_p, dig_q;
    int32_t ndraw;
    int32_t has_q;
    uint32_t thr_p, thr_q;
    uint64_t all_p, all_q;
    uint32_t t;        // MCS index at the start of the epoch
    uint32_t n_run;    // MCS to advance in this epoch (0: skip)
    BlockedGeometry geo;
};

// Arguments of the persistent ensemble kernel; the table, the order and the
// item count live in device memory so that one captured graph serves every
// epoch.
struct BatchLaunch {
    const BatchDesc* desc;
    const int32_t* order;    // slots in processing order
    const int32_t* n_items;  // number of entries of order to process
    int32_t* queue;          // work counter, reset to 0 before each launch
    int32_t lds_bytes;       // dynamic LDS per workgroup; states up to this size run from LDS
    int32_t depth;           // MCS per blocked pass in global memory (0: none)
    uint64_t* save;          // per-workgroup save areas for the blocked passes
    int64_t save_words;      // words per workgroup: 32 * depth * block threads
    int32_t* sync;           // arrival counters of split realizations, zeroed before each launch
    int32_t n_sync;          // number of counters
    int32_t* err;            // set if a barrier wait of a split realization ran out of patience
    // Behind an on-chip launch with teams: its decision, and the list, which has
    // the teams' realizations as well, that takes the other's place where it is
    // kOnChipApart, with a geometry per slot that goes before the descriptor's.
    const uint64_t* decision;  // nullptr: there is one list
    const int32_t* apart_order;
    const BlockedGeometry* apart_geometry;
    int32_t apart_items;
    int32_t* apart;            // (host memory) set in that case
};
constexpr uint64_t kOnChipApart = 3;

// Save-area words per persistent workgroup (and per part of a split
// realization) for blocked passes of up to `depth` MCS: each band (one group
// of W lanes) keeps its first and its last 2K rows, two sets of each, four
// arrays, one word per lane.
constexpr int64_t blocked_save_words(int depth, int block_threads)
{
    return 32 * (int64_t)depth * block_threads;
}

// An item of the work queue: slot in the low 20 bits, part in the bits above.
constexpr int kItemSlotBits = 20;
// Most parts one realization is split into.
constexpr int kMaxParts = 4;
// Deepest blocked pass of the persistent kernel (one 512-thread workgroup per
// CU; other shapes go to 2 MCS).
constexpr int kMaxBatchDepth = 4;

// The blocked-pass geometry of one realization split into `parts`
// workgroups: a depth K <= max_depth and a number of bands per workgroup (at
// most one per group of W lanes, groups beyond it idle) that leave every
// band at least 8K rows.  One workgroup keeps K = max_depth and idles groups
// if it must; a split realization first lowers K to keep every group busy
// (its parts are the ensemble's critical path).  Returns false if no K >= 1
// works (one workgroup needs two bands).
inline bool blocked_plan(int W, int Y, int max_depth, int block_threads, int parts, int* depth, int* bands)
{
    if (max_depth <= 0 || parts < 1 || (W != 8 && W != 16 && W != 32 && W != 64)) return false;
    const int all = block_threads / W;
    if (parts > 1)
        for (int K = max_depth; K >= 1; --K)
            if (Y / (all * parts) >= 8 * K && Y % (all * parts) == 0) {
                *depth = K;
                *bands = all;
                return true;
            }
    for (int K = max_depth; K >= 1; --K) {
        int nb = all;
        while (nb > 1 && Y / (nb * parts) < 8 * K) nb >>= 1;
        if (nb * parts >= 2 && Y / (nb * parts) >= 8 * K && Y % (nb * parts) == 0) {
            *depth = K;
            *bands = nb;
            return true;
        }
    }
    return false;
}

hipError_t launch_ensemble(const BatchLaunch& L, int block_threads, int words_per_lane, int grid, hipStream_t stream);
hipError_t launch_counter_reset(int32_t* counter, int32_t* sync, int32_t n_sync, hipStream_t stream);
// Workgroups of the persistent kernel with this shape that one compute unit
// holds at once (0 if unknown).
int ensemble_occupancy(int block_threads, int words_per_lane, int lds_bytes, int depth);

// A lattice in the registers of a team of workgroups (team.hpp).
constexpr int kTeamThreads = 1024;
constexpr int kTeamMessage = 128;  // 64-bit words per message and word of a lane: two for each of 64 lanes

// Rows per thread (2, 4 or 8; at most eight words) with which `parts` workgroups
// hold a lattice of Y rows of W words, or 0 (all of them powers of two).
inline int team_rows(int W, int64_t Y, int parts)
{
    if (W > 128 || Y < parts) return 0;
    const int64_t R = Y >> __builtin_ctz((unsigned)parts);
    for (int N = 2; N <= (W > 64 ? 4 : 8); N *= 2)
        if (R % N == 0 && R / N * (W > 64 ? 64 : W) <= kTeamThreads) return N;
    return 0;
}

// n <= kTeamMaxMcs MCS of one lattice (bit-mask mode, 16 <= W) in place by `parts`
// workgroups (4 <= parts <= kTeamMaxParts) of `rows` = team_rows rows per thread.
// The launches that share `ctl` follow one another on one stream and are not
// captured: each is given its number.
// A launch holds every compute unit, so it lasts some milliseconds at most (1.3 ms
// at 2^25 sites, 3 ms at 2^28, p = 1/2; the state's way in and out is a hundredth).
constexpr int kTeamMaxParts = 256;
constexpr int64_t kTeamMaxMcs = 512;

// Words of `ctl` that count within one launch hold the launch's number (mod
// 2^40) above the count, so that whatever earlier launches left in them counts
// nothing in this one: only launches whose team did not form write these words,
// and any number of others may lie between two of those.
constexpr int kTeamCountBits = 24;
static_assert((kTeamMaxMcs + 2) * 2 * kTeamMaxParts < 1 << kTeamCountBits, "every pass of every band has a number");
__host__ __device__ inline uint64_t team_count(uint64_t epoch, uint32_t n) { return (epoch << kTeamCountBits) | n; }
__host__ __device__ inline bool team_counts(uint64_t word, uint64_t epoch)
{
    return (word ^ (epoch << kTeamCountBits)) >> kTeamCountBits == 0;
}
__host__ __device__ inline uint32_t team_counted(uint64_t word, uint64_t epoch)
{
    return team_counts(word, epoch) ? (uint32_t)word & ((1u << kTeamCountBits) - 1u) : 0u;
}

struct TeamLaunch {
    SweepArgs a;     // a.S, a.t: the state and its MCS
    uint64_t* alt;   // the pass buffer
    int64_t n;
    uint64_t* ctl;   // team_words(W, parts), zero before the first launch
    uint64_t epoch;  // 1 for the first launch on ctl, 2 for the next, ...
    uint32_t tag;    // twice the MCS of the launches on ctl so far
    int32_t* err;    // (host memory) set if a wait ran out of patience
    int32_t* apart;  // (host memory) set if the team could not form
};
int64_t team_words(int32_t W, int parts);
hipError_t launch_team_clear(uint64_t* ctl, int32_t W, int parts, hipStream_t stream);
hipError_t launch_team(const TeamLaunch& L, bool has_q, int parts, int rows, hipStream_t stream);
void team_kernel_name(const SweepArgs& a, bool has_q, int rows, char* out, size_t n);

// After a launch whose teams did not form, this many steps of the lattice, or
// epochs of the ensemble, go without.  An attempt in vain costs a quarter of a
// millisecond, one to two hundredths of what these take where they are shortest
// (2^25 sites or one 2048^2 realization, two MCS each).
constexpr int32_t kTeamPause = 256;

// Realizations that stay on chip for an epoch (onchip.hip): bit-mask mode, in
// a team of d.parts workgroups with d.bands = team_rows rows per thread.
constexpr int kOnChipLevels = 5;  // teams of 16, 8, 4, 2 and 1 workgroups
constexpr int kOnChipMaxParts = 1 << (kOnChipLevels - 1);
struct OnChipLaunch {
    const BatchDesc* desc;
    const int32_t* order;  // slots: the lists for teams of 16 to 1 workgroups, one after another
    const int32_t* count;  // [kOnChipLevels] entries of each list
    int32_t* queue;        // [kOnChipLevels] entries taken, 0 before the launch
    uint64_t* team;        // onchip_team_words(grid), nullptr without teams
    int32_t* err;          // set if a wait ran out of patience
    int32_t* sync;         // the barrier counters (n_sync) of the kernel behind a launch with teams, which zeroes them
    int32_t n_sync;
};
int64_t onchip_team_words(int grid);
// Where a launch with teams leaves whether they formed.
const uint64_t* onchip_decision(const uint64_t* team);
// grid: workgroups, at most as many as run at once; teams: a list other than
// the last has entries.
hipError_t launch_onchip(const OnChipLaunch& L, int grid, bool teams, hipStream_t stream);
int onchip_occupancy();

hipError_t launch_philox_rate(int64_t threads, int32_t calls, uint32_t* sink, hipStream_t stream);

hipError_t launch_philox_test(const uint32_t* ctr, uint32_t k0, uint32_t k1, int64_t n,
                              uint32_t* out, hipStream_t stream);

}  // namespace sca
