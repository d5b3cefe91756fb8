// api.hip -- the C ABI declared in include/sca.h.
//
// Host side only: argument checks, the classification of p and q into the
// bit-mask path (dyadic) or the per-site compare path, the choice of launches
// for a number of MCS (even then odd sublattice each, Sec. I-A), and the
// device-to-host read-back of exact sums.
#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstdio>
#include <cstring>
#include <algorithm>
#include <map>
#include <mutex>
#include <new>
#include <vector>

#include "sca.h"
#include "sca_internal.hpp"

namespace sca {

// Acceptance parameters of one probability.
struct ProbCode {
    bool dyadic = false;
    int n = 0;              // fractional binary digits (dyadic)
    uint32_t digits = 0;    // bit i-1 = b_i
    uint64_t all = 0;       // ~0 when r == 1
    uint32_t thr = 0;       // per-site threshold, clamped to 32 bits
};

// What sca_step_ex runs for n_mcs MCS at (p, q): the acceptance path and the
// pass plan.  Groups of `depth` MCS run as fused passes alternating
// S -> pass buffer -> S (one HBM pass per group); the number of passes is
// kept even so that the caller's S holds the state after the call: an even
// number of `depth`-MCS passes, then the remainder r < 2*depth as two passes
// of ceil(r/2) and floor(r/2) MCS, or, for r = 1, two half-step launches.
// Lattices that one workgroup holds may run in place in one launch instead.
// The per-site path runs unfused from X = 8192 on: with many rows it is ALU-bound
// (2^14 squared: 52 us per half-step, 93 % of the issue rate); with few, 8192 x 64,
// it is not, and takes two launches per MCS all the same.
struct StepPlan {
    ProbCode P, Q;
    bool persite = false, has_q = false, draw_free = false;
    sca::XiMode mode = sca::XiMode::Mask;
    int32_t ndraw = 0;
    int32_t band = 0, depth = 0;
    int64_t n_pass = 0;
    int32_t tail1 = 0, tail2 = 0;
    bool whole = false;     // the lattice in one workgroup, in place: all MCS in one launch
    int32_t tile_rows = 0;  // rows per thread of the on-chip tiles, 0: row sweeps or half-step launches
    int32_t team_rows = 0;  // rows per thread of a team that holds the lattice; 0: no team
};

}  // namespace sca

using sca::ProbCode;
using sca::StepPlan;

struct sca_ctx {
    int64_t X = 0, Y = 0;
    int32_t W = 0, nb = 0;
    uint64_t seed = 0;
    uint64_t* S = nullptr;     // caller-owned state
    int64_t* aux = nullptr;    // caller-owned aux; aux[0] = h(0,0)
    hipStream_t stream = nullptr;
    int device = 0;
    int64_t t = 0;
    bool failed = false;
    int64_t* ws = nullptr;     // library-owned: partial sums [3Y], col[Y], res[8]
    int64_t* pinned = nullptr; // a result slot in host memory, or nullptr
    hipStream_t capture = nullptr;  // private stream for hipGraph capture (created on first use)
    uint64_t* alt = nullptr;        // caller-owned second state for the blocked passes (sca_set_pass_buffer)
    int32_t depth = -1;             // MCS per fused pass; -1 = automatic, 0 = never fuse
    int32_t band = 0;               // rows per workgroup in a fused pass; 0 = automatic
    // the plan of the last step, kept for the next one with the same arguments
    // (until the blocking settings or the pass buffer change)
    StepPlan plan;
    int64_t plan_n = -1;
    double plan_p = 0, plan_q = 0;
    unsigned plan_flags = 0;
    bool plan_team = false;
    // Teams (team.hip), for the lattices they serve: control words and messages
    // in device memory (library-owned; nullptr: no teams), workgroups, and the
    // launches and half-steps so far.  The slot `pinned` has two flags of theirs.
    uint64_t* team_ctl = nullptr;
    int32_t team_parts = 0;
    uint64_t team_epoch = 0;
    uint32_t team_tag = 0;
    int32_t team_pause = 0;  // steps to go without teams
};

namespace {

bool is_pow2(int64_t v) { return v > 0 && (v & (v - 1)) == 0; }

bool valid_size(int64_t X, int64_t Y)
{
    return is_pow2(X) && is_pow2(Y) && X >= 4 && Y >= 4 && X <= (1 << 17) && Y <= (1 << 17);
}

bool valid_prob(double r) { return r >= 0.0 && r <= 1.0; }  // false for NaN

// Restores the caller's current device on scope exit.
struct DeviceGuard {
    int prev = -1;
    bool ok = true;
    explicit DeviceGuard(int dev)
    {
        if (hipGetDevice(&prev) != hipSuccess) { ok = false; return; }
        if (prev != dev && hipSetDevice(dev) != hipSuccess) ok = false;
    }
    ~DeviceGuard()
    {
        int cur = -1;
        if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
    }
};

int fail(sca_ctx* c)
{
    if (c) c->failed = true;
    return SCA_EDEVICE;
}

// The word of a context's result slot that the team kernel sets: a wait ran out
// of patience [0], the team could not form [1].
int32_t* team_flags(const sca_ctx* c) { return reinterpret_cast<int32_t*>(c->pinned + 7); }

bool team_flag(const sca_ctx* c, int i)
{
    return c->team_ctl && reinterpret_cast<const volatile int32_t*>(c->pinned + 7)[i] != 0;
}

// Whether steps with these flags may run as a team.  Not as part of a graph:
// every launch has its number.
bool may_team(const sca_ctx* c, unsigned flags)
{
    return c->team_ctl && c->team_pause == 0 && !team_flag(c, 1) && !(flags & SCA_STEP_GRAPH);
}

// A step is on its way: the pause after a team that did not form begins (a launch
// still under way may set the flag once more) or gets shorter.
void count_pause(sca_ctx* c)
{
    if (team_flag(c, 1)) {
        reinterpret_cast<volatile int32_t*>(c->pinned + 7)[1] = 0;
        c->team_pause = sca::kTeamPause;
    } else if (c->team_pause > 0) {
        --c->team_pause;
    }
}

// Whether work enqueued on the stream now becomes part of a graph (or the stream
// cannot tell).
bool capturing(hipStream_t stream)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

int64_t* ws_col(sca_ctx* c) { return c->ws + 3 * c->Y; }
int64_t* ws_res(sca_ctx* c) { return c->ws + 4 * c->Y; }

ProbCode classify(double r)
{
    ProbCode c;
    const double scaled = std::ldexp(r, 32);  // exact
    const double fl = std::floor(scaled);
    c.dyadic = (fl == scaled);
    const uint64_t T = (uint64_t)fl;          // 0 .. 2^32
    c.all = (T >= (1ull << 32)) ? ~0ull : 0ull;
    c.thr = (T >= (1ull << 32)) ? 0xffffffffu : (uint32_t)T;
    if (c.dyadic && T < (1ull << 32)) {
        const uint32_t v = (uint32_t)T;       // r = v / 2^32
        for (int i = 1; i <= 32; ++i)
            if ((v >> (32 - i)) & 1u) {
                c.digits |= 1u << (i - 1);
                c.n = i;
            }
    }
    return c;
}

// Result slots: 64 bytes each of one page-locked block, which kernels write
// and the host reads after synchronizing the stream.  A copy from device
// memory to the stack instead is a launch of its own (2.8 us) and a bounce
// through the runtime's staging; with the slots and the sums in one launch a
// step and its moments at 128 x 128 take 20 us instead of 37 us.  The block is
// allocated on first use, 64 KiB once per process; a
// context takes one slot and gives it back, and goes without if none is left.
class ResultSlots {
public:
    int64_t* take()
    {
        std::lock_guard<std::mutex> lock(mu_);
        if (!block_ && !tried_) {
            tried_ = true;
            void* p = nullptr;
            if (hipHostMalloc(&p, kSlots * kWords * sizeof(int64_t), hipHostMallocPortable) == hipSuccess) {
                block_ = static_cast<int64_t*>(p);
                for (int i = kSlots - 1; i >= 0; --i) free_[n_free_++] = (int16_t)i;
            } else {
                (void)hipGetLastError();
            }
        }
        return n_free_ > 0 ? block_ + kWords * free_[--n_free_] : nullptr;
    }
    void give(int64_t* slot)
    {
        if (!slot) return;
        std::lock_guard<std::mutex> lock(mu_);
        free_[n_free_++] = (int16_t)((slot - block_) / kWords);
    }

private:
    static constexpr int kSlots = 1024, kWords = 8;
    std::mutex mu_;
    int64_t* block_ = nullptr;
    bool tried_ = false;
    int16_t free_[kSlots];
    int n_free_ = 0;
};

ResultSlots g_slots;

// Waits for the stream and reads n words that its last kernel left in `res`:
// a result slot, or device memory.
hipError_t fetch(hipStream_t stream, const int64_t* res, bool pinned, int64_t* host, size_t n)
{
    if (!pinned) {
        const hipError_t e = hipMemcpyAsync(host, res, n * sizeof(int64_t), hipMemcpyDeviceToHost, stream);
        if (e != hipSuccess) return e;
    }
    const hipError_t e = hipStreamSynchronize(stream);
    if (e == hipSuccess && pinned)
        for (size_t i = 0; i < n; ++i) host[i] = reinterpret_cast<const volatile int64_t*>(res)[i];
    return e;
}

__int128 join128(int64_t lo, int64_t hi) { return (__int128)(((unsigned __int128)(uint64_t)hi << 64) | (uint64_t)lo); }

bool fits64(__int128 v) { return v >= (__int128)INT64_MIN && v <= (__int128)INT64_MAX; }

// Moments from the sums r; SCA_OK or SCA_EOVERFLOW.
int moments_from(const int64_t r[7], int64_t X, int64_t Y, int64_t out3[3], double* w2)
{
    const __int128 s1 = join128(r[0], r[1]), s2 = join128(r[2], r[3]);
    if (!fits64(s1) || !fits64(s2)) return SCA_EOVERFLOW;
    const __int128 N = (__int128)X * Y;
    out3[0] = (int64_t)N;
    out3[1] = (int64_t)s1;
    out3[2] = (int64_t)s2;
    if (w2) *w2 = (double)(N * s2 - s1 * s1) / ((double)N * (double)N);
    return SCA_OK;
}

// Exact moments of a state at S with origin height *h0, using ws (partial
// sums [3Y], col[Y], res[8]) and, if not nullptr, the result slot `pinned`.
// *flag, a device word, returns in *flag_out with the result.  Returns SCA_OK,
// SCA_EDEVICE or SCA_EOVERFLOW.
int moments_of(const uint64_t* S, const int64_t* h0, int64_t X, int64_t Y, int32_t W, int32_t nb, int64_t* ws,
               int64_t* pinned, hipStream_t stream, int64_t out3[3], double* w2, const int32_t* flag = nullptr,
               int64_t* flag_out = nullptr)
{
    int64_t* res = pinned ? pinned : ws + 4 * Y;
    int64_t r[7];
    if (sca::launch_moments(S, h0, nullptr, nullptr, X, Y, W, nb, ws, res, flag, stream) != hipSuccess ||
        fetch(stream, res, pinned != nullptr, r, 7) != hipSuccess)
        return SCA_EDEVICE;
    if (flag_out) *flag_out = r[6];
    return moments_from(r, X, Y, out3, w2);
}

// Runs `enqueue` on a private capture stream into a hipGraph, then launches
// the instantiated graph once on `stream`.  The launch is synchronized before
// the graph is released.
template <typename F>
hipError_t run_as_graph(hipStream_t& capture, hipStream_t stream, F enqueue)
{
    if (!capture && hipStreamCreateWithFlags(&capture, hipStreamNonBlocking) != hipSuccess) return hipErrorUnknown;
    if (hipStreamBeginCapture(capture, hipStreamCaptureModeRelaxed) != hipSuccess) return hipErrorUnknown;
    const hipError_t e1 = enqueue(capture);
    hipGraph_t graph = nullptr;
    const hipError_t e2 = hipStreamEndCapture(capture, &graph);
    if (e1 != hipSuccess || e2 != hipSuccess || !graph) {
        if (graph) (void)hipGraphDestroy(graph);
        return e1 != hipSuccess ? e1 : (e2 != hipSuccess ? e2 : hipErrorUnknown);
    }
    hipGraphExec_t exec = nullptr;
    hipError_t e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e != hipSuccess) return e;
    e = hipGraphLaunch(exec, stream);
    const hipError_t es = hipStreamSynchronize(stream);
    (void)hipGraphExecDestroy(exec);
    return e != hipSuccess ? e : es;
}

// MCS per launch of a whole-lattice tile (a bound on how long one launch runs).
constexpr int64_t kWholeMcs = 1 << 14;

// The launch shape of a step is chosen by estimated time.  The estimates (in
// us) are fits to measurements on MI355X over lattices from 2^6 to 2^16 sites
// wide and high, good to some 20 %:
//  - V is the number of vector instructions per row word and half-step;
//  - a half-step of a tile with w waves per CU at work and N words per thread
//    takes V N/2 (4.7 + 0.44 w) ns, from one wave (p = 1: 0.13 us, p = 1/2:
//    0.24 us, p = 3/4, q = 1/4: 0.40 us, all latency) to sixteen (0.28, 0.58 and
//    1.0 us, all vector issue); a launch adds 2.6 us and 0.2 us per MB moved;
//  - with its words formed ahead, V (2.5 + 0.58 w) ns, and the first ones take
//    0.4 us and 5 V ns per launch;
//  - a half-step of a per-site tile takes 0.5 us and 5.8 ns (6.6 ns with
//    removals) for every word a CU draws for; unfused it takes 3.7 us, or the
//    vector issue of the chip, 24 us per 2^20 words;
//  - a half-step of a team (team.hpp) of N words per thread takes 0.12 us and the
//    vector issue of its 16 waves per CU, 8.25 V N ns, or the 1.27 us of a
//    message; a launch adds 6 us and 0.4 us per MB of state;
//  - a row sweep (fused.hpp) of b rows and d MCS walks b + 4d - 1 steps of
//    0.6 us (0.35 us at d = 1) for the row to arrive and 2d half-steps, each the longer of its
//    latency (p = 1/2 on rows of 2^16 sites: 0.21 us) and the share of the k
//    waves on its SIMD (0.065 k us); it moves its bytes at 4.7 TB/s, or 6.5 TB/s
//    where the caches hold both states;
//  - a half-step launch takes 2.95 us or its state's MB at about 5 TB/s.
// Against the rule before (bands by width alone, and none below X = 8192) 4489
// combinations of 140 sizes, five probabilities and 1 .. 60 MCS got faster by 2.5
// in the geometric mean, teams included (2^10 x 2^9 at p = 1/2: 5.2 to 0.9 us per
// MCS; 2^12 squared at p = 3/4, q = 1/4: 6.1 to 2.4 us; 2^14 squared at p = 1: 12 to
// 3.5 us), and none of 2 MCS and more slower by more than 7 % (2^13 x 2^12 at p = 1,
// 2 MCS: 13.9 to 15.0 us).  Single MCS of lattices above one workgroup's size are the
// two launches that they were.  The choice is not always the best: 2^12 x 2^16 at
// p = 1/2, 8 MCS, takes 86 us as a team and 77 us in tiles.
struct CostModel {
    double V, draws, mb;  // mb: the state in MB
    int64_t Y;
    int32_t W;
    bool has_q, draw_free, persite;

    CostModel(const sca_ctx* c, const StepPlan& pl)
        : V(30 + (pl.has_q ? 10 : 0) + 18 * pl.ndraw + 2 * pl.ndraw * (pl.has_q ? 2 : 1)), draws(pl.ndraw),
          mb(32e-6 * (double)c->Y * c->W), Y(c->Y), W(c->W), has_q(pl.has_q), draw_free(pl.draw_free), persite(pl.persite)
    {
    }
    // Whether `tiles` tiles of `rows` rows, two per thread, form the words of n
    // MCS ahead: with up to five waves of rows on a CU (with four a half-step gets
    // shorter by a sixth, with eight by nothing), and from three MCS on (the
    // first one's words are not ahead).
    bool ahead(int32_t tiles, int32_t rows, int32_t n) const
    {
        const int64_t waves = ((int64_t)rows / 2 * W + 63) / 64 * ((tiles + 255) / 256);
        return !persite && !draw_free && n > 2 && waves <= 5 && sca::tile_ahead(W, sca::TileShape{2, rows, 0, 0});
    }
    double team(int64_t n, int32_t words) const
    {
        return 6 + 0.4 * mb + 2.0 * (double)n * std::max(1.27, 0.00825 * V * words + 0.12);
    }
    double half(double waves, int32_t words) const { return V * words / 2 * (0.0047 + 0.00044 * waves); }
    // a half-step of a per-site tile with `words` words per CU to draw for
    double draw(double words) const { return words * (has_q ? 0.0066 : 0.0058); }
    double unfused() const
    {
        if (persite) return 2 * std::max(3.7, 2.2 + (double)Y * W * (has_q ? 3.0e-5 : 2.4e-5));
        return 2 * std::max(2.95, 0.37 * (1 + 0.03 * std::max(1, W / 64) + 0.025 * draws) * mb);
    }
    double whole(int64_t n) const
    {
        if (persite) return 2.6 + 2.0 * (double)n * (0.5 + draw((double)Y * W));
        const double waves = (double)((Y / 2 * W + 63) / 64);
        return 2.6 + 10 * mb + 2.0 * (double)n * (ahead(1, (int32_t)Y, (int32_t)n) ? half_ahead(waves) : half(waves, 2));
    }
    // The same with the words formed ahead (tile.hpp).
    double half_ahead(double waves) const { return V * (0.0025 + 0.00058 * waves); }
    double tile(int32_t N, int32_t b, int32_t d) const
    {
        const int I = W > 64 ? W / 64 : 1;
        const int threads = ((b + 4 * d) / N * (W / I) + 63) / 64 * 64;
        const int64_t per_cu = (Y / b + 255) / 256;  // workgroups on the busiest CU
        if (persite)
            return 2.6 + 2 * d * (0.5 * (double)((per_cu + 1) / 2) + draw((double)per_cu * (b + 2 * d) * W)) +
                   0.2 * mb * (2 + 4.0 * d / b);
        // workgroups a CU holds: of the two-row kernels by threads, of the others by registers
        if (N == 2 && ahead((int32_t)(Y / b), b + 4 * d, d))
            return 3.0 + 0.005 * V + 2 * d * half_ahead(threads / 64 * (double)(b + 2 * d) / (b + 4 * d) * (double)per_cu) +
                   0.2 * mb * (2 + 4.0 * d / b);
        const int64_t fit = std::max<int64_t>(1, (N == 2 ? 2048 : 1024) / threads);
        const int64_t rounds = (per_cu + fit - 1) / fit;
        const double busy = threads / 64 * (double)(b + 2 * d) / (b + 4 * d) * (double)std::min(per_cu, fit);
        return 2.6 + (double)rounds * 2 * d * half(busy, N * I) + 0.2 * mb * (2 + 4.0 * d / b);
    }
    double sweep(int32_t b, int32_t d) const
    {
        const double nw = W / 64;
        const double k = std::max(nw / 4, (double)(Y / b) * W / 65536.0);  // waves per SIMD
        const double lat = (0.07 + 0.08 * draws) * (nw > 1 ? 1.0 : 0.7) + 0.02 * std::log2(nw);
        const double step = draw_free ? (d >= 7 ? 0.45 + d * (0.03 + 0.025 * k) : d == 6 ? 1.25 : mb > 30 ? 1.05 : 0.75)
                                      : (d > 1 ? 0.6 : 0.35) + 2 * d * std::max(lat, k * (0.03 + 0.035 * draws));
        return 3.0 + std::max((b + 4.0 * d) * step, mb * (2 + 4.0 * d / b) / (mb > 100 ? 4.7 : 6.5));
    }
};

// Splits n MCS into an even number of passes of d MCS and two passes for the
// rest (make_plan); the estimated time of them all.
template <typename F>
double split_cost(int64_t n, int32_t d, F pass, double one)
{
    const int64_t np = (n / d) & ~(int64_t)1, rem = n - np * d;
    double t = np > 0 ? (double)np * pass(d) : 0.0;
    if (rem == 1) t += one;
    if (rem >= 2) t += pass((int32_t)((rem + 1) / 2)) + pass((int32_t)(rem / 2));
    return t;
}

// Words of a per-site tile at most: 32 KiB of acceptance words with removals.
constexpr int32_t kPersiteWords = 1024;

// Halo rows on either side of a tile's band: the 2 d that d MCS need, whole
// threads' worth.
int32_t tile_halo(int32_t N, int32_t d) { return (2 * d + N - 1) / N * N; }

bool tile_fits(int32_t W, int64_t Y, int32_t N, int32_t b, int32_t d, bool persite)
{
    const int I = W > 64 ? 2 : 1;
    // per site, the acceptance words of the whole tile lie in LDS twice
    if (persite && (N != 2 || W > 32 || (b + 4 * d) * W > kPersiteWords)) return false;
    return W <= 128 && (W <= 64 || N == 4) && Y >= b && b % N == 0 &&
           (b + 2 * tile_halo(N, d)) / N * (W / I) <= (I == 1 ? 1024 : 768);
}

// The tile of a pass of d MCS, and the mode of its acceptance words.
sca::TileShape tile_shape(const sca_ctx* c, const StepPlan& pl, int32_t d)
{
    if (pl.whole) return sca::TileShape{pl.tile_rows, (int32_t)c->Y, (int32_t)c->Y, 0};
    const int32_t halo = tile_halo(pl.tile_rows, d);
    return sca::TileShape{pl.tile_rows, pl.band + 2 * halo, pl.band, halo};
}

sca::XiMode tile_mode(const sca_ctx* c, const StepPlan& pl, const sca::TileShape& s, int64_t n_mcs)
{
    const bool ahead = s.rows_per_thread == 2 && CostModel(c, pl).ahead((int32_t)(c->Y / s.band), s.rows,
                                                                        (int32_t)std::min<int64_t>(n_mcs, 3));
    return ahead ? sca::XiMode::Ahead : pl.mode;
}

// The passes of n MCS at depth d: an even number of whole ones, and two for
// the rest unless that is a single MCS.
void set_passes(StepPlan& pl, int64_t n_mcs, bool fuse)
{
    pl.n_pass = fuse ? ((n_mcs / pl.depth) & ~(int64_t)1) : 0;
    const int64_t rem = n_mcs - pl.n_pass * pl.depth;
    pl.tail1 = (fuse && rem >= 2) ? (int32_t)((rem + 1) / 2) : 0;
    pl.tail2 = (fuse && rem >= 2) ? (int32_t)(rem / 2) : 0;
}

// Chooses by estimated time between half-step launches, the whole lattice in
// one workgroup or in a team of them, the on-chip tiles and the row sweeps.  Returns false where
// the half-step launches win.
bool plan_by_cost(const sca_ctx* c, int64_t n_mcs, bool team, StepPlan& pl)
{
    const int32_t W = c->W;
    const int64_t Y = c->Y;
    const CostModel m(c, pl);
    double best = (double)n_mcs * m.unfused();
    bool fuse = false;
    if (W < 64 && Y / 2 * W <= 1024 && (!pl.persite || Y * W <= kPersiteWords) && m.whole(n_mcs) < best) {
        best = m.whole(n_mcs);
        pl.whole = true;
        pl.tile_rows = 2;
    }
    if (!c->alt || n_mcs < 2) return false;
    auto consider = [&](double t, int32_t N, int32_t b, int32_t d) {
        if (t >= best) return;
        best = t;
        fuse = true;
        pl.whole = false;
        pl.tile_rows = N;
        pl.band = b;
        pl.depth = d;
    };
    const int32_t dmax = sca::max_fused_depth(W, pl.mode, pl.ndraw);
    // The sweep that the band and depth on entry describe (the shape of the
    // larger lattices scaled down) stays unless another shape is estimated to
    // be 15 % faster: more than the estimates err between shapes.
    const int32_t b0 = pl.band, d0 = std::min(pl.depth, dmax);
    if (d0 > 0 && sca::fused_supported(W, Y, b0, d0, pl.mode, pl.ndraw))
        consider(0.85 * split_cost(n_mcs, d0, [&](int32_t e) { return m.sweep(b0, e); }, m.unfused()), 0, b0, d0);
    // with 2 d >= n all of it is one pair of passes
    const int32_t half = (int32_t)std::min<int64_t>((n_mcs + 1) / 2, 64);
    for (int32_t b : {4, 8, 16, 32, 64, 128})
        for (int32_t dd : {1, 2, 3, 4, 6, 8, 10, 12, 16}) {
            const int32_t d = std::min(dd, half);
            for (int32_t N : {2, 4})
                if (tile_fits(W, Y, N, b, d, pl.persite))
                    consider(split_cost(n_mcs, d, [&](int32_t e) { return m.tile(N, b, e); }, m.unfused()), N, b, d);
            if (d == half) break;
        }
    for (int32_t b : {8, 16, 32, 64, 128, 256})
        for (int32_t dd : {1, 2, 3, 4, 6, 8, 10, 13}) {
            const int32_t d = std::min(dd, half);
            if (d > dmax) break;
            if (sca::fused_supported(W, Y, b, d, pl.mode, pl.ndraw))
                consider(split_cost(n_mcs, d, [&](int32_t e) { return m.sweep(b, e); }, m.unfused()), 0, b, d);
            if (d == half) break;
        }
    // A team where it is estimated to be a tenth faster, or a fifth on narrow
    // rows, whose tiles are estimated a little slow.  Without draws a
    // half-step is little more than its message, which eight words per thread
    // hide, and narrow rows leave the tiles little to repeat: 2^14 squared gets
    // faster by 1.7 (p = 1, 64 MCS: 379 to 224 us), 2^11 x 2^17 slower by 1.24.
    const int32_t N = team && !pl.persite ? sca::team_rows(W, Y, c->team_parts) : 0;
    const int32_t words = N * (W > 64 ? 2 : 1);
    if (N > 0 && (!pl.draw_free || (words == 8 && W >= 64))) {
        const int64_t rest = n_mcs % sca::kTeamMaxMcs;
        if ((double)(n_mcs / sca::kTeamMaxMcs) * m.team(sca::kTeamMaxMcs, words) + (rest ? m.team(rest, words) : 0) <
            (W < 64 ? 0.8 : 0.9) * best) {
            fuse = false;
            pl.tile_rows = 0;
            pl.whole = false;
            pl.team_rows = N;
        }
    }
    return fuse;
}

// team: the step may run as a team.
StepPlan make_plan(const sca_ctx* c, int64_t n_mcs, double p, double q, unsigned flags, bool team)
{
    StepPlan pl;
    pl.P = classify(p);
    pl.Q = classify(q);
    pl.persite = (flags & SCA_FORCE_PERSITE) || !pl.P.dyadic || !pl.Q.dyadic;
    pl.has_q = (q > 0.0);
    pl.mode = pl.persite ? sca::XiMode::PerSite : sca::XiMode::Mask;
    pl.ndraw = pl.persite ? 0 : (pl.P.n > pl.Q.n ? pl.P.n : pl.Q.n);
    const bool automatic = c->depth < 0 && c->band == 0;
    const int64_t nw = c->W >= 512 ? 8 : (c->W >= 64 ? c->W / 64 : 1);
    // Without random words (p, q in {0, 1}) a pass costs little more than
    // a shallower one as long as its window fits the registers: 13 MCS at
    // X = 2^16 and 8 below (the register-window kernels), 6 at X = 2^17 (the
    // LDS-window kernel with 1024-thread workgroups), on bands of up to 256
    // rows (about one workgroup per CU); passes with draws are ALU-bound and
    // do best at 4 MCS on bands of up to 128 rows.
    pl.draw_free = !pl.persite && pl.ndraw == 0;
    const int32_t tall = pl.draw_free ? 256 : 128;
    int32_t band = c->band;
    if (band == 0) {
        int64_t b = tall;
        while (b > 8 && c->Y / b < 2048 / nw) b >>= 1;
        band = (int32_t)b;
    }
    pl.band = band;
    const int32_t dmax = sca::max_fused_depth(c->W, pl.mode, pl.ndraw);
    int32_t depth = c->depth;
    if (depth < 0) {
        depth = pl.persite ? 0
                           : band >= 256 ? (pl.draw_free ? 13 : 4)
                           : band >= 128 ? (pl.draw_free ? 10 : 4)
                           : band >= 64 ? (pl.draw_free ? 5 : 3)
                           : band >= 32 ? 3
                           : band >= 16 ? 2
                                        : 1;
    }
    const bool may_fuse = !(flags & SCA_NO_FUSE) && (c->W < 64 ? c->depth != 0 : depth > 0) && n_mcs >= 1;
    // Lattices too small for full-height bands (and, from X = 8192 on, with the
    // pass buffer that all their passes need) go by cost, with draws also those
    // whose full-height bands make fewer than four waves per SIMD: 2^15 x 2^16 at
    // p = 15/16 takes 143 us per MCS at 4 MCS and 128 rows, 127 us at 3 and 64.
    const bool few_waves = !pl.draw_free && c->Y / band * nw < 4096;
    if (automatic && may_fuse && c->W <= 512 && (band < tall || few_waves) && (c->W < 64 || (c->alt && !pl.persite))) {
        pl.depth = depth;
        const bool fuse = plan_by_cost(c, n_mcs, team, pl);
        set_passes(pl, n_mcs, fuse);
        return pl;
    }
    if (c->W < 64) {
        // explicit depth and band, where they make a tile
        pl.depth = depth;
        bool fuse = may_fuse && depth > 0 && n_mcs >= 2 && c->alt != nullptr;
        if (fuse) {
            pl.tile_rows = tile_fits(c->W, c->Y, 2, band, depth, pl.persite)   ? 2
                           : tile_fits(c->W, c->Y, 4, band, depth, pl.persite) ? 4
                                                                               : 0;
            fuse = pl.tile_rows != 0;
        }
        set_passes(pl, n_mcs, fuse);
        return pl;
    }
    if (depth > dmax) depth = dmax;
    pl.depth = depth;
    set_passes(pl, n_mcs, may_fuse && n_mcs >= 2 && sca::fused_supported(c->W, c->Y, band, depth, pl.mode, pl.ndraw));
    return pl;
}

// Memory for teams, from 2^25 sites on (below, tiles are faster) up to what the
// compute units hold.  A context that gets none goes without, and so does one
// whose initialisation is being captured: a graph would clear the words at its
// launches instead of now.
void init_team(sca_ctx* c)
{
    int cus = 0;
    if (!c->pinned || c->W < 16 || c->X * c->Y < (1ll << 25) || capturing(c->stream) ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess)
        return;
    int parts = sca::kTeamMaxParts;
    while (parts > cus) parts /= 2;
    if (parts < 4 || sca::team_rows(c->W, c->Y, parts) == 0) return;
    uint64_t* ctl = nullptr;
    if (hipMalloc(&ctl, sizeof(uint64_t) * (size_t)sca::team_words(c->W, parts)) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    if (sca::launch_team_clear(ctl, c->W, parts, c->stream) != hipSuccess) {
        (void)hipFree(ctl);
        return;
    }
    team_flags(c)[0] = team_flags(c)[1] = 0;
    c->team_ctl = ctl;
    c->team_parts = parts;
}

hipError_t launch_team_step(sca_ctx* c, const sca::SweepArgs& a, const StepPlan& pl, int64_t n, hipStream_t stream)
{
    sca::TeamLaunch L{};
    L.a = a;
    L.alt = c->alt;
    L.n = n;
    L.ctl = c->team_ctl;
    L.epoch = ++c->team_epoch;
    L.tag = c->team_tag;
    L.err = team_flags(c);
    L.apart = team_flags(c) + 1;
    c->team_tag += 2u * (uint32_t)n;
    return sca::launch_team(L, pl.has_q, c->team_parts, pl.team_rows, stream);
}

sca::SweepArgs sweep_args(const sca_ctx* c, const StepPlan& pl)
{
    sca::SweepArgs a{};
    a.S = c->S;
    a.plane = c->Y * c->W;
    a.W = c->W;
    a.Y = (int32_t)c->Y;
    a.nb = c->nb;
    a.k0 = (uint32_t)c->seed;
    a.k1 = (uint32_t)(c->seed >> 32);
    a.h0 = c->aux;
    a.all_p = pl.P.all;
    a.all_q = pl.Q.all;
    if (pl.persite) {
        a.thr_p = pl.P.thr;
        a.thr_q = pl.Q.thr;
    } else {
        a.dig_p = pl.P.digits;
        a.dig_q = pl.Q.digits;
        a.ndraw = pl.ndraw;
    }
    return a;
}

}  // namespace

extern "C" {

size_t sca_state_words(int64_t X, int64_t Y)
{
    if (!valid_size(X, Y)) return 0;
    return (size_t)(4 * Y * (X >= 128 ? X / 128 : 1));
}

const char* sca_strerror(int code)
{
    switch (code) {
    case SCA_OK: return "ok";
    case SCA_EINVAL: return "invalid argument";
    case SCA_ENOMEM: return "device allocation failed";
    case SCA_EDEVICE: return "HIP call failed";
    case SCA_EOVERFLOW: return "exact result does not fit its output type";
    case SCA_ESTATE: return "context failed earlier";
    case SCA_EBUSY: return "capacity limit reached";
    case SCA_ENOBUF: return "a blocked pass needs the caller's pass buffer (sca_set_pass_buffer)";
    case SCA_ESCRATCH: return "lattice exceeds the static scratch of the allocation-free call (Y > SCA_NOALLOC_MAX_Y)";
    default: return "unknown status";
    }
}

int sca_init(sca_ctx** out, int64_t X, int64_t Y, uint64_t seed, void* slopes_dev, int64_t* aux_dev,
             void* hip_stream)
{
    if (!out || !slopes_dev || !aux_dev || !valid_size(X, Y)) return SCA_EINVAL;
    *out = nullptr;
    sca_ctx* c = new (std::nothrow) sca_ctx;
    if (!c) return SCA_ENOMEM;
    c->X = X;
    c->Y = Y;
    c->W = (int32_t)(X >= 128 ? X / 128 : 1);
    c->nb = (int32_t)(X >= 128 ? 64 : X / 2);
    c->seed = seed;
    c->S = static_cast<uint64_t*>(slopes_dev);
    c->aux = aux_dev;
    c->stream = static_cast<hipStream_t>(hip_stream);
    if (hipGetDevice(&c->device) != hipSuccess) { delete c; return SCA_EDEVICE; }
    if (hipMalloc(&c->ws, sizeof(int64_t) * (size_t)(4 * Y + 8)) != hipSuccess) {
        (void)hipGetLastError();
        delete c;
        return SCA_ENOMEM;
    }
    if (sca::launch_flat_init(c->S, Y, c->W, c->nb, c->aux, c->stream) != hipSuccess) {
        (void)hipFree(c->ws);
        delete c;
        return SCA_EDEVICE;
    }
    c->pinned = g_slots.take();
    init_team(c);
    *out = c;
    return SCA_OK;
}

int sca_step_ex(sca_ctx* c, int64_t n_mcs, double p, double q, unsigned flags)
{
    if (!c) return SCA_EINVAL;
    if (c->failed) return SCA_ESTATE;
    if (n_mcs < 0 || !valid_prob(p) || !valid_prob(q) ||
        (flags & ~(SCA_FORCE_PERSITE | SCA_STEP_GRAPH | SCA_NO_FUSE)))
        return SCA_EINVAL;
    if (c->t + n_mcs > (int64_t)UINT32_MAX) return SCA_EINVAL;
    if (n_mcs == 0) return SCA_OK;
    if (team_flag(c, 0)) return fail(c);
    const bool team = may_team(c, flags) && !capturing(c->stream);
    if (n_mcs != c->plan_n || p != c->plan_p || q != c->plan_q || flags != c->plan_flags || team != c->plan_team) {
        c->plan = make_plan(c, n_mcs, p, q, flags, team);
        c->plan_n = n_mcs;
        c->plan_p = p;
        c->plan_q = q;
        c->plan_flags = flags;
        c->plan_team = team;
    }
    const StepPlan& pl = c->plan;
    // the blocked passes alternate between S and the caller's pass buffer
    if (pl.n_pass + (pl.tail1 ? 2 : 0) > 0 && !c->alt) return SCA_ENOBUF;
    DeviceGuard dg(c->device);
    if (!dg.ok) return fail(c);

    sca::SweepArgs a = sweep_args(c, pl);
    const int64_t t0 = c->t;
    const int64_t n_fused = pl.n_pass * pl.depth + pl.tail1 + pl.tail2;
    auto enqueue = [&](hipStream_t st) -> hipError_t {
        if (pl.whole) {
            for (int64_t i = 0; i < n_mcs; i += kWholeMcs) {
                a.t = (uint32_t)(t0 + i);
                const sca::TileShape s = tile_shape(c, pl, 0);
                const int64_t n = std::min(kWholeMcs, n_mcs - i);
                const hipError_t e = sca::launch_tile(a, tile_mode(c, pl, s, n), pl.has_q, c->S, c->S, s, (int32_t)n, st);
                if (e != hipSuccess) return e;
            }
            return hipSuccess;
        }
        if (pl.team_rows > 0) {
            for (int64_t i = 0; i < n_mcs; i += sca::kTeamMaxMcs) {
                a.t = (uint32_t)(t0 + i);
                const hipError_t e = launch_team_step(c, a, pl, std::min(sca::kTeamMaxMcs, n_mcs - i), st);
                if (e != hipSuccess) return e;
            }
            return hipSuccess;
        }
        for (int64_t i = 0; i < pl.n_pass + (pl.tail1 ? 2 : 0); ++i) {
            const bool tail = i >= pl.n_pass;
            const int32_t d = !tail ? pl.depth : (i == pl.n_pass ? pl.tail1 : pl.tail2);
            a.t = (uint32_t)(t0 + (!tail ? i * pl.depth : pl.n_pass * pl.depth + (i == pl.n_pass ? 0 : pl.tail1)));
            const bool fwd = (i & 1) == 0;
            const uint64_t* src = fwd ? c->S : c->alt;
            uint64_t* dst = fwd ? c->alt : c->S;
            hipError_t e;
            if (pl.tile_rows > 0) {
                const sca::TileShape s = tile_shape(c, pl, d);
                e = sca::launch_tile(a, tile_mode(c, pl, s, d), pl.has_q, src, dst, s, d, st);
            } else {
                e = sca::launch_mcs_fused(a, pl.mode, pl.has_q, src, dst, pl.band, d, st);
            }
            if (e != hipSuccess) return e;
        }
        for (int64_t i = n_fused; i < n_mcs; ++i) {
            a.t = (uint32_t)(t0 + i);
            for (int parity = 0; parity < 2; ++parity) {
                a.parity = parity;
                const hipError_t e = sca::launch_halfstep(a, pl.mode, pl.has_q, st);
                if (e != hipSuccess) return e;
            }
        }
        return hipSuccess;
    };
    const hipError_t e = (flags & SCA_STEP_GRAPH) ? run_as_graph(c->capture, c->stream, enqueue) : enqueue(c->stream);
    if (e != hipSuccess) return fail(c);
    c->t += n_mcs;
    if (c->team_ctl) count_pause(c);
    return SCA_OK;
}

int sca_plan_step(const sca_ctx* c, int64_t n_mcs, double p, double q, unsigned flags, sca_step_plan* out)
{
    if (!c || !out || n_mcs < 0 || !valid_prob(p) || !valid_prob(q) ||
        (flags & ~(SCA_FORCE_PERSITE | SCA_STEP_GRAPH | SCA_NO_FUSE)))
        return SCA_EINVAL;
    const StepPlan pl = make_plan(c, n_mcs, p, q, flags, may_team(c, flags));
    std::memset(out, 0, sizeof *out);
    out->path = pl.persite ? SCA_PATH_PERSITE : (pl.draw_free ? SCA_PATH_DRAWFREE : SCA_PATH_MASK);
    out->band = pl.whole ? (int32_t)c->Y : pl.team_rows > 0 ? (int32_t)(c->Y / c->team_parts) : pl.band;
    out->n_pass = pl.n_pass;
    out->depth = pl.n_pass > 0 ? pl.depth : 0;
    out->tail1 = pl.tail1;
    out->tail2 = pl.tail2;
    out->n_unfused = pl.whole || pl.team_rows > 0 ? 0 : n_mcs - (pl.n_pass * pl.depth + pl.tail1 + pl.tail2);
    const sca::SweepArgs a = sweep_args(c, pl);
    if (pl.team_rows > 0) sca::team_kernel_name(a, pl.has_q, pl.team_rows, out->kernel, sizeof out->kernel);
    else if (pl.whole || (pl.n_pass > 0 && pl.tile_rows > 0))
        sca::tile_kernel_name(a, tile_mode(c, pl, tile_shape(c, pl, pl.depth), pl.whole ? n_mcs : pl.depth), pl.has_q,
                              pl.tile_rows, out->kernel, sizeof out->kernel);
    else if (pl.n_pass > 0) sca::fused_kernel_name(a, pl.mode, pl.has_q, pl.depth, out->kernel, sizeof out->kernel);
    else std::snprintf(out->kernel, sizeof out->kernel, "none");
    if (pl.tail1 && pl.tile_rows > 0)
        sca::tile_kernel_name(a, tile_mode(c, pl, tile_shape(c, pl, pl.tail1), pl.tail1), pl.has_q, pl.tile_rows,
                              out->tail_kernel, sizeof out->tail_kernel);
    else if (pl.tail1) sca::fused_kernel_name(a, pl.mode, pl.has_q, pl.tail1, out->tail_kernel, sizeof out->tail_kernel);
    else std::snprintf(out->tail_kernel, sizeof out->tail_kernel, "none");
    sca::halfstep_kernel_name(c->W, pl.mode, pl.has_q, out->halfstep_kernel, sizeof out->halfstep_kernel);
    return SCA_OK;
}

int sca_set_pass_buffer(sca_ctx* c, void* pass_dev, size_t bytes)
{
    if (!c) return SCA_EINVAL;
    if (c->failed) return SCA_ESTATE;
    const size_t need = sizeof(uint64_t) * (size_t)(4 * c->Y * c->W);
    if (!pass_dev) {
        c->alt = nullptr;
        c->plan_n = -1;
        return SCA_OK;
    }
    const uintptr_t a0 = (uintptr_t)pass_dev, s0 = (uintptr_t)c->S;
    if (bytes < need || (pass_dev && a0 < s0 + need && s0 < a0 + need)) return SCA_EINVAL;
    c->alt = static_cast<uint64_t*>(pass_dev);
    c->plan_n = -1;
    return SCA_OK;
}

int sca_reset(sca_ctx* c)
{
    if (!c) return SCA_EINVAL;
    if (c->failed) return SCA_ESTATE;
    DeviceGuard dg(c->device);
    if (!dg.ok) return fail(c);
    if (sca::launch_flat_init(c->S, c->Y, c->W, c->nb, c->aux, c->stream) != hipSuccess) return fail(c);
    c->t = 0;
    return SCA_OK;
}

int sca_restore(sca_ctx* c, const void* snap_dev, int64_t t)
{
    if (!c || !snap_dev || t < 0 || t > (int64_t)UINT32_MAX) return SCA_EINVAL;
    if (c->failed) return SCA_ESTATE;
    DeviceGuard dg(c->device);
    if (!dg.ok) return fail(c);
    const size_t words = (size_t)(4 * c->Y * c->W);
    const uint64_t* src = static_cast<const uint64_t*>(snap_dev);
    if (hipMemcpyAsync(c->S, src, words * sizeof(uint64_t), hipMemcpyDeviceToDevice, c->stream) != hipSuccess)
        return fail(c);
    if (hipMemcpyAsync(c->aux, src + words, sizeof(int64_t), hipMemcpyDeviceToDevice, c->stream) != hipSuccess)
        return fail(c);
    c->t = t;
    return SCA_OK;
}

int sca_step(sca_ctx* c, int64_t n_mcs, double p, double q) { return sca_step_ex(c, n_mcs, p, q, 0u); }

int sca_debug_halfstep(sca_ctx* c, int parity, const uint64_t* xi_p_dev, const uint64_t* xi_q_dev)
{
    if (!c) return SCA_EINVAL;
    if (c->failed) return SCA_ESTATE;
    if ((parity != 0 && parity != 1) || !xi_p_dev || !xi_q_dev) return SCA_EINVAL;
    DeviceGuard dg(c->device);
    if (!dg.ok) return fail(c);
    sca::SweepArgs a{};
    a.S = c->S;
    a.plane = c->Y * c->W;
    a.W = c->W;
    a.Y = (int32_t)c->Y;
    a.nb = c->nb;
    a.parity = parity;
    a.t = (uint32_t)c->t;
    a.xi_p = xi_p_dev;
    a.xi_q = xi_q_dev;
    a.h0 = c->aux;
    if (sca::launch_halfstep(a, sca::XiMode::Inject, true, c->stream) != hipSuccess) return fail(c);
    return SCA_OK;
}

int sca_debug_philox(const uint32_t* ctr_dev, uint32_t k0, uint32_t k1, int64_t n, uint32_t* out_dev,
                     void* hip_stream)
{
    if (n < 0 || (n > 0 && (!ctr_dev || !out_dev))) return SCA_EINVAL;
    if (sca::launch_philox_test(ctr_dev, k0, k1, n, out_dev, static_cast<hipStream_t>(hip_stream)) != hipSuccess)
        return SCA_EDEVICE;
    return SCA_OK;
}

int sca_debug_philox_rate(int64_t threads, int32_t calls, uint32_t* sink_dev, void* hip_stream)
{
    if (threads <= 0 || (threads % 256) != 0 || threads > ((int64_t)1 << 31) || calls <= 0 || !sink_dev)
        return SCA_EINVAL;
    if (sca::launch_philox_rate(threads, calls, sink_dev, static_cast<hipStream_t>(hip_stream)) != hipSuccess)
        return SCA_EDEVICE;
    return SCA_OK;
}

int sca_roughness(sca_ctx* c, int64_t out3[3], double* w2)
{
    if (!c || !out3) return SCA_EINVAL;
    if (c->failed) return SCA_ESTATE;
    DeviceGuard dg(c->device);
    if (!dg.ok) return fail(c);
    const int rc = moments_of(c->S, c->aux, c->X, c->Y, c->W, c->nb, c->ws, c->pinned, c->stream, out3, w2);
    if (rc == SCA_EDEVICE || team_flag(c, 0)) return fail(c);
    return rc;
}

// Moments of a caller's state without a context and without allocation: the
// row sums and the column prefix go to `scratch`, a static device array (one
// copy per GPU, held until the process ends).  Host code reaches it through
// the address hipGetSymbolAddress returns on each device, never through the
// array's name, which on the host is only a stand-in for the symbol.
static __device__ __align__(256) int64_t scratch[SCA_NOALLOC_SCRATCH_WORDS];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
int64_t* g_scratch[kMaxDevices];  // per device: the address of `scratch`, once looked up

// The address of `scratch` on the current device (looked up on the first call
// there), or nullptr on failure.
int64_t* scratch_on_current_device()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return nullptr;
        }
        g_scratch[dev] = static_cast<int64_t*>(ptr);
    }
    return g_scratch[dev];
}

}  // namespace

int sca_roughness_noalloc(const void* slopes_dev, const int64_t* aux_dev, int64_t X, int64_t Y, void* hip_stream,
                          int64_t out3[3], double* w2)
{
    if (Y > SCA_NOALLOC_MAX_Y) return SCA_ESCRATCH;
    if (!slopes_dev || !aux_dev || !out3 || !valid_size(X, Y)) return SCA_EINVAL;
    int64_t* ws = scratch_on_current_device();
    if (!ws) return SCA_EDEVICE;
    // the kernels write the partial sums and res[0, 7) before anything reads
    // them: nothing needs clearing between calls.
    const int32_t W = (int32_t)(X >= 128 ? X / 128 : 1);
    const int32_t nb = (int32_t)(X >= 128 ? 64 : X / 2);
    return moments_of(static_cast<const uint64_t*>(slopes_dev), aux_dev, X, Y, W, nb, ws, nullptr,
                      static_cast<hipStream_t>(hip_stream), out3, w2);
}

size_t sca_snapshot_bytes(const sca_ctx* c)
{
    if (!c) return 0;
    return (size_t)(4 * c->Y * c->W + 1) * sizeof(uint64_t);
}

int sca_snapshot(sca_ctx* c, void* snap_dev)
{
    if (!c || !snap_dev) return SCA_EINVAL;
    if (c->failed) return SCA_ESTATE;
    DeviceGuard dg(c->device);
    if (!dg.ok) return fail(c);
    const size_t words = (size_t)(4 * c->Y * c->W);
    uint64_t* dst = static_cast<uint64_t*>(snap_dev);
    if (hipMemcpyAsync(dst, c->S, words * sizeof(uint64_t), hipMemcpyDeviceToDevice, c->stream) != hipSuccess)
        return fail(c);
    if (hipMemcpyAsync(dst + words, c->aux, sizeof(int64_t), hipMemcpyDeviceToDevice, c->stream) != hipSuccess)
        return fail(c);
    return SCA_OK;
}

int sca_autocorr(sca_ctx* c, const void* snap_dev, int64_t out4[4], double* c_ts)
{
    if (!c || !snap_dev || !out4) return SCA_EINVAL;
    if (c->failed) return SCA_ESTATE;
    DeviceGuard dg(c->device);
    if (!dg.ok) return fail(c);
    const uint64_t* snap = static_cast<const uint64_t*>(snap_dev);
    const int64_t* snap_h0 = reinterpret_cast<const int64_t*>(snap + 4 * c->Y * c->W);
    int64_t* res = c->pinned ? c->pinned : ws_res(c);
    int64_t r[7];
    if (sca::launch_moments(c->S, c->aux, snap, snap_h0, c->X, c->Y, c->W, c->nb, c->ws, res, nullptr, c->stream) !=
            hipSuccess ||
        fetch(c->stream, res, c->pinned != nullptr, r, 7) != hipSuccess || team_flag(c, 0))
        return fail(c);
    const __int128 st = join128(r[0], r[1]), sts = join128(r[2], r[3]), ss = join128(r[4], r[5]);
    if (!fits64(st) || !fits64(sts) || !fits64(ss)) return SCA_EOVERFLOW;
    const __int128 N = (__int128)c->X * c->Y;
    out4[0] = (int64_t)N;
    out4[1] = (int64_t)sts;
    out4[2] = (int64_t)st;
    out4[3] = (int64_t)ss;
    if (c_ts) *c_ts = (double)(N * sts - st * ss) / ((double)N * (double)N);
    return SCA_OK;
}

int sca_get_meta(sca_ctx* c, int64_t* t, int64_t* h0)
{
    if (!c) return SCA_EINVAL;
    if (c->failed) return SCA_ESTATE;
    if (t) *t = c->t;
    if (h0) {
        DeviceGuard dg(c->device);
        if (!dg.ok) return fail(c);
        int64_t* res = c->pinned ? c->pinned : c->aux;
        if (c->pinned && hipMemcpyAsync(res, c->aux, sizeof(int64_t), hipMemcpyDeviceToHost, c->stream) != hipSuccess)
            return fail(c);
        if (fetch(c->stream, res, c->pinned != nullptr, h0, 1) != hipSuccess || team_flag(c, 0)) return fail(c);
    }
    return SCA_OK;
}

int sca_set_blocking(sca_ctx* c, int32_t depth, int32_t band)
{
    if (!c || depth < -1 || depth > 13 || band < 0 || (band > 0 && (band < 4 || (band & (band - 1)) != 0)))
        return SCA_EINVAL;
    c->depth = depth;
    c->band = band;
    c->plan_n = -1;
    return SCA_OK;
}

int sca_set_time(sca_ctx* c, int64_t t)
{
    if (!c || t < 0 || t > (int64_t)UINT32_MAX) return SCA_EINVAL;
    if (c->failed) return SCA_ESTATE;
    c->t = t;
    return SCA_OK;
}

int sca_heights(sca_ctx* c, int64_t y0, int64_t ny, int32_t* out_dev)
{
    if (!c) return SCA_EINVAL;
    if (c->failed) return SCA_ESTATE;
    if (y0 < 0 || ny < 0 || y0 + ny > c->Y || (ny > 0 && !out_dev)) return SCA_EINVAL;
    if (ny == 0) return SCA_OK;
    DeviceGuard dg(c->device);
    if (!dg.ok) return fail(c);
    int64_t h0 = 0;
    int64_t* res = c->pinned ? c->pinned : ws_res(c);
    if (sca::launch_column(c->S, c->aux, c->Y, c->W, ws_col(c), res, c->stream) != hipSuccess ||
        fetch(c->stream, res, c->pinned != nullptr, &h0, 1) != hipSuccess || team_flag(c, 0))
        return fail(c);
    // |h(x,y) - h(0,0)| <= x + y for any slope field
    if (h0 > INT32_MAX - c->X - c->Y || h0 < INT32_MIN + c->X + c->Y) return SCA_EOVERFLOW;
    if (sca::launch_heights(c->S, c->X, c->Y, c->W, ws_col(c), y0, ny, out_dev, c->stream) != hipSuccess)
        return fail(c);
    return SCA_OK;
}

void sca_destroy(sca_ctx* c)
{
    if (!c) return;
    {
        DeviceGuard dg(c->device);
        (void)hipStreamSynchronize(c->stream);
        (void)hipFree(c->ws);
        (void)hipFree(c->team_ctl);
        if (c->capture) (void)hipStreamDestroy(c->capture);
    }
    g_slots.give(c->pinned);
    delete c;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Ensembles
// ---------------------------------------------------------------------------
namespace {

constexpr size_t kArenaAlign = 256;

size_t state_bytes(int64_t X, int64_t Y)
{
    const size_t words = (size_t)(4 * Y * (X >= 128 ? X / 128 : 1)) + 1;  // + h(0,0)
    return (words * sizeof(uint64_t) + kArenaAlign - 1) / kArenaAlign * kArenaAlign;
}

// First-fit allocator over [0, size) with coalescing of freed ranges.
class ArenaAllocator {
public:
    void reset(size_t size)
    {
        free_.clear();
        if (size) free_[0] = size;
    }
    bool alloc(size_t bytes, size_t* off)
    {
        for (auto it = free_.begin(); it != free_.end(); ++it) {
            if (it->second >= bytes) {
                *off = it->first;
                const size_t rest = it->second - bytes;
                const size_t start = it->first + bytes;
                free_.erase(it);
                if (rest) free_[start] = rest;
                return true;
            }
        }
        return false;
    }
    void release(size_t off, size_t bytes)
    {
        auto it = free_.emplace(off, bytes).first;
        auto nx = std::next(it);
        if (nx != free_.end() && it->first + it->second == nx->first) {
            it->second += nx->second;
            free_.erase(nx);
        }
        if (it != free_.begin()) {
            auto pv = std::prev(it);
            if (pv->first + pv->second == it->first) {
                pv->second += it->second;
                free_.erase(it);
            }
        }
    }
    size_t free_bytes() const
    {
        size_t s = 0;
        for (const auto& kv : free_) s += kv.second;
        return s;
    }

private:
    std::map<size_t, size_t> free_;  // offset -> length
};

struct SlotHost {
    bool used = false;
    sca_req req{};
    size_t offset = 0, bytes = 0;
    int64_t t = 0;          // MCS reached once the enqueued epochs have run
    int32_t W = 0, nb = 0;
    int32_t instructions = 0;  // vector instructions per word and half-step, about
    sca::BatchDesc desc{};     // static part; the rest is set per epoch
};

// A realization with work in an epoch.
struct EpochItem {
    int64_t run, sites, cost;  // MCS, site updates, vector instructions of a lane
    int32_t slot, W, Y;
    int32_t parts, rows;       // on chip: workgroups (0: not there) and rows per thread
    bool mask;
};

bool valid_req(const sca_req& r)
{
    return valid_size(r.X, r.Y) && r.X <= 8192 && valid_prob(r.p) && valid_prob(r.q) && r.n_mcs >= 0 &&
           r.n_mcs <= (int64_t)UINT32_MAX && (r.flags & ~SCA_FORCE_PERSITE) == 0 && r.reserved == 0;
}

bool valid_cfg(const sca_batch_config& c)
{
    return (c.block_threads == 256 || c.block_threads == 512 || c.block_threads == 1024) && c.blocks_per_cu >= 1 &&
           c.blocks_per_cu <= 8 && c.lds_bytes >= 0 && c.lds_bytes <= 65536 && (c.lds_bytes % 8) == 0 &&
           (c.order == 0 || c.order == 1) && (c.words_per_lane == 1 || c.words_per_lane == 2) && c.depth >= 0 &&
           (c.depth <= 2 || (c.depth <= sca::kMaxBatchDepth && c.block_threads == 512 && c.blocks_per_cu == 1)) &&
           (c.max_parts == 1 || c.max_parts == 2 || c.max_parts == sca::kMaxParts);
}

}  // namespace

struct sca_batch {
    int device = 0;
    hipStream_t stream = nullptr;
    hipStream_t capture = nullptr;
    uint8_t* arena = nullptr;
    size_t arena_bytes = 0;
    int32_t max_slots = 0;
    int num_cus = 0;
    std::vector<SlotHost> slots;
    std::vector<int32_t> free_slots;  // stack of free slot ids
    ArenaAllocator alloc;
    sca_batch_config cfg{512, 2, 65536, 0, 1, 2, 1};
    uint64_t* d_save = nullptr;     // save areas of the blocked passes: grid x save words per workgroup,
                                    // then grid x save words for the parts of split realizations
    size_t save_bytes = 0;
    bool prepared = false;          // the next three are up to date with the configuration
    sca::BatchLaunch launch{};      // the persistent kernel's arguments
    int64_t save_words = 0;         // per workgroup (and per part)
    int32_t resident = 0;           // workgroups of that launch that run at once
    int32_t* d_sync = nullptr;      // barrier counters of split realizations (one per part slot of the grid)
    uint64_t* d_team = nullptr;     // formation, posts and messages of on-chip teams (allocated on first use)
    bool no_teams = false;          // there was no memory for them
    int32_t team_pause = 0;         // epochs to go without
    int32_t cu_grid = 0;            // workgroups of the on-chip launch: one per compute unit, 0 if it does not fit
    int32_t* d_err = nullptr;       // set by a barrier wait that gave up
    int32_t* h_err = nullptr;       // pinned copy of d_err, written after each launch
    hipEvent_t err_copied = nullptr;
    bool err_pending = false;
    // device (library-owned)
    sca::BatchDesc* d_desc = nullptr;
    int32_t* d_order = nullptr;
    int32_t* d_counters = nullptr;  // kCounters words, see below
    int64_t* d_ws = nullptr;        // moments workspace for Y up to 131072
    // sca_batch_collect: kCollect result slots of 8 words (the first one is also
    // sca_batch_roughness's), behind them as many items, a word that a launch sets
    // whose teams could not form, and two lists for those in turn; pinned
    int64_t* results = nullptr;
    int apart_at = 0;               // the list of the last epoch with teams
    // pinned staging
    sca::BatchDesc* h_desc = nullptr;
    int32_t* h_order = nullptr;
    int32_t* h_count = nullptr;
    hipEvent_t staged = nullptr;
    bool staged_pending = false;
    // flat initialisation of many admitted realizations
    sca::FlatItem* h_flat = nullptr;  // pinned staging
    sca::FlatItem* d_flat = nullptr;
    hipEvent_t flat_staged = nullptr;
    bool flat_pending = false;
    hipGraphExec_t exec = nullptr;
    bool failed = false;
    // an epoch's lists, kept for their memory
    std::vector<EpochItem> epoch_items;
    std::vector<std::pair<int64_t, int32_t>> epoch_work, epoch_apart, epoch_chip[sca::kOnChipLevels];
    std::vector<int32_t> epoch_whole, epoch_plain;
};

namespace {

// The launch counters, staged and copied with the order: the persistent
// kernel's item count and queue, then the on-chip kernel's list lengths
// and queues (the copy zeroes the queues).
enum {
    kItems = 0,
    kQueue = 1,
    kOnChipCount = 4,
    kOnChipQueue = kOnChipCount + sca::kOnChipLevels,
    kCounters = kOnChipQueue + sca::kOnChipLevels
};

constexpr int32_t kCollect = 256;  // realizations per launch and wait of sca_batch_collect

sca::MomentsItem* collect_items(const sca_batch* b)
{
    return reinterpret_cast<sca::MomentsItem*>(b->results + 8 * kCollect);
}

int32_t* batch_apart(const sca_batch* b) { return reinterpret_cast<int32_t*>(collect_items(b) + kCollect); }

// The list of an epoch for teams that do not form, and its geometries by slot.  An
// epoch's launches may still read one of the two of them when the next is planned;
// the one before has ended, as this epoch waited for the last one's copies.
size_t apart_orders(const sca_batch* b) { return ((size_t)b->max_slots + (size_t)b->num_cus * 8 + 1) / 2 * 2; }

size_t apart_bytes(const sca_batch* b)
{
    return sizeof(sca::BlockedGeometry) * (size_t)b->max_slots + sizeof(int32_t) * apart_orders(b);
}

sca::BlockedGeometry* apart_geometry(const sca_batch* b)
{
    return reinterpret_cast<sca::BlockedGeometry*>(reinterpret_cast<uint8_t*>(batch_apart(b)) + sizeof(int64_t) +
                                                   apart_bytes(b) * (size_t)b->apart_at);
}

int32_t* apart_order(const sca_batch* b) { return reinterpret_cast<int32_t*>(apart_geometry(b) + b->max_slots); }

int bfail(sca_batch* b)
{
    if (b) b->failed = true;
    return SCA_EDEVICE;
}

void batch_free(sca_batch* b)
{
    if (b->exec) (void)hipGraphExecDestroy(b->exec);
    if (b->staged) (void)hipEventDestroy(b->staged);
    if (b->flat_staged) (void)hipEventDestroy(b->flat_staged);
    (void)hipFree(b->d_flat);
    (void)hipHostFree(b->h_flat);
    if (b->capture) (void)hipStreamDestroy(b->capture);
    (void)hipFree(b->d_desc);
    (void)hipFree(b->d_order);
    (void)hipFree(b->d_counters);
    (void)hipFree(b->d_ws);
    (void)hipFree(b->d_save);
    (void)hipFree(b->d_sync);
    (void)hipFree(b->d_team);
    (void)hipFree(b->d_err);
    (void)hipHostFree(b->h_err);
    if (b->err_copied) (void)hipEventDestroy(b->err_copied);
    (void)hipHostFree(b->h_desc);
    (void)hipHostFree(b->h_order);
    (void)hipHostFree(b->h_count);
    (void)hipHostFree(b->results);
    delete b;
}

// The persistent kernel's arguments in the current configuration, with the save
// areas that they name (no launch of another configuration is in flight: callers
// synchronize first).
void prepare_launch(sca_batch* b)
{
    if (b->prepared) return;
    const int grid = b->num_cus * b->cfg.blocks_per_cu;
    int32_t depth = b->cfg.depth;
    int64_t save_words = sca::blocked_save_words(depth, b->cfg.block_threads);
    // per-workgroup save areas, then as many again for the parts of split realizations
    const size_t need = sizeof(uint64_t) * (size_t)save_words * (size_t)grid * 2;
    if (need > b->save_bytes) {
        (void)hipFree(b->d_save);
        b->d_save = nullptr;
        b->save_bytes = 0;
        if (hipMalloc(&b->d_save, need) == hipSuccess) {
            b->save_bytes = need;
        } else {
            (void)hipGetLastError();
            depth = 0;  // no room for the save areas: unblocked half-steps
            save_words = 0;
        }
    }
    b->save_words = depth > 0 ? save_words : 0;
    const int occ = sca::ensemble_occupancy(b->cfg.block_threads, b->cfg.words_per_lane, b->cfg.lds_bytes, depth);
    b->resident = std::min(grid, occ * b->num_cus);
    sca::BatchLaunch L{};
    L.desc = b->d_desc;
    L.order = b->d_order;
    L.n_items = b->d_counters + kItems;
    L.queue = b->d_counters + kQueue;
    L.lds_bytes = b->cfg.lds_bytes;
    L.depth = depth;
    L.save = b->d_save;
    L.save_words = save_words;
    L.sync = b->d_sync;
    L.n_sync = grid;
    L.err = b->d_err;
    b->launch = L;
    b->prepared = true;
}

// Captures the epoch graph: reset the work counter, then the persistent kernel.
// The table, order and count are read from device memory, so the graph is reused
// for every epoch until the configuration changes.
hipError_t capture_epoch_graph(sca_batch* b)
{
    const int grid = b->num_cus * b->cfg.blocks_per_cu;
    if (!b->capture && hipStreamCreateWithFlags(&b->capture, hipStreamNonBlocking) != hipSuccess)
        return hipErrorUnknown;
    if (hipStreamBeginCapture(b->capture, hipStreamCaptureModeRelaxed) != hipSuccess) return hipErrorUnknown;
    hipError_t e1 = sca::launch_counter_reset(b->d_counters + kQueue, b->d_sync, grid, b->capture);
    if (e1 == hipSuccess)
        e1 = sca::launch_ensemble(b->launch, b->cfg.block_threads, b->cfg.words_per_lane, grid, b->capture);
    hipGraph_t graph = nullptr;
    const hipError_t e2 = hipStreamEndCapture(b->capture, &graph);
    if (e1 != hipSuccess || e2 != hipSuccess || !graph) {
        if (graph) (void)hipGraphDestroy(graph);
        return e1 != hipSuccess ? e1 : (e2 != hipSuccess ? e2 : hipErrorUnknown);
    }
    const hipError_t e = hipGraphInstantiate(&b->exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    return e;
}

}  // namespace

extern "C" {

size_t sca_batch_state_bytes(int64_t X, int64_t Y)
{
    if (!valid_size(X, Y)) return 0;
    return state_bytes(X, Y);
}

int sca_batch_create(sca_batch** out, int32_t max_slots, void* arena_dev, size_t arena_bytes, void* hip_stream)
{
    if (!out || max_slots <= 0 || max_slots > (1 << 20) || (!arena_dev && arena_bytes)) return SCA_EINVAL;
    *out = nullptr;
    sca_batch* b = new (std::nothrow) sca_batch;
    if (!b) return SCA_ENOMEM;
    b->stream = static_cast<hipStream_t>(hip_stream);
    b->arena = static_cast<uint8_t*>(arena_dev);
    b->arena_bytes = arena_bytes;
    b->max_slots = max_slots;
    try {
        b->slots.resize((size_t)max_slots);
        b->free_slots.reserve((size_t)max_slots);
    } catch (...) {
        delete b;
        return SCA_ENOMEM;
    }
    for (int32_t s = max_slots - 1; s >= 0; --s) b->free_slots.push_back(s);
    b->alloc.reset(arena_bytes);
    if (hipGetDevice(&b->device) != hipSuccess ||
        hipDeviceGetAttribute(&b->num_cus, hipDeviceAttributeMultiprocessorCount, b->device) != hipSuccess) {
        delete b;
        return SCA_EDEVICE;
    }
    // the work queue holds one item per realization, plus one more per extra
    // part of a split realization (at most one part per persistent workgroup
    // in all, and at most 8 of those per compute unit)
    const size_t nd = sizeof(sca::BatchDesc) * (size_t)max_slots,
                 no = sizeof(int32_t) * ((size_t)max_slots + (size_t)b->num_cus * 8);
    if (hipMalloc(&b->d_desc, nd) != hipSuccess || hipMalloc(&b->d_order, no) != hipSuccess ||
        hipMalloc(&b->d_counters, kCounters * sizeof(int32_t)) != hipSuccess ||
        hipMalloc(&b->d_ws, sizeof(int64_t) * (size_t)(4 * 131072 + 8)) != hipSuccess ||
        hipHostMalloc(&b->h_desc, nd, hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc(&b->h_order, no, hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc(&b->h_count, kCounters * sizeof(int32_t), hipHostMallocDefault) != hipSuccess ||
        hipEventCreateWithFlags(&b->staged, hipEventDisableTiming) != hipSuccess ||
        hipMalloc(&b->d_flat, sizeof(sca::FlatItem) * (size_t)max_slots) != hipSuccess ||
        hipHostMalloc(&b->h_flat, sizeof(sca::FlatItem) * (size_t)max_slots, hipHostMallocDefault) != hipSuccess ||
        hipEventCreateWithFlags(&b->flat_staged, hipEventDisableTiming) != hipSuccess ||
        hipMalloc(&b->d_sync, sizeof(int32_t) * (size_t)b->num_cus * 8) != hipSuccess ||
        hipMalloc(&b->d_err, sizeof(int32_t)) != hipSuccess ||
        hipHostMalloc(&b->h_err, sizeof(int32_t), hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc(&b->results, kCollect * (8 * sizeof(int64_t) + sizeof(sca::MomentsItem)) + sizeof(int64_t) + 2 * apart_bytes(b),
                      hipHostMallocDefault) != hipSuccess ||
        hipEventCreateWithFlags(&b->err_copied, hipEventDisableTiming) != hipSuccess ||
        hipMemsetAsync(b->d_err, 0, sizeof(int32_t), b->stream) != hipSuccess) {
        (void)hipGetLastError();
        batch_free(b);
        return SCA_ENOMEM;
    }
    std::memset(b->h_desc, 0, nd);
    *b->h_err = 0;
    *batch_apart(b) = 0;
    b->cu_grid = sca::onchip_occupancy() > 0 ? b->num_cus : 0;
    *out = b;
    return SCA_OK;
}

int sca_batch_set_config(sca_batch* b, const sca_batch_config* cfg)
{
    if (!b || !cfg || !valid_cfg(*cfg)) return SCA_EINVAL;
    if (b->failed) return SCA_ESTATE;
    const bool same = cfg->block_threads == b->cfg.block_threads && cfg->blocks_per_cu == b->cfg.blocks_per_cu &&
                      cfg->lds_bytes == b->cfg.lds_bytes && cfg->order == b->cfg.order &&
                      cfg->words_per_lane == b->cfg.words_per_lane && cfg->depth == b->cfg.depth;
    if (same) {
        b->cfg.max_parts = cfg->max_parts;  // a host-side choice: the graph stays
        return SCA_OK;
    }
    DeviceGuard dg(b->device);
    if (!dg.ok) return bfail(b);
    // the old graph may still be in flight on the stream
    if (hipStreamSynchronize(b->stream) != hipSuccess) return bfail(b);
    b->cfg = *cfg;
    b->prepared = false;
    if (b->exec) {
        (void)hipGraphExecDestroy(b->exec);
        b->exec = nullptr;
    }
    return SCA_OK;
}

int sca_batch_get_config(const sca_batch* b, sca_batch_config* cfg)
{
    if (!b || !cfg) return SCA_EINVAL;
    *cfg = b->cfg;
    return SCA_OK;
}

int sca_batch_admit(sca_batch* b, const sca_req* reqs, int32_t n, int32_t* slots_out)
{
    if (!b || n < 0 || (n > 0 && (!reqs || !slots_out))) return SCA_EINVAL;
    if (b->failed) return SCA_ESTATE;
    for (int32_t i = 0; i < n; ++i)
        if (!valid_req(reqs[i])) return SCA_EINVAL;
    if ((size_t)n > b->free_slots.size()) return SCA_EBUSY;
    // all or nothing: place every state first
    std::vector<size_t> offs((size_t)n);
    int32_t placed = 0;
    for (; placed < n; ++placed) {
        if (!b->alloc.alloc(state_bytes(reqs[placed].X, reqs[placed].Y), &offs[(size_t)placed])) break;
    }
    if (placed < n) {
        for (int32_t i = 0; i < placed; ++i)
            b->alloc.release(offs[(size_t)i], state_bytes(reqs[i].X, reqs[i].Y));
        return SCA_EBUSY;
    }
    DeviceGuard dg(b->device);
    if (!dg.ok) return bfail(b);
    // few states go as an argument of their launch, many through a staged table,
    // which is free once the previous table's copy has run
    sca::FlatItem few[sca::kFlatFew];
    sca::FlatItem* flat = few;
    if (n > sca::kFlatFew) {
        if (b->flat_pending && hipEventSynchronize(b->flat_staged) != hipSuccess) return bfail(b);
        b->flat_pending = false;
        flat = b->h_flat;
    }
    int32_t n_flat = 0;
    for (int32_t i = 0; i < n; ++i) {
        const sca_req& r = reqs[i];
        const int32_t slot = b->free_slots.back();
        b->free_slots.pop_back();
        SlotHost& s = b->slots[(size_t)slot];
        s.used = true;
        s.req = r;
        s.offset = offs[(size_t)i];
        s.bytes = state_bytes(r.X, r.Y);
        s.t = 0;
        s.W = (int32_t)(r.X >= 128 ? r.X / 128 : 1);
        s.nb = (int32_t)(r.X >= 128 ? 64 : r.X / 2);
        const ProbCode P = classify(r.p), Q = classify(r.q);
        const bool persite = (r.flags & SCA_FORCE_PERSITE) || !P.dyadic || !Q.dyadic;
        sca::BatchDesc& d = s.desc;
        d = sca::BatchDesc{};
        d.S = reinterpret_cast<uint64_t*>(b->arena + s.offset);
        d.plane = r.Y * s.W;
        d.h0 = reinterpret_cast<int64_t*>(d.S + 4 * d.plane);
        d.W = s.W;
        d.Y = (int32_t)r.Y;
        d.nb = s.nb;
        d.mode = persite ? 1 : 0;
        d.k0 = (uint32_t)r.seed;
        d.k1 = (uint32_t)(r.seed >> 32);
        d.all_p = P.all;
        d.all_q = Q.all;
        d.has_q = r.q > 0.0 ? 1 : 0;
        if (persite) {
            d.thr_p = P.thr;
            d.thr_q = Q.thr;
        } else {
            d.dig_p = P.digits;
            d.dig_q = Q.digits;
            d.ndraw = P.n > Q.n ? P.n : Q.n;
        }
        const int32_t nd = persite ? 32 : d.ndraw;
        s.instructions = 30 + 10 * d.has_q + 18 * nd + 2 * nd * (1 + d.has_q);
        // states of up to 2^20 words share one launch; larger ones get a launch of their own
        if (4 * d.plane <= ((int64_t)1 << 20)) {
            flat[n_flat++] = sca::flat_item(d.S, r.Y, s.W, s.nb, d.h0);
        } else if (sca::launch_flat_init(d.S, r.Y, s.W, s.nb, d.h0, b->stream) != hipSuccess) {
            return bfail(b);
        }
        slots_out[i] = slot;
    }
    if (flat == few) {
        if (sca::launch_flat_init_few(few, n_flat, b->stream) != hipSuccess) return bfail(b);
    } else if (n_flat > 0) {
        if (hipMemcpyAsync(b->d_flat, b->h_flat, sizeof(sca::FlatItem) * (size_t)n_flat, hipMemcpyHostToDevice,
                           b->stream) != hipSuccess ||
            hipEventRecord(b->flat_staged, b->stream) != hipSuccess ||
            sca::launch_flat_init_many(b->d_flat, n_flat, b->stream) != hipSuccess)
            return bfail(b);
        b->flat_pending = true;
    }
    return SCA_OK;
}

}  // extern "C"

namespace {

// Whether the smallest realizations go to the persistent kernel's LDS after all.
// On chip each takes a workgroup of 1024 threads, one per compute unit, mostly idle
// below 512 words per sublattice; workgroups of 256 threads run up to three such
// states side by side on a unit.  With many of them that is faster, with few the
// latency of one counts, which the on-chip kernel has the lower: 60 MCS of 8192
// lattices of 128^2 at p = 15/16 take 3.2 ms on chip and 1.5 ms in LDS, of 256 of
// them 140 and 181 us.  Larger workgroups are no faster (512 threads, 2 per unit:
// 0.65 us per half-step of a unit at p = 1/2, on chip 0.46), nor is one per unit.
// Times in us, fitted to 4^2 .. 256^2 and 512 x 256 at p = 1/2, 3/4, 15/16 and 1; the
// estimate has to be 15 % worse before a case that LDS can serve stays on chip.
struct SmallStates {
    static constexpr int kLdsPerCu = 160 * 1024;
    double rounds_in_lds;               // of a compute unit for one state
    double chip = 0, chip_longest = 0;  // of all of them on chip, and of the longest
    double lds = 0, lds_longest = 0;    // and in LDS

    explicit SmallStates(const sca_batch_config& c)
        : rounds_in_lds(c.blocks_per_cu >= 3 && 3 * c.lds_bytes <= kLdsPerCu ? 1 : 1.45)
    {
    }
    static bool served(const sca_batch_config& c)
    {
        return c.block_threads == 256 && c.blocks_per_cu >= 2 && 2 * c.lds_bytes <= kLdsPerCu;
    }
    static bool fits(const sca_batch_config& c, const EpochItem& it)
    {
        const int64_t words = (int64_t)it.Y * it.W;
        return it.mask && words <= 512 && 32 * words <= c.lds_bytes;
    }
    void add(const EpochItem& it)
    {
        const int64_t words = (int64_t)it.Y * it.W;
        const double h = 2 * (double)it.run, V = (double)it.cost / ((double)it.run * (double)words);
        const double on_chip = 9 + h * (0.12 + 0.0048 * V + (words >= 128 ? 0.1 : 0)), loops = words > 256 ? 2 : 1;
        chip += on_chip;
        chip_longest = std::max(chip_longest, on_chip);
        lds += (7 + h * (0.126 + 0.002 * V) * loops) * rounds_in_lds;
        lds_longest = std::max(lds_longest, 15 + h * (0.75 + 0.004 * V) * loops);
    }
    // others: the same for the rest of the on-chip realizations
    bool in_lds(int cus, double others, double others_longest) const
    {
        // beyond one round the last ones do not come out even: 661 of 32^2 make three
        const double tail = std::max(0.0, std::min(0.4 * chip_longest, chip / cus - chip_longest));
        const double together = std::max((chip + others) / cus + tail, std::max(chip_longest, others_longest));
        return chip > 0 &&
               std::max(others / cus, others_longest) + std::max(lds / cus, lds_longest) < 1.15 * together;
    }
};

// One epoch in which slot s advances mcs_of(s) MCS (clamped to its budget).
template <typename F>
int batch_epoch(sca_batch* b, F mcs_of, int32_t* active_out)
{
    if (b->failed) return SCA_ESTATE;
    DeviceGuard dg(b->device);
    if (!dg.ok) return bfail(b);
    if (b->err_pending && hipEventQuery(b->err_copied) == hipSuccess) {
        b->err_pending = false;
        if (*b->h_err) return bfail(b);  // a split realization's barrier gave up: its state is not valid
    }
    // the staging buffers are free once the previous epoch's copies have run
    if (b->staged_pending && hipEventSynchronize(b->staged) != hipSuccess) return bfail(b);
    b->staged_pending = false;
    // The slots with work, in a table of their own: the slots themselves lie far apart.
    auto& items = b->epoch_items;
    items.clear();
    int32_t hi = -1;
    int64_t total = 0;
    for (int32_t slot = 0; slot < b->max_slots; ++slot) {
        const SlotHost& s = b->slots[(size_t)slot];
        if (!s.used) continue;
        const int64_t run = std::min(mcs_of(s), s.req.n_mcs - s.t);
        if (run <= 0) continue;
        EpochItem it;
        it.slot = hi = slot;
        it.W = s.W;
        it.Y = (int32_t)s.req.Y;
        it.mask = s.desc.mode == 0;
        it.run = run;
        it.sites = run * s.req.X * s.req.Y;
        it.cost = run * s.req.Y * s.W * s.instructions;
        total += it.cost;
        items.push_back(it);
    }
    if (active_out) *active_out = (int32_t)items.size();
    if (items.empty()) return SCA_OK;
    // A graph of an epoch would replay whatever the staging buffers hold by then.
    if (capturing(b->stream)) return bfail(b);
    // After teams that could not form come epochs without.
    volatile int32_t* const apart = batch_apart(b);
    if (*apart != 0) {
        *apart = 0;
        b->team_pause = sca::kTeamPause;
    }
    const bool paused = b->team_pause > 0;
    if (paused) --b->team_pause;
    // On chip (unless the configuration keeps states in the arena) go the
    // bit-mask realizations that up to sixteen workgroups hold, with as few
    // workgroups as do, or more where each would have more than half of the
    // average work per compute unit and its rows per thread can still be halved.
    // Work is counted in vector instructions (p = 15/16 takes more than twice
    // those of p = 1/2 per site).  512 realizations of 2^6 to 2^11 squared: 3.6 ms;
    // with a whole average as the line 4.4 ms, with a third or a sixth of it 1.5
    // and 5 % more, with sites for work and a whole average 5.2 ms.
    const int64_t chip_share = b->cu_grid > 0 ? total / (2 * b->cu_grid) : 0;
    auto place = [&](int max_parts) {  // whether there are teams
        bool teams = false;
        for (EpochItem& it : items) {
            it.parts = 0;
            if (b->cfg.lds_bytes == 0 || !it.mask) continue;
            for (int32_t P = 1; P <= max_parts; P *= 2) {
                const int N = sca::team_rows(it.W, it.Y, P);
                if (N == 0) continue;
                const bool more = b->cfg.order == 0 && it.cost >= (chip_share + 1) * P && N > 2 && 2 * P <= max_parts;
                if (more && sca::team_rows(it.W, it.Y, 2 * P) > 0) continue;
                it.parts = P;
                it.rows = N;
                teams = teams || P > 1;
                break;
            }
        }
        return teams;
    };
    bool teams = place(std::min(paused || b->no_teams ? 1 : sca::kOnChipMaxParts, b->cu_grid));
    if (teams && !b->d_team &&
        hipMalloc(&b->d_team, sizeof(uint64_t) * (size_t)sca::onchip_team_words(b->cu_grid)) != hipSuccess) {
        (void)hipGetLastError();
        b->d_team = nullptr;
        b->no_teams = true;
        teams = place(1);
    }
    if (SmallStates::served(b->cfg)) {
        SmallStates small(b->cfg);
        double others = 0, others_longest = 0;
        for (const EpochItem& it : items) {
            if (it.parts == 0) continue;
            if (SmallStates::fits(b->cfg, it)) {
                small.add(it);
            } else {
                const double V = (double)it.cost / ((double)it.run * it.W * it.Y);
                const double t = 9 + 2 * (double)it.run * (0.12 + 0.006 * V * it.rows);
                others += t * it.parts;
                others_longest = std::max(others_longest, t);
            }
        }
        if (small.in_lds(b->cu_grid, others, others_longest))
            for (EpochItem& it : items)
                if (SmallStates::fits(b->cfg, it)) it.parts = 0;
    }
    // The lists, as items with a key: on chip by size of team, the persistent
    // kernel's, and, should the teams not form, its list with everything but the
    // single workgroups' realizations.
    auto &work = b->epoch_work, &apart_work = b->epoch_apart;
    work.clear();
    apart_work.clear();
    for (auto& list : b->epoch_chip) list.clear();
    int64_t work_total = 0, apart_total = 0;
    for (int32_t i = 0; i < (int32_t)items.size(); ++i) {
        const EpochItem& it = items[(size_t)i];
        const SlotHost& s = b->slots[(size_t)it.slot];
        sca::BatchDesc& d = b->h_desc[it.slot];
        d = s.desc;
        d.t = (uint32_t)s.t;
        d.n_run = (uint32_t)it.run;
        d.geo = sca::BlockedGeometry{0, it.parts > 0 ? it.rows : 0, std::max(it.parts, 1), 0, nullptr};
        if (it.parts > 0) {
            b->epoch_chip[sca::kOnChipLevels - 1 - __builtin_ctz((unsigned)it.parts)].emplace_back(it.cost, i);
        } else {
            work.emplace_back(it.sites, i);
            work_total += it.sites;
        }
        if (teams && it.parts != 1) {
            apart_work.emplace_back(it.sites, i);
            apart_total += it.sites;
        }
    }
    b->epoch_whole.reserve(items.size());  // nothing is allocated once the first kernel is launched
    b->epoch_plain.reserve(items.size());
    const auto longer = [](const std::pair<int64_t, int32_t>& x, const std::pair<int64_t, int32_t>& y) {
        return x.first > y.first;
    };
    // The save areas and their depth decide which realizations can run blocked.
    if (!work.empty()) prepare_launch(b);
    const int32_t grid = b->num_cus * b->cfg.blocks_per_cu;
    // The persistent kernel's list of `list` (site updates in all: sum) into `order`;
    // returns its length.  geometry(slot) is where the realization's goes.
    // Realizations that run as temporally blocked passes go first (the
    // kernel takes them in a phase of their own), and among them the split
    // ones: a blocked realization with more work than the average per
    // persistent workgroup runs on parts = the smallest power of two that
    // brings its share under that average (at most max_parts, as the band
    // geometry allows), while the parts in all stay within `room`, a number of
    // persistent workgroups that the device runs at once, so that every part
    // is taken by a running workgroup's first pop.
    int32_t n_split = 0;
    auto list_work = [&](std::vector<std::pair<int64_t, int32_t>>& list, int64_t sum, int32_t room, int32_t* order,
                         auto&& geometry) {
        if (b->cfg.order == 0) std::stable_sort(list.begin(), list.end(), longer);
        const int64_t avg = sum / grid;
        const int32_t max_depth = b->save_words > 0 ? b->cfg.depth : 0;
        int32_t parts_used = 0, split = 0, n = 0;
        auto &whole = b->epoch_whole, &plain = b->epoch_plain;
        whole.clear();
        plain.clear();
        for (const auto& w : list) {
            const EpochItem& it = items[(size_t)w.second];
            sca::BlockedGeometry g{0, 0, 1, 0, nullptr};
            if (it.mask)
                (void)sca::blocked_plan(it.W, it.Y, max_depth, b->cfg.block_threads, 1, &g.depth, &g.bands);
            if (g.depth > 0 && b->cfg.order == 0)
                for (int32_t p2 = 2; p2 <= b->cfg.max_parts && w.first / (p2 / 2) > avg; p2 *= 2) {
                    int32_t K2 = 0, nb2 = 0;
                    if (parts_used + p2 > room ||
                        !sca::blocked_plan(it.W, it.Y, max_depth, b->cfg.block_threads, p2, &K2, &nb2))
                        break;
                    g.parts = p2;
                    g.depth = K2;
                    g.bands = nb2;
                }
            if (g.parts > 1) {
                g.sync_idx = split++;
                g.save = b->d_save + (size_t)b->save_words * (size_t)(grid + parts_used);
                parts_used += g.parts;
                for (int32_t m = 0; m < g.parts; ++m) order[n++] = it.slot | (m << sca::kItemSlotBits);
            } else {
                (g.depth > 0 ? whole : plain).push_back(it.slot);
            }
            geometry(it.slot) = g;
        }
        for (const int32_t slot : whole) order[n++] = slot;
        for (const int32_t slot : plain) order[n++] = slot;
        n_split += split;
        return n;
    };
    const int32_t n_work = list_work(work, work_total, b->resident, b->h_order,
                                     [b](int32_t slot) -> sca::BlockedGeometry& { return b->h_desc[slot].geo; });
    int32_t count = n_work;
    std::memset(b->h_count, 0, kCounters * sizeof(int32_t));
    b->h_count[kItems] = n_work;
    for (int i = 0; i < sca::kOnChipLevels; ++i) {
        auto& list = b->epoch_chip[i];
        if (b->cfg.order == 0) std::stable_sort(list.begin(), list.end(), longer);
        b->h_count[kOnChipCount + i] = (int32_t)list.size();
        for (const auto& w : list) b->h_order[count++] = items[(size_t)w.second].slot;
    }
    const bool on_chip = count > n_work;
    if (hipMemcpyAsync(b->d_desc, b->h_desc, sizeof(sca::BatchDesc) * (size_t)(hi + 1), hipMemcpyHostToDevice,
                       b->stream) != hipSuccess ||
        hipMemcpyAsync(b->d_order, b->h_order, sizeof(int32_t) * (size_t)count, hipMemcpyHostToDevice, b->stream) !=
            hipSuccess ||
        hipMemcpyAsync(b->d_counters, b->h_count, kCounters * sizeof(int32_t), hipMemcpyHostToDevice, b->stream) !=
            hipSuccess ||
        hipEventRecord(b->staged, b->stream) != hipSuccess)
        return bfail(b);
    b->staged_pending = true;
    if (on_chip) {
        const sca::OnChipLaunch L{b->d_desc,
                                  b->d_order + n_work,
                                  b->d_counters + kOnChipCount,
                                  b->d_counters + kOnChipQueue,
                                  teams ? b->d_team : nullptr,
                                  b->d_err,
                                  b->d_sync,
                                  teams ? grid : 0};
        if (sca::launch_onchip(L, b->cu_grid, teams, b->stream) != hipSuccess) return bfail(b);
    }
    if (teams) {
        // Behind teams the persistent kernel takes the list that became of them, in a
        // launch of this epoch's own.  The list for teams that did not form is
        // made here, while the others run, and read where the host wrote it, if at
        // all: on the device it cost the epochs that need none of it some 15 us.
        // Splits use half of the workgroups at most, as something else holds others.
        prepare_launch(b);
        b->apart_at ^= 1;
        int32_t* const order = apart_order(b);
        sca::BlockedGeometry* const geometry = apart_geometry(b);
        sca::BatchLaunch L = b->launch;
        L.decision = sca::onchip_decision(b->d_team);
        L.apart_items = list_work(apart_work, apart_total, b->resident / 2, order,
                                  [geometry](int32_t slot) -> sca::BlockedGeometry& { return geometry[slot]; });
        L.apart_order = order;
        L.apart_geometry = geometry;
        L.apart = batch_apart(b);
        if (sca::launch_ensemble(L, b->cfg.block_threads, b->cfg.words_per_lane, grid, b->stream) != hipSuccess)
            return bfail(b);
    } else if (n_work > 0) {
        if (!b->exec && capture_epoch_graph(b) != hipSuccess) return bfail(b);
        if (hipGraphLaunch(b->exec, b->stream) != hipSuccess) return bfail(b);
    }
    if ((n_split > 0 || teams) && !b->err_pending) {
        if (hipMemcpyAsync(b->h_err, b->d_err, sizeof(int32_t), hipMemcpyDeviceToHost, b->stream) != hipSuccess ||
            hipEventRecord(b->err_copied, b->stream) != hipSuccess)
            return bfail(b);
        b->err_pending = true;
    }
    for (const EpochItem& it : items) b->slots[(size_t)it.slot].t += it.run;
    return SCA_OK;
}

}  // namespace

extern "C" {

int sca_batch_run(sca_batch* b, int64_t mcs_epoch, int32_t* active_out)
{
    if (!b || mcs_epoch < 0) return SCA_EINVAL;
    try {
        return batch_epoch(b, [mcs_epoch](const SlotHost&) { return mcs_epoch; }, active_out);
    } catch (const std::bad_alloc&) {  // of its lists, ahead of every launch
        return SCA_ENOMEM;
    }
}

int sca_batch_run_work(sca_batch* b, int64_t site_updates, int32_t* active_out)
{
    if (!b || site_updates <= 0) return SCA_EINVAL;
    try {
        return batch_epoch(
            b,
            [site_updates](const SlotHost& s) {
                const int64_t q = site_updates / (s.req.X * s.req.Y);
                return q > 0 ? q : (int64_t)1;
            },
            active_out);
    } catch (const std::bad_alloc&) {
        return SCA_ENOMEM;
    }
}

int sca_batch_slot(const sca_batch* b, int32_t slot, sca_slot_info* out)
{
    if (!b || !out || slot < 0 || slot >= b->max_slots || !b->slots[(size_t)slot].used) return SCA_EINVAL;
    const SlotHost& s = b->slots[(size_t)slot];
    out->X = s.req.X;
    out->Y = s.req.Y;
    out->t = s.t;
    out->n_mcs = s.req.n_mcs;
    out->seed = s.req.seed;
    out->slopes_dev = s.desc.S;
    out->h0_dev = s.desc.h0;
    return SCA_OK;
}

int sca_batch_roughness(sca_batch* b, int32_t slot, int64_t out3[3], double* w2)
{
    if (!b || !out3 || slot < 0 || slot >= b->max_slots || !b->slots[(size_t)slot].used) return SCA_EINVAL;
    if (b->failed) return SCA_ESTATE;
    DeviceGuard dg(b->device);
    if (!dg.ok) return bfail(b);
    const SlotHost& s = b->slots[(size_t)slot];
    // d_err comes with the sums: a barrier that gave up in an earlier launch shows there
    int64_t err = 0;
    const int rc = moments_of(s.desc.S, s.desc.h0, s.req.X, s.req.Y, s.W, s.nb, b->d_ws, b->results, b->stream, out3, w2,
                              b->d_err, &err);
    if (rc == SCA_EDEVICE || err) return bfail(b);
    return rc;
}

int sca_batch_collect(sca_batch* b, const int32_t* slots, int32_t n, sca_collected* out)
{
    if (!b || n < 0 || (n > 0 && (!slots || !out))) return SCA_EINVAL;
    for (int32_t i = 0; i < n; ++i)
        if (slots[i] < 0 || slots[i] >= b->max_slots || !b->slots[(size_t)slots[i]].used) return SCA_EINVAL;
    if (b->failed) return SCA_ESTATE;
    DeviceGuard dg(b->device);
    if (!dg.ok) return bfail(b);
    sca::MomentsItem* const items = collect_items(b);
    for (int32_t i0 = 0; i0 < n; i0 += kCollect) {
        const int32_t m = std::min(n - i0, kCollect);
        int32_t n_items = 0;
        for (int32_t i = 0; i < m; ++i) {
            const SlotHost& s = b->slots[(size_t)slots[i0 + i]];
            int64_t* const res = b->results + 8 * i;
            if (sca::moments_in_one_block(s.req.Y, s.W))
                items[n_items++] = sca::MomentsItem{s.desc.S, s.desc.h0, res, (int32_t)s.req.Y, s.W, s.nb};
            else if (sca::launch_moments(s.desc.S, s.desc.h0, nullptr, nullptr, s.req.X, s.req.Y, s.W, s.nb, b->d_ws, res,
                                         b->d_err, b->stream) != hipSuccess)
                return bfail(b);
        }
        if (sca::launch_moments_many(items, n_items, b->d_err, b->stream) != hipSuccess ||
            hipStreamSynchronize(b->stream) != hipSuccess)
            return bfail(b);
        for (int32_t i = 0; i < m; ++i) {
            const SlotHost& s = b->slots[(size_t)slots[i0 + i]];
            int64_t r[7];
            for (int k = 0; k < 7; ++k) r[k] = reinterpret_cast<const volatile int64_t*>(b->results)[8 * i + k];
            if (r[6]) return bfail(b);
            sca_collected& o = out[i0 + i];
            o.status = moments_from(r, s.req.X, s.req.Y, o.moments, &o.w2);
            o.h0 = r[4];
        }
    }
    return SCA_OK;
}

int sca_debug_batch_teams(const sca_batch* b)
{
    if (!b) return SCA_EINVAL;
    return b->cu_grid > 0 && !b->no_teams && b->team_pause == 0 &&
           *const_cast<const volatile int32_t*>(batch_apart(b)) == 0;
}

int sca_batch_release(sca_batch* b, int32_t slot)
{
    if (!b || slot < 0 || slot >= b->max_slots || !b->slots[(size_t)slot].used) return SCA_EINVAL;
    SlotHost& s = b->slots[(size_t)slot];
    b->alloc.release(s.offset, s.bytes);
    s = SlotHost{};
    b->free_slots.push_back(slot);
    return SCA_OK;
}

void sca_batch_destroy(sca_batch* b)
{
    if (!b) return;
    {
        DeviceGuard dg(b->device);
        (void)hipStreamSynchronize(b->stream);
        batch_free(b);
    }
}

}  // extern "C"
