// team.hpp -- a lattice held in the registers of a team of workgroups for many
// MCS, shared by the ensembles (onchip.hip) and the single lattice (team.hip).
//
// A workgroup of 1024 threads holds up to 8192 words per sublattice (tile.hpp);
// a team of workgroups holds a larger lattice, each its share of consecutive
// rows.  State moves through memory once per launch, and nothing is computed
// twice: after each half-step the workgroups hand their neighbours the one row
// of y-slopes that both sides update in turn.
//
// That hand-over is a message in device memory without fences: a word goes as
// two 64-bit stores, each half of it beside the 32-bit number of the message,
// and the receiver polls until both numbers are the awaited one.  Two slots per
// sender and direction suffice: a workgroup sends message k only after it has
// taken its neighbour's message k-1, which that neighbour sent after taking
// message k-2 from the slot that k overwrites.  Before the first half-step a
// message that carries the first values plays the same part.  The two rows in
// question come first in a half-step, so that messages travel while the other
// rows are updated.  From sending to taking a message 1.25 us go by (a half-step
// of little work takes that long), as much as half a half-step of eight rows per
// thread without random words.
//
// Every wait gives up after two minutes, or when another has, and waits no more.
//
// The workgroups of a team have to run at the same time, which kernels on other
// streams can prevent for good: each XCD dispatches its share of a grid by
// itself, so two launches that start together can each hold some XCDs, and no
// team of either has all its workgroups.  So a launch forms first: the last of
// its workgroups to arrive decides to go on, or, after a quarter of a millisecond,
// one that waits decides that there will be no teams.
#pragma once

#include "sca_internal.hpp"
#include "tile.hpp"

namespace sca {
namespace {

constexpr int kThreads = kTeamThreads;
constexpr int kStride = kThreads + 64;  // LDS words per sublattice: one per thread, then the row behind the last
constexpr uint64_t kPatience = 120ull * 100000000ull;  // ticks of the 100 MHz clock

__device__ __forceinline__ void post(uint64_t* p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t peek(const uint64_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Words of a launch's formation, each on a line of its own; `epoch` numbers the
// launches since they were zero, from 1.
enum Formation { kArrivals = 0, kDecision = 16, kFormationWords = 32 };
constexpr uint64_t kFormationTime = 25000;  // ticks of the 100 MHz clock: 0.25 ms (all arrive within 0.01 ms on a free device)

// One thread: the launch's decision, 2 epoch (go on) or 2 epoch + 1 (apart), if
// there is none yet the one wanted.
__device__ __forceinline__ uint64_t decide(uint64_t* ctl, uint64_t epoch, uint64_t want)
{
    uint64_t v = peek(ctl + kDecision);
    while (v < 2 * epoch)
        if (__hip_atomic_compare_exchange_strong(ctl + kDecision, &v, want, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
            return want;
    return v;
}

// One thread of each of the launch's `parts` workgroups.
__device__ __forceinline__ void arrive(uint64_t* ctl, uint64_t epoch, uint64_t parts)
{
    const uint64_t before = __hip_atomic_fetch_add(ctl + kArrivals, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (before + 1 == epoch * parts) decide(ctl, epoch, 2 * epoch);
}

// The same thread: whether all of them run at the same time.
__device__ __forceinline__ bool formed(uint64_t* ctl, uint64_t epoch)
{
    const uint64_t since = __builtin_amdgcn_s_memrealtime();
    uint64_t v;
    while ((v = peek(ctl + kDecision)) < 2 * epoch) {
        __builtin_amdgcn_s_sleep(1);
        if (__builtin_amdgcn_s_memrealtime() - since > kFormationTime) v = decide(ctl, epoch, 2 * epoch + 1);
    }
    return v == 2 * epoch;
}

// Whether a wait should go on: false once it has lasted too long or another
// workgroup has given up.
struct Patience {
    int32_t* err;
    bool broken = false;
    uint64_t since = 0;
    uint32_t polls = 0;

    __device__ __forceinline__ void begin() { polls = 0; }
    __device__ __forceinline__ bool wait()
    {
        if (broken) return false;
        __builtin_amdgcn_s_sleep(1);
        if ((++polls & 1023u) != 0) return true;
        const uint64_t now = __builtin_amdgcn_s_memrealtime();
        if (polls == 1024u) since = now;
        const bool late = now - since > kPatience;
        if (late) __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        broken = late || __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) != 0;
        return !broken;
    }
};

// 64-bit words of a message of rows of I words per lane, and of all messages of
// one workgroup (two directions, two slots each).
template <int I>
constexpr int kMessage = I * kTeamMessage;
template <int I>
constexpr int kSlots = 4 * kMessage<I>;

// The ends of a workgroup's rows within its team.
template <int I>
struct TeamEdge {
    bool on;                      // the team has more than one workgroup (scalar)
    bool first_wave, last_wave;   // the wave holds the first / last row group (scalars)
    bool first, last;             // this lane does
    int gl;                       // this lane's first word of the row
    uint64_t *to_prev, *to_next;  // messages (slot 0 of each; scalars)
    const uint64_t *from_prev, *from_next;
    uint32_t tag;                 // the message that this half-step takes; it gives the next
    bool more;                    // another half-step follows (scalar)
    Patience* patience;

    __device__ __forceinline__ void send(uint64_t* dst, bool lane_on, const uint64_t (&v)[I], uint32_t number) const
    {
        uint64_t* const p = dst + (number & 1u) * kMessage<I> + 2 * gl;
        if (lane_on) {
#pragma unroll
            for (int k = 0; k < I; ++k) {
                post(p + 128 * k, ((uint64_t)number << 32) | (uint32_t)v[k]);
                post(p + 128 * k + 1, ((uint64_t)number << 32) | (v[k] >> 32));
            }
        }
    }
    __device__ __forceinline__ void receive(const uint64_t* src, bool lane_on, uint64_t (&v)[I]) const
    {
        const uint64_t* const p = src + (tag & 1u) * kMessage<I> + 2 * gl;
        uint64_t lo[I], hi[I];
        patience->begin();
        do {
            bool there = true;
            if (lane_on) {
#pragma unroll
                for (int k = 0; k < I; ++k) {
                    lo[k] = peek(p + 128 * k);
                    hi[k] = peek(p + 128 * k + 1);
                    there = there && (uint32_t)(lo[k] >> 32) == tag && (uint32_t)(hi[k] >> 32) == tag;
                }
            }
            if (__all(there)) break;
        } while (patience->wait());
#pragma unroll
        for (int k = 0; k < I; ++k)
            if (lane_on) v[k] = (lo[k] & 0xffffffffull) | (hi[k] << 32);
    }
    __device__ __forceinline__ void take(uint64_t (&B)[I], uint64_t (&Cn)[I])
    {
        if (!on) return;
        if (first_wave) receive(from_prev, first, B);
        if (last_wave) receive(from_next, last, Cn);
    }
    __device__ __forceinline__ void give_first(const uint64_t (&B)[I])
    {
        if (on && first_wave && more) send(to_prev, first, B, tag + 1u);
    }
    __device__ __forceinline__ void give_last(const uint64_t (&Cn)[I])
    {
        if (on && last_wave && more) send(to_next, last, Cn, tag + 1u);
    }
};

// LDS words of a workgroup: the y-slopes that change hands, then, where an odd
// number of draws keeps its last one there, a word per thread and word held.
template <int N, int I>
constexpr int kTeamLds = 2 * I * kStride + (N * I >= 8 ? N * I * kThreads : 0);

// n MCS from MCS a.t on of the lattice at S (a.plane, a.W, a.Y), N rows of I
// words per lane and thread, in a team of `parts` workgroups of which this is
// `member`.  tag: the last message number that the team used; this uses 2 n.
// ready: called once the rows are in registers; false (for the whole team) ends
// the run with the lattice as it was, and team_run returns false.
template <int G, int N, int I, bool HASQ, Draws DR, class F>
__device__ __forceinline__ bool team_run(SweepArgs a, uint64_t* S, uint32_t n, uint64_t* xch, uint64_t* ly, int parts,
                                         int member, uint32_t tag, Patience& patience, F&& ready)
{
    const int lanes = I > 1 ? 64 : a.W, lg = __builtin_ctz((unsigned)lanes);  // of a row
    const int R = a.Y / parts, groups = R / N;
    const int tid = (int)threadIdx.x, grp = tid >> lg, gl = tid & (lanes - 1);
    const bool active = grp < groups;
    const int w0 = __builtin_amdgcn_readfirstlane(tid) >> lg, w1 = (__builtin_amdgcn_readfirstlane(tid) + 63) >> lg;
    const int64_t P = a.plane;

    TileThread<G, N, I, XiMode::Mask, HASQ, DR, (N * I >= 8)> th;
    th.rl = RowLanes{lanes, a.nb, gl == 0, gl == lanes - 1, (tid & 32) != 0};
    th.own = tid;
    th.nxt = !active ? tid : (grp + 1 < groups ? tid + lanes : (parts > 1 ? kThreads + gl : gl));
    th.stride = kStride;
    th.kept = ly + 2 * I * kStride + tid;
    th.lifts = 0;
    const int y0 = member * R + grp * N;
    th.W = (uint32_t)a.W;
    th.g0 = (uint32_t)y0 * th.W + (uint32_t)gl;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (i % 2 == 0) th.org[i / 2] = active && y0 + i == 0 && gl == 0;
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int k = 0; k < I; ++k) {
                const int64_t w = (int64_t)th.g(i) + 64 * k;
                th.x[i][p][k] = active ? S[(int64_t)p * P + w] : 0ull;
                th.y[i][p][k] = active ? S[(int64_t)(2 + p) * P + w] : 0ull;
            }
    }
    const bool last = active && grp == groups - 1, edge = last && parts > 1;
    const int64_t behind = (int64_t)((y0 + N) & (a.Y - 1)) * a.W + gl;  // the row behind the last one
    uint64_t yb[2][I] = {};
    if (edge)
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int k = 0; k < I; ++k) yb[p][k] = S[(int64_t)(2 + p) * P + behind + 64 * k];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int k = 0; k < I; ++k) {
            ly[(p * I + k) * kStride + tid] = th.y[0][p][k];
            if (edge) ly[(p * I + k) * kStride + kThreads + gl] = yb[p][k];
        }

    TeamEdge<I> e;
    e.on = parts > 1;
    e.first_wave = w0 == 0;
    e.last_wave = w0 <= groups - 1 && groups - 1 <= w1;
    e.first = grp == 0;
    e.last = last;
    e.gl = gl;
    const int b0 = (int)blockIdx.x - member;  // the team's first workgroup
    const int bp = b0 + (member + parts - 1) % parts, bn = b0 + (member + 1) % parts;
    e.to_prev = xch + (int64_t)blockIdx.x * kSlots<I>;
    e.to_next = e.to_prev + 2 * kMessage<I>;
    e.from_prev = xch + (int64_t)bp * kSlots<I> + 2 * kMessage<I>;
    e.from_next = xch + (int64_t)bn * kSlots<I>;
    e.patience = &patience;
    e.tag = tag + 1u;
    if (!ready()) return false;
    if (e.on) {  // the values that the first half-step takes
        if (e.first_wave) e.send(e.to_prev, e.first, th.y[0][1], e.tag);
        if (e.last_wave) e.send(e.to_next, e.last, yb[0], e.tag);
    }

    const bool idle = w0 >= groups;
    for (uint32_t m = 0; m < n; ++m) {
        e.more = true;
        th.template halfstep<0>(a, ly, 0, R - 1, idle, e);
        ++e.tag;
        e.more = m + 1 < n;
        th.template halfstep<1>(a, ly, 0, R - 1, idle, e);
        ++e.tag;
        ++a.t;
    }
    __syncthreads();
    if (!active) return true;
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int k = 0; k < I; ++k) th.y[0][p][k] = ly[(p * I + k) * kStride + tid];
#pragma unroll
    for (int i = 0; i < N; ++i) {
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int k = 0; k < I; ++k) {
                const int64_t w = (int64_t)th.g(i) + 64 * k;
                S[(int64_t)p * P + w] = th.x[i][p][k];
                // after an odd half-step the even y-slopes of a workgroup's first row
                // are with the team's workgroup before it
                if (i > 0 || p > 0 || parts == 1 || grp > 0) S[(int64_t)(2 + p) * P + w] = th.y[i][p][k];
            }
    }
    if (edge)
#pragma unroll
        for (int k = 0; k < I; ++k) S[2 * P + behind + 64 * k] = ly[k * kStride + kThreads + gl];
    if (th.lifts != 0) atomicAdd((unsigned long long*)a.h0, (unsigned long long)(2 * (int64_t)th.lifts));
    return true;
}

}  // namespace
}  // namespace sca
