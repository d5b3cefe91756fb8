// team.hip -- one lattice of 2^25 to 2^28 sites in the registers of the whole
// chip: a team of workgroups, one per compute unit (team.hpp), that advances any
// number of MCS in one launch and in place.
//
// Lattices of this size are too small for the row sweeps' tall bands and too
// large for the tiles: bands of 16 to 32 rows compute every row 1.25 to 1.5
// times, and the state passes through memory every few MCS.  Here it does so
// once per call.  Bound by vector issue with eight words per thread, by the
// 1.25 us of a message per half-step with two.  us for 64 MCS with the sweeps or
// tiles, and as a team:
//                    p = 1/2      3/4, 1/4      15/16          p = 1
//   2^14 x 2^14    941 -> 426   1355 -> 642   1678 -> 846   379 -> 224
//   2^13 x 2^15    902 -> 492   1211 -> 720   1547 -> 949   451 -> 293
//   2^12 x 2^16    791 -> 539   1017 -> 772   1354 -> 990
// A launch without MCS would take about 33 us at 2^28 sites: 27 us for the state's
// way in and out, the rest until the team has formed.
//
// All workgroups have to run at the same time for that (team.hpp).  Apart, they
// take half-steps of bands of rows in memory from a common list, in an order in
// which each depends on earlier entries only: any number of workgroups, one after
// another if need be, completes them.  The host learns of it and launches no more
// teams for that lattice.
#include <cstdio>

#include "sca_internal.hpp"
#include "team.hpp"

namespace sca {
namespace {

// Control words ahead of the messages, each on a line of its own.
enum Control { kTicket = kFormationWords, kDone = kTicket + 32, kControl = kDone + kTeamMaxParts };

// Thread 0: the next entry of the list.
__device__ __forceinline__ uint32_t take_ticket(const TeamLaunch& L)
{
    uint64_t v = peek(L.ctl + kTicket);
    for (;;) {
        const uint32_t k = team_counted(v, L.epoch);
        if (__hip_atomic_compare_exchange_strong(L.ctl + kTicket, &v, team_count(L.epoch, k + 1u), __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            return k;
    }
}

// The launch's MCS by half-steps in memory.  Entry k is half-step k / parts of
// band k % parts; band c needs half-step h-1 of the bands c-1, c and c+1.
template <int G, int I, bool HASQ>
__device__ void run_apart(const TeamLaunch& L, int parts, uint32_t* s_entry, Patience& patience)
{
    SweepArgs a = L.a;
    const int R = a.Y / parts;
    const uint32_t total = 2u * (uint32_t)L.n * (uint32_t)parts;
    const int tid = (int)threadIdx.x, lane = tid & 63, step = kThreads / G;
    for (;;) {
        __syncthreads();
        if (tid == 0) *s_entry = take_ticket(L);
        __syncthreads();
        const uint32_t k = __builtin_amdgcn_readfirstlane(*s_entry);
        if (k >= total) break;
        const uint32_t h = k / (uint32_t)parts;
        const int c = (int)(k % (uint32_t)parts);
        if (tid == 0 && h > 0)
            for (int d = parts - 1; d <= parts + 1; ++d) {
                patience.begin();
                while (team_counted(peek(L.ctl + kDone + (c + d) % parts), L.epoch) < h && patience.wait()) {
                }
            }
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        a.t = L.a.t + h / 2;
        a.parity = (int)(h & 1u);
        for (int r0 = 0; r0 < R; r0 += step) {
            const int r = r0 + tid / G;
            halfstep_rows<G, I, XiMode::Mask, HASQ>(a, a.S, r < R ? (int64_t)c * R + r : (int64_t)a.Y, lane);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __syncthreads();
        if (tid == 0) post(L.ctl + kDone + c, team_count(L.epoch, h + 1u));
    }
}

template <int G, int N, int I, bool HASQ, Draws DR>
__global__ __launch_bounds__(kThreads) void team_kernel(TeamLaunch L)
{
    __shared__ uint64_t ly[kTeamLds<N, I>];
    __shared__ uint32_t s_word;
    const int parts = (int)gridDim.x;
    if (threadIdx.x == 0) arrive(L.ctl, L.epoch, (uint64_t)parts);
    Patience patience{L.err};
    const bool done = team_run<G, N, I, HASQ, DR>(
        L.a, L.a.S, (uint32_t)L.n, L.ctl + kControl, ly, parts, (int)blockIdx.x, L.tag, patience, [&] {
            if (threadIdx.x == 0) s_word = formed(L.ctl, L.epoch) ? 1u : 0u;
            __syncthreads();
            return __builtin_amdgcn_readfirstlane(s_word) != 0u;
        });
    if (done) return;
    if (threadIdx.x == 0) __hip_atomic_store(L.apart, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if constexpr (I == 2) run_apart<64, 2, HASQ>(L, parts, &s_word, patience);
    else if (L.a.W == 64) run_apart<64, 1, HASQ>(L, parts, &s_word, patience);
    else if (L.a.W == 32) run_apart<32, 1, HASQ>(L, parts, &s_word, patience);
    else run_apart<16, 1, HASQ>(L, parts, &s_word, patience);
}

__global__ __launch_bounds__(256) void team_clear_kernel(uint64_t* p, int64_t n)
{
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256) p[k] = 0;
}

template <int G, int N, int I, class F>
hipError_t with_mode(const SweepArgs& a, bool has_q, F&& f)
{
    if (a.ndraw & 1)
        return has_q ? f(team_kernel<G, N, I, true, Draws::OddTail>) : f(team_kernel<G, N, I, false, Draws::OddTail>);
    return has_q ? f(team_kernel<G, N, I, true, Draws::Even>) : f(team_kernel<G, N, I, false, Draws::Even>);
}

template <class F>
hipError_t with_team_kernel(const SweepArgs& a, bool has_q, int rows, F&& f)
{
    if (a.W == 128) {
        switch (rows) {
        case 2: return with_mode<64, 2, 2>(a, has_q, f);
        case 4: return with_mode<64, 4, 2>(a, has_q, f);
        default: return hipErrorInvalidValue;
        }
    }
    switch (rows) {
    case 2: return with_mode<-1, 2, 1>(a, has_q, f);
    case 4: return with_mode<-1, 4, 1>(a, has_q, f);
    case 8: return with_mode<-1, 8, 1>(a, has_q, f);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

int64_t team_words(int32_t W, int parts) { return kControl + (int64_t)parts * (W > 64 ? kSlots<2> : kSlots<1>); }

hipError_t launch_team_clear(uint64_t* ctl, int32_t W, int parts, hipStream_t stream)
{
    hipLaunchKernelGGL(team_clear_kernel, dim3(256), dim3(256), 0, stream, ctl, team_words(W, parts));
    return hipGetLastError();
}

hipError_t launch_team(const TeamLaunch& L, bool has_q, int parts, int rows, hipStream_t stream)
{
    if (team_rows(L.a.W, L.a.Y, parts) != rows || L.a.W < 16 || parts < 4 || parts > kTeamMaxParts || L.n <= 0 ||
        L.n > kTeamMaxMcs)
        return hipErrorInvalidValue;
    return with_team_kernel(L.a, has_q, rows, [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)parts), dim3(kThreads), 0, stream, L);
        return hipGetLastError();
    });
}

// The kernel launch_team runs.
void team_kernel_name(const SweepArgs& a, bool has_q, int rows, char* out, size_t n)
{
    std::snprintf(out, n, "team_kernel<%d,%d,%d,%s,%s>", a.W == 128 ? 64 : -1, rows, a.W == 128 ? 2 : 1,
                  has_q ? "true" : "false", (a.ndraw & 1) ? "OddTail" : "Even");
}

}  // namespace sca
