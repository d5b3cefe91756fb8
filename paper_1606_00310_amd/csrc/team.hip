// team.hip -- one lattice of 2^25 to 2^28 sites in the registers of the whole
// chip: a team of workgroups, one per compute unit (team.hpp), that advances any
// number of MCS in one launch and in place.
//
// Lattices of this size are too small for the row sweeps' tall bands and too
// large for the tiles: bands of 16 to 32 rows compute every row 1.25 to 1.5
// times, and the state passes through memory every few MCS.  Here it does so
// once per call.  Bound by vector issue with eight words per thread, by the
// 1.25 us of a message per half-step with two.  (With eight words 2 to 19 registers
// of the 128 that 1024 threads leave go to scratch.)  us for 64 MCS with the sweeps or
// tiles, and as a team:
//                    p = 1/2      3/4, 1/4      15/16          p = 1
//   2^14 x 2^14    941 -> 426   1355 -> 642   1678 -> 846   379 -> 224
//   2^13 x 2^15    902 -> 492   1211 -> 720   1547 -> 949   451 -> 293
//   2^12 x 2^16    791 -> 539   1017 -> 772   1354 -> 990
// A launch without MCS would take about 33 us at 2^28 sites: 27 us for the state's
// way in and out, the rest until the team has formed.
//
// All workgroups have to run at the same time for that (team.hpp).  Apart, they
// take passes over bands of rows from a common list, in an order in which each
// depends on earlier entries only: any number of workgroups, one after another if
// need be, completes them.  The host learns of it, and that lattice's next 256
// steps go without a team.
#include <cstdio>

#include "sca_internal.hpp"
#include "team.hpp"

namespace sca {
namespace {

// Control words ahead of the messages, each on a line of its own.
enum Control { kTicket = kFormationWords, kDone = kTicket + 32, kControl = kDone + 2 * kTeamMaxParts };

// Thread 0, once: the count of entries taken starts from none.
__device__ __forceinline__ void begin_tickets(const TeamLaunch& L)
{
    uint64_t v = peek(L.ctl + kTicket);
    while (!team_counts(v, L.epoch))
        if (__hip_atomic_compare_exchange_strong(L.ctl + kTicket, &v, team_count(L.epoch, 0), __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            break;
}

// Thread 0: the next entry of the list.  (An addition: with a compare and exchange
// 255 workgroups that ask at once wait 0.3 to 0.5 ms for each other.)
__device__ __forceinline__ uint32_t take_ticket(const TeamLaunch& L)
{
    return team_counted(
        __hip_atomic_fetch_add(L.ctl + kTicket, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), L.epoch);
}

// The launch's MCS as passes over bands of rows, out of place between the lattice
// and the pass buffer: a tile of as many rows as the threads hold, half of them
// the band and the rest its halo, which allows rows / 8 MCS per pass.  Entry k is
// pass k / bands of band k % bands, and pass j of band c needs pass j - 1 of the
// bands c-1, c and c+1: what it reads, and what still read the rows that it writes.
// The passes are even in number, so that the last one writes the lattice.
// One thread per workgroup makes its writes visible and sees the others'; in every
// wave the fences, each of the XCD's whole L2, would wait for each other.  64 MCS
// beside a kernel that holds a compute unit, without the wait for the team to form:
// 2^14 x 2^14 sites at p = 1/2 0.95 ms, as in the row sweeps that the step takes
// without teams (69 ms half-step by half-step in memory, with fences in every wave);
// 2^12 x 2^16 1.1 ms (69 ms).
template <int G, int N, int I, bool HASQ, Draws DR>
__device__ __forceinline__ void run_apart(const TeamLaunch& L, uint64_t* ly, uint32_t* s_entry, Patience& patience)
{
    SweepArgs a = L.a;
    const int lanes = I > 1 ? 64 : a.W, lg = __builtin_ctz((unsigned)lanes);  // of a row
    const int groups = kThreads >> lg, rows = groups * N, band = rows / 2, halo = rows / 4;
    const uint32_t bands = (uint32_t)(a.Y / band), most = (uint32_t)halo / 2;
    const uint32_t n = (uint32_t)L.n, passes = 2u * ((n + 2u * most - 1u) / (2u * most));
    const int tid = (int)threadIdx.x, grp = tid >> lg, gl = tid & (lanes - 1), r0 = grp * N;
    const int w0 = __builtin_amdgcn_readfirstlane(tid);
    const int wlo = (w0 >> lg) * N, whi = ((w0 + 63) >> lg) * N + N - 1;  // the wave's rows
    const int64_t P = a.plane;

    TileThread<G, N, I, XiMode::Mask, HASQ, DR, (N * I >= 8)> th;
    th.rl = RowLanes{lanes, a.nb, gl == 0, gl == lanes - 1, (tid & 32) != 0};
    th.own = tid;
    th.nxt = grp + 1 < groups ? tid + lanes : gl;
    th.stride = kStride;
    th.kept = ly + 2 * I * kStride + tid;
    th.W = (uint32_t)a.W;
    NoEdge edge;
    if (tid == 0) begin_tickets(L);
    for (;;) {
        __syncthreads();
        if (tid == 0) *s_entry = take_ticket(L);
        __syncthreads();
        const uint32_t k = __builtin_amdgcn_readfirstlane(*s_entry);
        if (k >= passes * bands) break;
        const uint32_t j = k / bands, c = k % bands;
        if (tid == 0 && j > 0) {
            for (uint32_t d = bands - 1; d <= bands + 1; ++d) {
                patience.begin();
                while (team_counted(peek(L.ctl + kDone + (c + d) % bands), L.epoch) < j && patience.wait()) {
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
        const uint32_t m0 = n * j / passes, m1 = n * (j + 1) / passes;
        const uint64_t* const src = (j & 1u) ? L.alt : a.S;
        uint64_t* const dst = (j & 1u) ? a.S : L.alt;
        const int y0 = ((int)c * band - halo + r0) & (a.Y - 1);
        th.g0 = (uint32_t)y0 * th.W + (uint32_t)gl;
        th.lifts = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if (i % 2 == 0) th.org[i / 2] = y0 + i == 0 && gl == 0 && r0 + i >= halo && r0 + i < halo + band;
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int q = 0; q < I; ++q) {
                    const int64_t w = (int64_t)th.g(i) + 64 * q;
                    th.x[i][p][q] = src[(int64_t)p * P + w];
                    th.y[i][p][q] = src[(int64_t)(2 + p) * P + w];
                }
        }
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int q = 0; q < I; ++q) ly[(p * I + q) * kStride + tid] = th.y[0][p][q];
        a.t = L.a.t + m0;
        int lo = halo - 2 * (int)(m1 - m0), hi = halo + band + 2 * (int)(m1 - m0) - 2;
        for (uint32_t m = m0; m < m1; ++m, ++a.t) {
            th.template halfstep<0>(a, ly, lo, hi, whi < lo || wlo > hi, edge);
            ++lo;
            --hi;
            th.template halfstep<1>(a, ly, lo, hi, whi < lo || wlo > hi, edge);
            ++lo;
            --hi;
        }
        __syncthreads();
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int q = 0; q < I; ++q) th.y[0][p][q] = ly[(p * I + q) * kStride + tid];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if (r0 + i < halo || r0 + i >= halo + band) continue;
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int q = 0; q < I; ++q) {
                    const int64_t w = (int64_t)th.g(i) + 64 * q;
                    dst[(int64_t)p * P + w] = th.x[i][p][q];
                    dst[(int64_t)(2 + p) * P + w] = th.y[i][p][q];
                }
        }
        if (th.lifts != 0) atomicAdd((unsigned long long*)a.h0, (unsigned long long)(2 * (int64_t)th.lifts));
        __syncthreads();
        if (tid == 0) __hip_atomic_store(L.ctl + kDone + c, team_count(L.epoch, j + 1u), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
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
    run_apart<G, N, I, HASQ, DR>(L, ly, &s_word, patience);
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
