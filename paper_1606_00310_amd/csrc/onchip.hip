// onchip.hip -- realizations of an ensemble that stay in the registers of one
// or a few compute units for a whole epoch.
//
// A workgroup holds a lattice of up to 1024 x 1024, larger ones spread over a
// team of 2 to 16 workgroups (team.hpp).  Each size of team has message slots
// of its own, since its neighbours are others.
//
// Teams are fixed groups of workgroups, sixteen, then eight, four, two and one:
// all teams of sixteen work through the list of realizations for sixteen
// workgroups, longest first, then each half of them goes on with the list for
// eight, and so on.  The first workgroup of a team takes the next realization
// and posts it to the others.  A wait is therefore for workgroups in the same
// list of the same team, in lockstep through their messages.  Where the launch's
// workgroups do not get to run at the same time, the realizations for teams go
// through the persistent kernel (batch.hip), which is launched behind this one with
// a second list for that case; the host learns of it, and that ensemble's next 256
// epochs go without teams.
//
// Bound by vector issue: p = 1/2, 3/4 and 15/16 take some 50, 70 and 110
// instructions per word and half-step and run at 3.7e13, 2.6e13 and 1.8e13 site
// updates/s with 256 lattices of 1024^2 or 64 of 2048^2.  The 4096 realizations
// of 2^6 to 2^11 squared, 100 to 10^4 MCS, took 0.62 s in blocked passes
// through memory and take 0.36 s; a 2048^2 lattice alone at p = 1/2 takes 2.4 us
// per MCS on a team of sixteen, whose half-steps wait for messages (3.8 us on
// eight; p = 15/16: 4.0 and 7.1 us).  A workgroup
// per CU: eight rows per thread fill the 128 registers that 1024 threads leave, and
// 67 more go to scratch in this one kernel of all twelve forms (96 bytes per lane).
#include "sca_internal.hpp"
#include "team.hpp"

namespace sca {
namespace {

constexpr int kLevels = kOnChipLevels;
constexpr int kMailSlots = 16;  // posts of a team; a member lags at most half a team behind the first

// A descriptor in scalar registers: it is the same for the whole workgroup.
__device__ __forceinline__ BatchDesc load_desc(const BatchDesc* table, int32_t slot)
{
    static_assert(sizeof(BatchDesc) % 4 == 0, "descriptor of whole dwords");
    BatchDesc d = table[slot];
    uint32_t w[sizeof(BatchDesc) / 4];
    __builtin_memcpy(w, &d, sizeof(BatchDesc));
#pragma unroll
    for (unsigned i = 0; i < sizeof(BatchDesc) / 4; ++i) w[i] = __builtin_amdgcn_readfirstlane(w[i]);
    __builtin_memcpy(&d, w, sizeof(BatchDesc));
    return d;
}

__device__ __host__ constexpr int64_t mail_words(int grid) { return (int64_t)kLevels * grid * kMailSlots; }

__device__ __forceinline__ SweepArgs sweep_args(const BatchDesc& d)
{
    SweepArgs a{};
    a.plane = d.plane;
    a.W = d.W;
    a.Y = d.Y;
    a.nb = d.nb;
    a.t = d.t;
    a.k0 = d.k0;
    a.k1 = d.k1;
    a.dig_p = d.dig_p;
    a.dig_q = d.dig_q;
    a.ndraw = d.ndraw;
    a.all_p = d.all_p;
    a.all_q = d.all_q;
    a.h0 = d.h0;
    return a;
}

// The epoch of one realization, N rows per thread.
template <int N>
__device__ __forceinline__ void run_rows(const BatchDesc& d, uint64_t* xch, uint64_t* ly, int parts, int member,
                                         uint32_t tag, Patience& patience)
{
    const SweepArgs a = sweep_args(d);
    const bool odd = (d.ndraw & 1) != 0;
    const auto ready = [] { return true; };
    if (d.has_q) {
        if (odd) team_run<-1, N, 1, true, Draws::OddTail>(a, d.S, d.n_run, xch, ly, parts, member, tag, patience, ready);
        else team_run<-1, N, 1, true, Draws::Even>(a, d.S, d.n_run, xch, ly, parts, member, tag, patience, ready);
    } else {
        if (odd) team_run<-1, N, 1, false, Draws::OddTail>(a, d.S, d.n_run, xch, ly, parts, member, tag, patience, ready);
        else team_run<-1, N, 1, false, Draws::Even>(a, d.S, d.n_run, xch, ly, parts, member, tag, patience, ready);
    }
}

__global__ __launch_bounds__(kThreads) void onchip_kernel(OnChipLaunch L)
{
    __shared__ uint64_t ly[kTeamLds<8, 1>];
    __shared__ int32_t s_item;
    Patience patience{L.err};
    uint64_t* const mails = L.team + kFormationWords;
    uint64_t* const messages = mails + mail_words((int)gridDim.x);
    bool teams = false;
    if (L.team) {
        if (threadIdx.x == 0) {
            arrive(L.team, 1, gridDim.x);
            s_item = formed(L.team, 1) ? 1 : 0;
        }
        __syncthreads();
        teams = __builtin_amdgcn_readfirstlane(s_item) != 0;
    }
    uint32_t tag = 0;
    int32_t first = 0;
    for (int level = 0; level < kLevels; ++level) {
        const int parts = kOnChipMaxParts >> level;
        const int32_t count = parts == 1 || teams ? L.count[level] : 0;
        const int team = (int)blockIdx.x / parts, member = (int)blockIdx.x % parts;
        const bool whole_team = (team + 1) * parts <= (int)gridDim.x;
        uint64_t* const xch = messages + (int64_t)level * gridDim.x * kSlots<1>;
        uint64_t* const mail = mails + ((int64_t)level * gridDim.x + team) * kMailSlots;
        for (uint32_t seq = 1; count > 0 && whole_team; ++seq) {
            __syncthreads();  // the last realization is finished with LDS
            if (threadIdx.x == 0) {
                int32_t item = count;
                if (member == 0) {
                    item = atomicAdd(L.queue + level, 1);
                    if (parts > 1) post(mail + seq % kMailSlots, ((uint64_t)seq << 32) | (uint32_t)item);
                } else {
                    patience.begin();
                    do {
                        const uint64_t v = peek(mail + seq % kMailSlots);
                        if ((uint32_t)(v >> 32) == seq) {
                            item = (int32_t)(uint32_t)v;
                            break;
                        }
                    } while (patience.wait());
                }
                s_item = item;
            }
            __syncthreads();
            const int32_t item = __builtin_amdgcn_readfirstlane(s_item);
            if (item >= count) break;
            const BatchDesc d = load_desc(L.desc, __builtin_amdgcn_readfirstlane(L.order[first + item]));
            switch (d.geo.bands) {
            case 2: run_rows<2>(d, xch, ly, parts, member, tag, patience); break;
            case 4: run_rows<4>(d, xch, ly, parts, member, tag, patience); break;
            default: run_rows<8>(d, xch, ly, parts, member, tag, patience); break;
            }
            tag += 2u * d.n_run;
        }
        first += L.count[level];
    }
}

// Zeroes the formation, posts and messages of the last launch, and the barrier
// counters of the kernel behind this one.
__global__ __launch_bounds__(256) void onchip_reset_kernel(uint64_t* p, int64_t n, int32_t* sync, int32_t n_sync)
{
    for (int32_t k = (int32_t)(blockIdx.x * 256 + threadIdx.x); k < n_sync; k += (int32_t)(gridDim.x * 256)) sync[k] = 0;
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256) p[k] = 0;
}

}  // namespace

int64_t onchip_team_words(int grid)
{
    return kFormationWords + mail_words(grid) + (int64_t)(kLevels - 1) * grid * kSlots<1>;
}

const uint64_t* onchip_decision(const uint64_t* team) { return team + kDecision; }

hipError_t launch_onchip(const OnChipLaunch& L, int grid, bool teams, hipStream_t stream)
{
    if (teams != (L.team != nullptr)) return hipErrorInvalidValue;
    if (teams) {
        hipLaunchKernelGGL(onchip_reset_kernel, dim3(256), dim3(256), 0, stream, L.team, onchip_team_words(grid),
                           L.sync, L.n_sync);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(onchip_kernel, dim3((unsigned)grid), dim3(kThreads), 0, stream, L);
    return hipGetLastError();
}

int onchip_occupancy()
{
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, onchip_kernel, kThreads, 0) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return n;
}

}  // namespace sca
