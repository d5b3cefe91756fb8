// onchip.hip -- realizations of an ensemble that stay in the registers of one
// or a few compute units for a whole epoch.
//
// A workgroup of 1024 threads holds up to 8192 words per sublattice (eight
// rows of one word column per thread, tile.hpp), which is a 1024 x 1024
// lattice; larger ones spread over a team of 2, 4 or 8 workgroups, each with
// its share of consecutive rows.  State moves through memory once per epoch
// instead of once per pass, and nothing is computed twice: after each
// half-step the workgroups of a team hand their neighbours the one row of
// y-slopes that both sides update in turn.
//
// That hand-over is a message in device memory without fences: a word goes as
// two 64-bit stores, each half of it beside the 32-bit number of the message,
// and the receiver polls until both numbers are the awaited one.  Two slots per
// sender and direction suffice: a workgroup sends message k only after it has
// taken its neighbour's message k-1, which that neighbour sent after taking
// message k-2 from the slot that k overwrites.  Between two realizations a
// message that carries the first values plays the same part, and each size of
// team has slots of its own, since its neighbours are others.  The two rows in
// question come first in a half-step (a few microseconds), so that messages
// travel while the other rows are updated.
//
// Teams are fixed groups of workgroups, eight, then four, two and one:
// all teams of eight work through the list of realizations for eight
// workgroups, longest first, then each half of them goes on with the list for
// four, and so on.  The first workgroup of a team takes the next realization
// and posts it to the others.  A wait is therefore for workgroups in the same
// list of the same team, in lockstep through their messages; only a launch that
// shares the device with others waits longer, for its own workgroups to be
// started.  Every wait gives up after two minutes, sets *err and waits no more.
//
// Bound by vector issue: p = 1/2, 3/4 and 15/16 take some 50, 70 and 110
// instructions per word and half-step and run at 3.7e13, 2.6e13 and 1.8e13 site
// updates/s with 256 lattices of 1024^2 or 64 of 2048^2.  The 4096 realizations
// of 2^6 to 2^11 squared, 100 to 10^4 MCS, took 0.62 s in blocked passes
// through memory and take 0.36 s; a 2048^2 lattice alone at p = 1/2 takes 3.7 us
// per MCS on a team of eight, whose half-steps wait for messages.  A workgroup
// per CU: eight rows per thread fill the 128 registers that 1024 threads leave.
#include "sca_internal.hpp"
#include "tile.hpp"

namespace sca {
namespace {

constexpr int kThreads = kOnChipThreads;
constexpr int kStride = kThreads + 64;  // LDS words per sublattice: one per thread, then the row behind the last
constexpr int kLevels = 4;              // teams of 8, 4, 2 and 1 workgroups
constexpr int kMailSlots = 8;           // posts of a team; a member lags at most half a team behind the first
constexpr int kMessage = 128;           // 64-bit words per message: two for each of 64 lanes
constexpr int kSlots = 4 * kMessage;    // a workgroup's messages in one level: two directions, two slots each
constexpr uint64_t kPatience = 120ull * 100000000ull;  // ticks of the 100 MHz clock

__device__ __forceinline__ void post(uint64_t* p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t peek(const uint64_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
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
        if (late) __hip_atomic_fetch_or(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        broken = late || __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
        return !broken;
    }
};

// The ends of a workgroup's rows within its team.
struct TeamEdge {
    bool on;                      // the team has more than one workgroup (scalar)
    bool first_wave, last_wave;   // the wave holds the first / last row group (scalars)
    bool first, last;             // this lane does
    int gl;                       // this lane's word of the row
    uint64_t *to_prev, *to_next;  // messages (slot 0 of each; scalars)
    const uint64_t *from_prev, *from_next;
    uint32_t tag;                 // the message that this half-step takes; it gives the next
    bool more;                    // another half-step follows (scalar)
    Patience* patience;

    __device__ __forceinline__ void send(uint64_t* dst, bool lane_on, uint64_t v, uint32_t number) const
    {
        uint64_t* const p = dst + (number & 1u) * kMessage + 2 * gl;
        if (lane_on) {
            post(p, ((uint64_t)number << 32) | (uint32_t)v);
            post(p + 1, ((uint64_t)number << 32) | (v >> 32));
        }
    }
    __device__ __forceinline__ uint64_t receive(const uint64_t* src, bool lane_on, uint64_t v) const
    {
        const uint64_t* const p = src + (tag & 1u) * kMessage + 2 * gl;
        uint64_t lo = 0, hi = 0;
        patience->begin();
        do {
            bool there = true;
            if (lane_on) {
                lo = peek(p);
                hi = peek(p + 1);
                there = (uint32_t)(lo >> 32) == tag && (uint32_t)(hi >> 32) == tag;
            }
            if (__all(there)) break;
        } while (patience->wait());
        return lane_on ? (lo & 0xffffffffull) | (hi << 32) : v;
    }
    __device__ __forceinline__ void take(uint64_t (&B)[1], uint64_t (&Cn)[1])
    {
        if (!on) return;
        if (first_wave) B[0] = receive(from_prev, first, B[0]);
        if (last_wave) Cn[0] = receive(from_next, last, Cn[0]);
    }
    __device__ __forceinline__ void give_first(const uint64_t (&B)[1])
    {
        if (on && first_wave && more) send(to_prev, first, B[0], tag + 1u);
    }
    __device__ __forceinline__ void give_last(const uint64_t (&Cn)[1])
    {
        if (on && last_wave && more) send(to_next, last, Cn[0], tag + 1u);
    }
};

// The epoch of one realization, N rows per thread, in a team of `parts`
// workgroups of which this is `member`.  tag: the last message number used.
template <int N, bool HASQ, Draws DR>
__device__ __forceinline__ void run_item(const BatchDesc& d, uint64_t* xch, uint64_t* ly, int parts, int member,
                                         uint32_t tag, Patience& patience)
{
    SweepArgs a{};
    a.W = d.W;
    a.nb = d.nb;
    a.t = d.t;
    a.k0 = d.k0;
    a.k1 = d.k1;
    a.dig_p = d.dig_p;
    a.dig_q = d.dig_q;
    a.ndraw = d.ndraw;
    a.all_p = d.all_p;
    a.all_q = d.all_q;

    const int G = d.W, lg = __builtin_ctz((unsigned)G);
    const int R = d.Y / parts, groups = R / N;
    const int tid = (int)threadIdx.x, grp = tid >> lg, gl = tid & (G - 1);
    const bool active = grp < groups;
    const int w0 = __builtin_amdgcn_readfirstlane(tid) >> lg, w1 = (__builtin_amdgcn_readfirstlane(tid) + 63) >> lg;
    const int64_t P = d.plane;
    const int ymask = d.Y - 1;
    uint64_t* const S = d.S;

    TileThread<-1, N, 1, XiMode::Mask, HASQ, DR> th;
    th.rl = RowLanes{G, d.nb, gl == 0, gl == G - 1, (tid & 32) != 0};
    th.own = tid;
    th.nxt = !active ? tid : (grp + 1 < groups ? tid + G : (parts > 1 ? kThreads + gl : gl));
    th.stride = kStride;
    th.kept = ly + 2 * kStride + tid;
    th.lifts = 0;
    const int y0 = member * R + grp * N;
    th.W = (uint32_t)G;
    th.g0 = (uint32_t)y0 * th.W + (uint32_t)gl;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (i % 2 == 0) th.org[i / 2] = active && y0 + i == 0 && gl == 0;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            th.x[i][p][0] = active ? S[(int64_t)p * P + th.g(i)] : 0ull;
            th.y[i][p][0] = active ? S[(int64_t)(2 + p) * P + th.g(i)] : 0ull;
        }
    }
    const bool last = active && grp == groups - 1;
    const int64_t behind = (int64_t)((y0 + N) & ymask) * G + gl;  // the row behind the last one
    uint64_t yb[2] = {0, 0};
    if (last && parts > 1)
        for (int p = 0; p < 2; ++p) yb[p] = S[(int64_t)(2 + p) * P + behind];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        ly[p * kStride + tid] = th.y[0][p][0];
        if (last && parts > 1) ly[p * kStride + kThreads + gl] = yb[p];
    }

    TeamEdge e;
    e.on = parts > 1;
    e.first_wave = w0 == 0;
    e.last_wave = w0 <= groups - 1 && groups - 1 <= w1;
    e.first = grp == 0;
    e.last = last;
    const int b0 = (int)blockIdx.x - member;  // the team's first workgroup
    const int bp = b0 + (member + parts - 1) % parts, bn = b0 + (member + 1) % parts;
    uint64_t* const own = xch + (int64_t)blockIdx.x * kSlots;
    e.gl = gl;
    e.to_prev = own;
    e.to_next = own + 2 * kMessage;
    e.from_prev = xch + (int64_t)bp * kSlots + 2 * kMessage;
    e.from_next = xch + (int64_t)bn * kSlots;
    e.patience = &patience;
    e.tag = tag + 1u;
    if (e.on) {  // the values that the first half-step takes
        if (e.first_wave) e.send(e.to_prev, e.first, th.y[0][1][0], e.tag);
        if (e.last_wave) e.send(e.to_next, e.last, yb[0], e.tag);
    }

    const bool idle = w0 >= groups;
    for (uint32_t m = 0; m < d.n_run; ++m) {
        e.more = true;
        th.template halfstep<0>(a, ly, 0, R - 1, idle, e);
        ++e.tag;
        e.more = m + 1 < d.n_run;
        th.template halfstep<1>(a, ly, 0, R - 1, idle, e);
        ++e.tag;
        ++a.t;
    }
    __syncthreads();
    if (!active) return;
#pragma unroll
    for (int p = 0; p < 2; ++p) th.y[0][p][0] = ly[p * kStride + tid];
#pragma unroll
    for (int i = 0; i < N; ++i) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            S[(int64_t)p * P + th.g(i)] = th.x[i][p][0];
            // after an odd half-step the even y-slopes of a workgroup's first row
            // are with the team's workgroup before it
            if (i > 0 || p > 0 || parts == 1 || grp > 0) S[(int64_t)(2 + p) * P + th.g(i)] = th.y[i][p][0];
        }
    }
    if (last && parts > 1) S[2 * P + behind] = ly[kThreads + gl];
    if (th.lifts != 0) atomicAdd((unsigned long long*)d.h0, (unsigned long long)(2 * (int64_t)th.lifts));
}

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

template <int N>
__device__ __forceinline__ void run_rows(const BatchDesc& d, uint64_t* xch, uint64_t* ly, int parts, int member,
                                         uint32_t tag, Patience& patience)
{
    const bool odd = (d.ndraw & 1) != 0;
    if (d.has_q) {
        if (odd) run_item<N, true, Draws::OddTail>(d, xch, ly, parts, member, tag, patience);
        else run_item<N, true, Draws::Even>(d, xch, ly, parts, member, tag, patience);
    } else {
        if (odd) run_item<N, false, Draws::OddTail>(d, xch, ly, parts, member, tag, patience);
        else run_item<N, false, Draws::Even>(d, xch, ly, parts, member, tag, patience);
    }
}

__global__ __launch_bounds__(kThreads) void onchip_kernel(OnChipLaunch L)
{
    // the y-slopes that change hands, then the kept draws of eight rows per thread
    __shared__ uint64_t ly[2 * kStride + 8 * kThreads];
    __shared__ int32_t s_item;
    Patience patience{L.err};
    uint32_t tag = 0;
    int32_t first = 0;
    for (int level = 0; level < kLevels; ++level) {
        const int parts = 8 >> level;
        const int32_t count = L.count[level];
        const int team = (int)blockIdx.x / parts, member = (int)blockIdx.x % parts;
        const bool whole_team = (team + 1) * parts <= (int)gridDim.x;
        uint64_t* const xch = L.xch + (int64_t)level * gridDim.x * kSlots;
        uint64_t* const mail = L.mail + ((int64_t)level * gridDim.x + team) * kMailSlots;
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
            switch (d.bands) {
            case 2: run_rows<2>(d, xch, ly, parts, member, tag, patience); break;
            case 4: run_rows<4>(d, xch, ly, parts, member, tag, patience); break;
            default: run_rows<8>(d, xch, ly, parts, member, tag, patience); break;
            }
            tag += 2u * d.n_run;
        }
        first += count;
    }
}

// Zeroes the posts and messages of the last launch.
__global__ __launch_bounds__(256) void onchip_reset_kernel(uint64_t* p, int64_t n)
{
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256) p[k] = 0;
}

}  // namespace

int64_t onchip_mail_words(int grid) { return (int64_t)kLevels * grid * kMailSlots; }
int64_t onchip_message_words(int grid) { return (int64_t)(kLevels - 1) * grid * kSlots; }

hipError_t launch_onchip(const OnChipLaunch& L, int grid, bool teams, hipStream_t stream)
{
    if (teams) {  // L.xch follows L.mail
        hipLaunchKernelGGL(onchip_reset_kernel, dim3(256), dim3(256), 0, stream, L.mail,
                           onchip_mail_words(grid) + onchip_message_words(grid));
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
