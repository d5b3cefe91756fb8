// tile.hip -- launches of the on-chip tiles (tile.hpp) for one lattice: the
// whole lattice in one workgroup, or one band per workgroup with its halo.
#include <algorithm>
#include <cstdio>

#include "sca_internal.hpp"
#include "tile.hpp"

namespace sca {
namespace {

struct TileLaunch {
    SweepArgs a;          // a.t: the first MCS
    const uint64_t* src;
    uint64_t* dst;
    int32_t rows;         // rows per tile
    int32_t band;         // of these, the rows written: tile rows halo .. halo+band-1
    int32_t halo;         // 0: the tile is the whole lattice
    int32_t n;            // MCS
    int32_t threads;      // ahead mode: threads that hold rows, whole waves
};

// Threads of a workgroup at most: with two words per lane the rows take more
// than the 128 VGPRs that 1024 threads leave each.
template <int I>
constexpr int kTileThreads = I == 1 ? 1024 : 768;

template <int G, int N, int I, XiMode MODE, bool HASQ, Draws DR>
__global__ __launch_bounds__(kTileThreads<I>) void tile_kernel(TileLaunch L)
{
    extern __shared__ uint64_t ly[];  // [sublattice][word i][thread]
    const SweepArgs& a = L.a;
    // rows / N groups of G lanes, rounded up to whole waves
    const int T = MODE == XiMode::Ahead ? L.threads : (int)blockDim.x;
    constexpr int L2G = G == 0 ? 0 : __builtin_ctz(G == 0 ? 1u : (unsigned)G);  // log2 of the lanes per row
    constexpr int GL = 1 << L2G;
    const int groups = L.rows / N;
    const int tid = (int)threadIdx.x;
    const int grp = tid >> L2G, gl = tid & (GL - 1);
    const bool active = grp < groups;

    TileThread<G, N, I, MODE, HASQ, DR> th;
    th.rl = RowLanes{GL, a.nb, gl == 0, gl == GL - 1, (tid & 32) != 0};
    // idle threads of the last wave (fewer groups than fit) keep an LDS word of
    // their own beside the tile's
    th.own = tid;
    th.nxt = !active ? tid : (grp + 1 < groups ? tid + GL : gl);
    th.stride = T;
    th.lifts = 0;
    const int r0 = grp * N;                       // first tile row of this thread
    const int y0 = (int)blockIdx.x * L.band - L.halo + r0;
    const int ymask = a.Y - 1;
    // (y0 is a multiple of N: a thread's rows do not wrap)
    th.W = (uint32_t)a.W;
    th.g0 = (uint32_t)(y0 & ymask) * th.W + (uint32_t)gl;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int y = (y0 & ymask) + i;
        if (i % 2 == 0) th.org[i / 2] = active && y == 0 && gl == 0 && r0 + i >= L.halo && r0 + i < L.halo + L.band;
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int k = 0; k < I; ++k) {
                const int64_t w = (int64_t)th.g(i) + 64 * k;
                th.x[i][p][k] = active ? L.src[(int64_t)p * a.plane + w] : 0ull;
                th.y[i][p][k] = active ? L.src[(int64_t)(2 + p) * a.plane + w] : 0ull;
            }
    }
    if constexpr (MODE == XiMode::PerSite) {
        const int used = a.nb > 8 ? 31 - __builtin_clz((unsigned)a.nb) - 3 : 0;
        th.ps = PerSiteTile{ly + 2 * T, L.rows << L2G, L2G, used, (int)blockIdx.x * L.band - L.halo, ymask, HASQ};
        th.xrow = active ? (r0 << L2G) + gl : 0;
    }
    if constexpr (MODE == XiMode::Ahead) {
        th.ahead = AheadTile{ly + 2 * T, L.rows << L2G, L2G, (int)blockIdx.x * L.band - L.halo, ymask, HASQ ? 1 : 0};
        th.xrow = active ? (r0 << L2G) + gl : 0;
        for (int w = tid; w < th.ahead.words; w += (int)blockDim.x) {
            uint64_t tail = 0;
            th.ahead.template generate<0, HASQ, DR>(a, w, tail);
            th.ahead.template generate<1, HASQ, DR>(a, w, tail);
        }
    }
    if (MODE != XiMode::Ahead || tid < T)
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int k = 0; k < I; ++k) ly[(p * I + k) * T + tid] = th.y[0][p][k];

    // tile rows of this wave, and the rows that half-step h has to get right
    const int w0 = __builtin_amdgcn_readfirstlane(tid);
    const int wlo = (w0 >> L2G) * N, whi = ((w0 + 63) >> L2G) * N + N - 1;
    int lo = L.halo > 0 ? L.halo - 2 * L.n : 0;
    int hi = L.halo > 0 ? L.halo + L.band + 2 * L.n - 2 : L.rows - 1;
    const int shrink = L.halo > 0 ? 1 : 0;
    SweepArgs ah = a;
    NoEdge edge;
    // one wave of rows orders its half-steps by itself and meets the others once
    // per MCS
    const bool alone = MODE == XiMode::Ahead && T == 64;
    if (MODE == XiMode::Ahead && w0 >= T) {
        if constexpr (MODE == XiMode::Ahead) {
            // a thread forms a word for both half-steps, or the second set of
            // waves those of the odd ones
            const int per_set = (th.ahead.words + 63) / 64 * 64;
            const bool split = T + per_set < (int)blockDim.x, second = w0 - T >= per_set;
            const int w = tid - T - (second ? per_set : 0);
            for (int m = 0; m < L.n; ++m) {
                ++ah.t;
                lo += 2 * shrink;
                hi -= 2 * shrink;
                const bool mine = w >= lo << L2G && w < (hi + 1) << L2G && m + 1 < L.n;
                uint64_t tail = 0;
                __syncthreads();
                if (mine && !second) th.ahead.template generate<0, HASQ, DR>(ah, w, tail);
                if (!alone) __syncthreads();
                if (mine && !split) th.ahead.template generate<1, HASQ, DR>(ah, w, tail);
                if (mine && second) th.ahead.template generate<1, HASQ, Draws::Any>(ah, w, tail);
            }
        }
        __syncthreads();
        return;
    }
    for (int m = 0; m < L.n; ++m) {
        th.template halfstep<0>(ah, ly, lo, hi, whi < lo || wlo > hi, edge);
        lo += shrink;
        hi -= shrink;
        th.template halfstep<1>(ah, ly, lo, hi, whi < lo || wlo > hi, edge, alone);
        lo += shrink;
        hi -= shrink;
        ++ah.t;
    }
    __syncthreads();
    if (!active) return;
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int k = 0; k < I; ++k) th.y[0][p][k] = ly[(p * I + k) * T + tid];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (r0 + i < L.halo || r0 + i >= L.halo + L.band) continue;
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int k = 0; k < I; ++k) {
                const int64_t w = (int64_t)th.g(i) + 64 * k;
                L.dst[(int64_t)p * a.plane + w] = th.x[i][p][k];
                L.dst[(int64_t)(2 + p) * a.plane + w] = th.y[i][p][k];
            }
    }
    if (th.lifts != 0) atomicAdd((unsigned long long*)a.h0, (unsigned long long)(2 * (int64_t)th.lifts));
}

template <int G, int N, int I, XiMode MODE, bool HASQ, Draws DR>
hipError_t launch(const TileLaunch& L0, hipStream_t stream)
{
    int threads = (L0.rows / N * (G == 0 ? 1 : G) + 63) / 64 * 64;
    size_t lds = 0;
    if (MODE == XiMode::PerSite) {
        // helpers for the acceptance words: a thread for each byte of the rows a
        // half-step needs on average
        const int words = L0.rows * (G == 0 ? 1 : G);
        const int bytes = (L0.rows - L0.halo) * (G == 0 ? 1 : G) * 8;
        threads = std::max(threads, std::min(1024, (bytes + 63) / 64 * 64));
        lds = (size_t)(HASQ ? 4 : 2) * words * sizeof(uint64_t);
    }
    TileLaunch L = L0;
    if (MODE == XiMode::Ahead) {
        // A thread for each word; two for rows of one wave, which do not hold up
        // the second set within an MCS, unless p and q have a single digit, whose
        // one draw serves both half-steps.
        const int words = L.rows * (G == 0 ? 1 : G);
        L.threads = threads;
        lds = (size_t)(HASQ ? 8 : 4) * words * sizeof(uint64_t);
        threads += (words + 63) / 64 * 64 * (threads == 64 && L.a.ndraw > 1 ? 2 : 1);
    }
    const int grid = L.a.Y / L.band;
    if (threads > kTileThreads<I> || L.rows % N != 0 || L.a.Y % L.band != 0 || L.rows < L.band + 2 * L.halo ||
        (L.halo == 0 ? (grid != 1 || L.rows != L.a.Y) : (L.halo % 2 != 0 || L.halo < 2 * L.n)))
        return hipErrorInvalidValue;
    lds += (size_t)2 * I * threads * sizeof(uint64_t);
    if (lds > 65536) return hipErrorInvalidValue;
    hipLaunchKernelGGL((tile_kernel<G, N, I, MODE, HASQ, DR>), dim3((unsigned)grid), dim3((unsigned)threads), lds,
                       stream, L);
    return hipGetLastError();
}

template <int G, int N, int I>
hipError_t launch_mode(const TileLaunch& L, XiMode mode, bool has_q, hipStream_t stream)
{
    if (mode == XiMode::PerSite) {
        if constexpr (N == 2 && G < 64)
            return has_q ? launch<G, N, I, XiMode::PerSite, true, Draws::Any>(L, stream)
                         : launch<G, N, I, XiMode::PerSite, false, Draws::Any>(L, stream);
    }
    if (mode == XiMode::Ahead) {
        if constexpr (N == 2) {
            if (L.a.ndraw & 1)
                return has_q ? launch<G, N, I, XiMode::Ahead, true, Draws::OddTail>(L, stream)
                             : launch<G, N, I, XiMode::Ahead, false, Draws::OddTail>(L, stream);
            if (L.a.ndraw > 0)
                return has_q ? launch<G, N, I, XiMode::Ahead, true, Draws::Even>(L, stream)
                             : launch<G, N, I, XiMode::Ahead, false, Draws::Even>(L, stream);
        }
    }
    if (mode != XiMode::Mask) return hipErrorInvalidValue;
    if (L.a.ndraw == 0)
        return has_q ? launch<G, N, I, XiMode::Fixed, true, Draws::Any>(L, stream)
                     : launch<G, N, I, XiMode::Fixed, false, Draws::Any>(L, stream);
    if (L.a.ndraw & 1)
        return has_q ? launch<G, N, I, XiMode::Mask, true, Draws::OddTail>(L, stream)
                     : launch<G, N, I, XiMode::Mask, false, Draws::OddTail>(L, stream);
    return has_q ? launch<G, N, I, XiMode::Mask, true, Draws::Even>(L, stream)
                 : launch<G, N, I, XiMode::Mask, false, Draws::Even>(L, stream);
}

template <int N>
hipError_t launch_width(const TileLaunch& L, XiMode mode, bool has_q, hipStream_t stream)
{
    switch (L.a.W) {
    case 1: return L.a.nb < 64 ? launch_mode<0, N, 1>(L, mode, has_q, stream) : launch_mode<1, N, 1>(L, mode, has_q, stream);
    case 2: return launch_mode<2, N, 1>(L, mode, has_q, stream);
    case 4: return launch_mode<4, N, 1>(L, mode, has_q, stream);
    case 8: return launch_mode<8, N, 1>(L, mode, has_q, stream);
    case 16: return launch_mode<16, N, 1>(L, mode, has_q, stream);
    case 32: return launch_mode<32, N, 1>(L, mode, has_q, stream);
    case 64: return launch_mode<64, N, 1>(L, mode, has_q, stream);
    case 128: return N == 4 ? launch_mode<64, 4, 2>(L, mode, has_q, stream) : hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_tile(const SweepArgs& a, XiMode mode, bool has_q, const uint64_t* src, uint64_t* dst,
                       const TileShape& s, int32_t n_mcs, hipStream_t stream)
{
    if (n_mcs <= 0) return hipSuccess;
    const TileLaunch L{a, src, dst, s.rows, s.band, s.halo, n_mcs, 0};
    switch (s.rows_per_thread) {
    case 2: return launch_width<2>(L, mode, has_q, stream);
    case 4: return launch_width<4>(L, mode, has_q, stream);
    default: return hipErrorInvalidValue;
    }
}

// The kernel launch_tile runs (see launch_width and launch_mode).
void tile_kernel_name(const SweepArgs& a, XiMode mode, bool has_q, int32_t rows_per_thread, char* out, size_t n)
{
    const int G = a.W == 1 && a.nb < 64 ? 0 : (a.W < 64 ? a.W : 64);
    const char* const odd = a.ndraw & 1 ? "OddTail" : "Even";
    char words[24];
    if (mode == XiMode::PerSite || a.ndraw == 0)
        std::snprintf(words, sizeof words, mode == XiMode::PerSite ? "PerSite" : "Fixed");
    else
        std::snprintf(words, sizeof words, "%s,%s", mode == XiMode::Ahead ? "Ahead" : "Mask", odd);
    std::snprintf(out, n, "tile_kernel<%d,%d,%d,%s,%s>", G, rows_per_thread, a.W > 64 ? a.W / 64 : 1, words,
                  has_q ? "true" : "false");
}

}  // namespace sca
