// tile.hpp -- all rows of a tile advanced together, half-step by half-step,
// with the state on chip: the sweep of small and mid-sized lattices.
//
// The blocked sweeps of fused.hpp walk down a band row by row, which needs
// many bands to fill the chip; a lattice of 2^12 rows has none to spare.  Here
// a workgroup holds every row of its tile at once: a thread owns N
// consecutive rows of one word column (two for the smallest latency), a row
// of W words lies in W neighbouring lanes (or, from 128 words on, I words per
// lane of one wave), and each half-step updates the whole tile between two
// workgroup barriers.
//
// The x-slopes never leave their thread's registers: bits cross word
// boundaries by lane rotations.  The y-slopes of a row are used by the row
// itself in one half-step and, as the y+ slopes, by the row above it in the
// other, so those of a thread's first row change hands every half-step
// through one LDS word per array, and those of its other rows stay in
// registers.  A word in LDS has one reader and writer per half-step, so one
// barrier per half-step is all the ordering there is.
//
// A tile is either a whole periodic lattice (one workgroup, any number of
// MCS, in place), or a band of rows with enough rows around it for n MCS:
// half-step h (0 .. 2n-1) then has to be right only in the rows
// -2n+h .. band+2n-2-h of the band, and waves that hold none of them skip it.
// The row behind the tile's last one wraps to its first, which is the
// periodic neighbour in the first form and outside that cone in the second.
//
// What bounds it: with a wave or two per CU the chain of one half-step (LDS
// write, barrier, LDS read, the row's masks: 0.13 us at p = 1, 0.16 us at p =
// 1/2), with eight and more waves the vector issue.  Against two launches per
// MCS (2.8 us each, 1.6 us of it in the kernel): 128 x 128 at p = 1/2, 1000 MCS,
// 5.80 to 0.30 ms; 2^12 x 2^12 at p = 3/4, q = 1/4, 6.1 to 2.4 us per MCS, of
// which half is the recomputed halo (16-row bands, 12 MCS per pass).
#pragma once

#include "halfstep.hpp"

namespace sca {
namespace {

// The lanes of a row.  G lanes hold it (a power of two up to 64); G = 0: one
// lane whose word has fewer than 64 bits in use; G = -1: known at run time.
struct RowLanes {
    int G, nb;         // run-time G and the used bits per word (scalars; G = -1, nb also G = 0)
    bool first, last;  // this lane holds the row's first / last word
    bool upper;        // lane 32 or above
};

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
}

// Lane i of an aligned group of G lanes receives v from lane (i+1) mod G of
// its group (group_next) or from lane (i-1) mod G (group_prev): quad permutes
// for G = 2 and 4, two DPP row shifts and a select for G = 8, row rotates for
// G = 16 (a DPP row of 16 lanes is the group), the wavefront rotate for
// G = 64 and, with the two wrapping lanes from scalars, G = 32.  G is a
// template argument: with a scalar branch on it a pass of 8 MCS over 2^12 x
// 2^12 sites at p = 1 took 15.0 us instead of 10.6 us.
template <int G>
__device__ __forceinline__ uint32_t group_next(uint32_t v, const RowLanes& r)
{
    if constexpr (G == 1) return v;
    if constexpr (G == 2) return dpp<0xb1 /* quad_perm 1,0,3,2 */>(v);
    if constexpr (G == 4) return dpp<0x39 /* quad_perm 1,2,3,0 */>(v);
    if constexpr (G == 8) {
        const uint32_t n = dpp<0x101 /* row_shl:1 */>(v), w = dpp<0x117 /* row_shr:7 */>(v);
        return r.last ? w : n;
    }
    if constexpr (G == 16) return dpp<0x12f /* row_ror:15 */>(v);
    if constexpr (G == 64) return from_next_lane(v);
    if constexpr (G < 0) {
        switch (r.G) {
        case 1: return v;
        case 2: return group_next<2>(v, r);
        case 4: return group_next<4>(v, r);
        case 8: return group_next<8>(v, r);
        case 16: return group_next<16>(v, r);
        case 32: return group_next<32>(v, r);
        default: return group_next<64>(v, r);
        }
    }
    if constexpr (G == 32) {
        const uint32_t n = from_next_lane(v);
        const uint32_t v0 = (uint32_t)__builtin_amdgcn_readlane((int)v, 0);
        const uint32_t v32 = (uint32_t)__builtin_amdgcn_readlane((int)v, 32);
        const uint32_t w = r.upper ? v32 : v0;
        return r.last ? w : n;
    }
}

template <int G>
__device__ __forceinline__ uint32_t group_prev(uint32_t v, const RowLanes& r)
{
    if constexpr (G == 1) return v;
    if constexpr (G == 2) return dpp<0xb1 /* quad_perm 1,0,3,2 */>(v);
    if constexpr (G == 4) return dpp<0x93 /* quad_perm 3,0,1,2 */>(v);
    if constexpr (G == 8) {
        const uint32_t p = dpp<0x111 /* row_shr:1 */>(v), w = dpp<0x107 /* row_shl:7 */>(v);
        return r.first ? w : p;
    }
    if constexpr (G == 16) return dpp<0x121 /* row_ror:1 */>(v);
    if constexpr (G == 64) return from_prev_lane(v);
    if constexpr (G < 0) {
        switch (r.G) {
        case 1: return v;
        case 2: return group_prev<2>(v, r);
        case 4: return group_prev<4>(v, r);
        case 8: return group_prev<8>(v, r);
        case 16: return group_prev<16>(v, r);
        case 32: return group_prev<32>(v, r);
        default: return group_prev<64>(v, r);
        }
    }
    if constexpr (G == 32) {
        const uint32_t p = from_prev_lane(v);
        const uint32_t v31 = (uint32_t)__builtin_amdgcn_readlane((int)v, 31);
        const uint32_t v63 = (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
        const uint32_t w = r.upper ? v63 : v31;
        return r.first ? w : p;
    }
}

// Acceptance words (mask mode) of M words at once, the M Philox calls of each
// draw side by side: mask_words (halfstep.hpp) word by word, for an even
// number of draws or an odd one whose shared draw is kept in tail.
template <Draws DR, bool HASQ, int M>
__device__ __forceinline__ void mask_words_side_by_side(const SweepArgs& a, const uint32_t (&g)[M], uint64_t (&xp)[M],
                                                        uint64_t (&xq)[M], uint64_t (&tail)[M])
{
    static_assert(DR != Draws::Any, "the number of draws is even or keeps its tail");
#pragma unroll
    for (int m = 0; m < M; ++m) xp[m] = xq[m] = 0;
    auto fold = [&](int m, uint64_t r, int d) {
        xp[m] = fold_digit(r, xp[m], (a.dig_p >> d) & 1u);
        if (HASQ) xq[m] = fold_digit(r, xq[m], (a.dig_q >> d) & 1u);
    };
    int j = ((a.ndraw + 1) >> 1) - 1;  // the last call
    if constexpr (DR == Draws::OddTail) {
#pragma unroll
        for (int m = 0; m < M; ++m) {
            uint64_t r = tail[m];
            if (a.parity == 0) {
                const u32x4 o = philox_word(g[m], a.t, 2u * (uint32_t)j, a.k0, a.k1);
                r = (uint64_t)o.v0 | ((uint64_t)o.v1 << 32);
                tail[m] = (uint64_t)o.v2 | ((uint64_t)o.v3 << 32);
            }
            fold(m, r, 2 * j);
        }
        --j;
    }
    for (; j >= 0; --j) {
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const u32x4 o = philox_word(g[m], a.t, 2u * (uint32_t)j + (uint32_t)a.parity, a.k0, a.k1);
            fold(m, (uint64_t)o.v2 | ((uint64_t)o.v3 << 32), 2 * j + 1);
            fold(m, (uint64_t)o.v0 | ((uint64_t)o.v1 << 32), 2 * j);
        }
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
        xp[m] |= a.all_p;
        if (HASQ) xq[m] |= a.all_q;
    }
}

// One half-step of one row: A, B on-site x- and y- slopes, C the y+ slopes
// (the next row's other-sublattice y- words), D the x+ slopes (this row's
// other-sublattice x- words), all I words of this lane (word i*64 + lane).
// SH: the row's x+ neighbours sit one site further, across the word edge.
// mp, mq: the masks of word 0.
template <int G, bool SH, int I, bool HASQ>
__device__ __forceinline__ void tile_row(const RowLanes& rl, uint64_t (&A)[I], uint64_t (&B)[I], uint64_t (&C)[I],
                                         uint64_t (&D)[I], const uint64_t (&xp)[I], const uint64_t (&xq)[I],
                                         uint64_t& mp0, uint64_t& mq0)
{
    static_assert(I == 1 || I == 2, "one or two words per lane");
    uint64_t XP[I], M[I];
    if constexpr (!SH) {
#pragma unroll
        for (int i = 0; i < I; ++i) XP[i] = D[i];
    } else if (G == 0 || (G < 0 && rl.nb < 64)) {
        XP[0] = (D[0] >> 1) | ((D[0] & 1ull) << (rl.nb - 1));
    } else if constexpr (G != 0) {
        uint32_t nl[I];
#pragma unroll
        for (int i = 0; i < I; ++i) nl[i] = group_next<G>((uint32_t)D[i], rl);
        if constexpr (I == 2) {  // the last lane of word 0 continues in the first lane of word 1, and round
            const uint32_t n0 = nl[0];
            nl[0] = rl.last ? nl[1] : n0;
            nl[1] = rl.last ? n0 : nl[1];
        }
#pragma unroll
        for (int i = 0; i < I; ++i) {
            const uint32_t lo = (uint32_t)D[i], hi = (uint32_t)(D[i] >> 32);
            XP[i] = (uint64_t)__builtin_amdgcn_alignbit(hi, lo, 1u) |
                    ((uint64_t)__builtin_amdgcn_alignbit(nl[i], hi, 1u) << 32);
        }
    }
#pragma unroll
    for (int i = 0; i < I; ++i) {
        const uint64_t mp = bitop3<0x80>(bitop3<0x02>(A[i], B[i], XP[i]), C[i], xp[i]);  // xi & ~A & ~B & XP & C
        const uint64_t mq = HASQ ? bitop3<0x20>(bitop3<0x40>(A[i], B[i], XP[i]), C[i], xq[i])  // xi & A & B & ~XP & ~C
                                 : 0ull;
        if (i == 0) {
            mp0 = mp;
            mq0 = mq;
        }
        M[i] = mp | mq;
        A[i] ^= M[i];
        B[i] ^= M[i];
        C[i] ^= M[i];
    }
    if constexpr (!SH) {
#pragma unroll
        for (int i = 0; i < I; ++i) D[i] ^= M[i];
    } else if (G == 0 || (G < 0 && rl.nb < 64)) {
        D[0] ^= ((M[0] << 1) | (M[0] >> (rl.nb - 1))) & ((1ull << rl.nb) - 1ull);
    } else if constexpr (G != 0) {
        uint32_t ph[I];
#pragma unroll
        for (int i = 0; i < I; ++i) ph[i] = group_prev<G>((uint32_t)(M[i] >> 32), rl);
        if constexpr (I == 2) {
            const uint32_t p0 = ph[0];
            ph[0] = rl.first ? ph[1] : p0;
            ph[1] = rl.first ? p0 : ph[1];
        }
#pragma unroll
        for (int i = 0; i < I; ++i) {
            const uint32_t lo = (uint32_t)M[i], hi = (uint32_t)(M[i] >> 32);
            D[i] ^= (uint64_t)__builtin_amdgcn_alignbit(lo, ph[i], 31u) |
                    ((uint64_t)__builtin_amdgcn_alignbit(hi, lo, 31u) << 32);
        }
    }
}

// Per-site acceptance words of a tile (one word per lane).  A word takes 16
// Philox calls, too many for the few waves that hold a small tile's rows, so
// the whole workgroup forms them, eight sites (two calls) of a word per thread
// and byte, into one of two buffers in LDS; the barrier that starts the
// half-step orders them like the slopes, and the buffer of the half-step before
// is free again behind it.  Bound by vector issue beyond a few hundred words per
// CU: 1024 x 1024 at p = 0.95, 20 MCS and moments, took 255 us in half-step
// launches of 4.3 us (one lane per word, two waves on half of the CUs) and takes
// 69 us.
struct PerSiteTile {
    uint64_t* xi;   // [sublattice][p, q][tile row][word]
    int words;      // words of the tile
    int lw;         // log2 of the words per row
    int lk;         // log2 of the bytes in use per word
    int y0, ymask;  // lattice row of tile row 0
    bool has_q;

    __device__ __forceinline__ uint64_t* buffer(int parity) const { return xi + (parity ? (has_q ? 2 : 1) * words : 0); }

    // The words of tile rows lo .. hi for sublattice a.parity at MCS a.t.
    template <bool HASQ>
    __device__ __forceinline__ void generate(const SweepArgs& a, int lo, int hi) const
    {
        uint8_t* const out = reinterpret_cast<uint8_t*>(buffer(a.parity));
        const int end = (hi + 1) << (lw + lk);
        for (int i = (lo << (lw + lk)) + (int)threadIdx.x; i < end; i += (int)blockDim.x) {
            const int w = i >> lk, k = i & ((1 << lk) - 1);
            const int row = (y0 + (w >> lw)) & ymask;
            const uint32_t g = ((uint32_t)row << lw) + (uint32_t)(w & ((1 << lw) - 1));
            const uint32_t c2 = 4u * (uint32_t)k + (uint32_t)a.parity;  // calls 2k and 2k+1
            const u32x4 o1 = philox4x32_10(g, a.t, c2 + 2u, 0u, a.k0, a.k1);
            const u32x4 o0 = philox4x32_10(g, a.t, c2, 0u, a.k0, a.k1);
            out[8 * w + k] = (uint8_t)shift_in_compares(shift_in_compares(0u, o1, a.thr_p), o0, a.thr_p);
            if (HASQ)
                out[8 * (words + w) + k] = (uint8_t)shift_in_compares(shift_in_compares(0u, o1, a.thr_q), o0, a.thr_q);
        }
    }
};

// Acceptance words of a tile of few waves (one word per lane, mask mode),
// formed by further waves of the workgroup one MCS ahead.  They depend on
// counters alone, so that the rows' waves keep only the chain through the slopes
// while the other SIMDs of the CU, idle otherwise, run the Philox calls.  Two
// buffers in LDS, one per MCS in turn; the barrier that starts an MCS orders them.
// Bound by that chain with one wave of rows (0.13 us without words), by the
// producers' chain with more draws, by vector issue from four waves on.  us per
// half-step before and after, p = 1/2; p = 3/4, q = 1/4; p = 15/16:
//   one wave   (128 x 128)  0.225 to 0.159, 0.39 to 0.23, 0.50 to 0.33
//   two waves  (512 x 64)   0.273 to 0.211, 0.45 to 0.32, 0.57 to 0.40
//   four waves (256 x 256)  0.306 to 0.247, 0.51 to 0.42, 0.64 to 0.53
struct AheadTile {
    uint64_t* xi;   // [MCS mod 2][sublattice][p, q][tile row][word]
    int words;      // words of the tile
    int lw;         // log2 of the words per row
    int y0, ymask;  // lattice row of tile row 0
    int q;          // 1 with removals

    __device__ __forceinline__ uint64_t* buffer(uint32_t t, int parity) const
    {
        return xi + ((int)(2 * (t & 1u)) + parity) * (words << q);
    }

    // Word w of the tile for sublattice PI at MCS a.t; tail as in mask_words.
    template <int PI, bool HASQ, Draws DR>
    __device__ __forceinline__ void generate(SweepArgs a, int w, uint64_t& tail) const
    {
        const uint32_t row = (uint32_t)((y0 + (w >> lw)) & ymask);
        a.parity = PI;
        uint64_t xp, xq;
        mask_words<DR>(a, (row << lw) + (uint32_t)(w & ((1 << lw) - 1)), HASQ, xp, xq, &tail);
        uint64_t* const out = buffer(a.t, PI) + w;
        out[0] = xp;
        if (HASQ) out[words] = xq;
    }
};

// What a half-step does at the tile's first and last row beyond the tile:
// nothing, where the tile wraps or its halo runs out.
struct NoEdge {
    template <int I>
    __device__ __forceinline__ void take(uint64_t (&)[I], uint64_t (&)[I])
    {
    }
    template <int I>
    __device__ __forceinline__ void give_first(const uint64_t (&)[I])
    {
    }
    template <int I>
    __device__ __forceinline__ void give_last(const uint64_t (&)[I])
    {
    }
};

// The rows of one thread and the half-step over them.  KEEP: draws kept from
// one half-step to the next wait in LDS instead of registers.
template <int G, int N, int I, XiMode MODE, bool HASQ, Draws DR, bool KEEP = false>
struct TileThread {
    static_assert(N % 2 == 0, "the alignment of row i is that of i");
    static_assert(I == 1 || G == 64, "a row of several words per lane fills a wave");
    // Rows whose random words are formed together: two words' worth.  With two
    // words per thread those are all of a half-step, formed before the barrier
    // it starts with and so off the path from write to read.  Words that others
    // form come from LDS behind the barrier.
    static constexpr bool PRE = N * I <= 2 && MODE != XiMode::PerSite && MODE != XiMode::Ahead;
    static constexpr int NX = N >= 8 ? 1 : 2 / I;
    // The shared last draw of an odd number of draws waits for the odd half-step.
    static constexpr bool TAIL = DR == Draws::OddTail && MODE == XiMode::Mask;
    static constexpr bool TAIL_LDS = TAIL && KEEP;

    uint64_t x[N][2][I];  // x-slopes by sublattice
    uint64_t y[N][2][I];  // y-slopes; row 0 only within a half-step
    uint64_t tail[TAIL && !TAIL_LDS ? N : 1][I];
    uint64_t* kept;       // word k of row i at (i * I + k) * blockDim.x (TAIL_LDS)
    uint32_t g0;          // canonical index of row 0's word 0 (the rows lie W apart)
    uint32_t W;
    RowLanes rl;
    int own, nxt;         // LDS index of this thread's first row and of the next thread's (stride words apart per i)
    int stride;           // LDS words per (sublattice, i)
    uint32_t org[N / 2];  // 1 in the lane and even row that hold site (0,0) (never in a halo row)
    int32_t lifts;        // (lifts - drops) of site (0,0)
    PerSiteTile ps;       // per-site mode
    AheadTile ahead;      // ahead mode
    int xrow;             // index of the first row's word in a buffer of acceptance words

    // The rows of a half-step are independent; they go first, last, then the
    // ones between, so that the two that a neighbouring tile waits for come
    // early.
    static constexpr __device__ int row(int m) { return m == 0 ? 0 : m == 1 ? N - 1 : m - 1; }

    __device__ __forceinline__ uint32_t g(int i) const { return g0 + (uint32_t)i * W; }

    // Acceptance words of rows row(m0) .. row(m0 + NX - 1).
    __device__ __forceinline__ void words(const SweepArgs& a, int m0, uint64_t (&xp)[NX][I], uint64_t (&xq)[NX][I])
    {
        if constexpr (MODE == XiMode::Mask) {
            uint32_t gg[NX * I];
            uint64_t p[NX * I], q[NX * I], t[NX * I];
#pragma unroll
            for (int m = 0; m < NX * I; ++m) {
                gg[m] = g(row(m0 + m / I)) + 64u * (m % I);
                // With many rows per thread the products of the word index that
                // every Philox call starts with are formed anew each time: kept
                // across the half-steps they take four registers per row.
                if constexpr (N * I >= 4) asm volatile("" : "+v"(gg[m]));
                t[m] = 0;
                if constexpr (TAIL_LDS) {
                    if (a.parity == 1) t[m] = kept[(row(m0 + m / I) * I + m % I) * (int)blockDim.x];
                } else if constexpr (TAIL) {
                    t[m] = tail[row(m0 + m / I)][m % I];
                }
            }
            mask_words_side_by_side<DR, HASQ>(a, gg, p, q, t);
#pragma unroll
            for (int m = 0; m < NX * I; ++m) {
                if constexpr (TAIL_LDS) {
                    if (a.parity == 0) kept[(row(m0 + m / I) * I + m % I) * (int)blockDim.x] = t[m];
                } else if constexpr (TAIL) {
                    tail[row(m0 + m / I)][m % I] = t[m];
                }
                xp[m / I][m % I] = p[m];
                xq[m / I][m % I] = q[m];
            }
        } else {
#pragma unroll
            for (int m = 0; m < NX * I; ++m) {
                xp[m / I][m % I] = a.all_p;
                xq[m / I][m % I] = a.all_q;
                if constexpr (MODE == XiMode::Ahead) {
                    const uint64_t* w = ahead.buffer(a.t, a.parity) + xrow + (row(m0 + m) << ahead.lw);
                    xp[m][0] = w[0];
                    if (HASQ) xq[m][0] = w[ahead.words];
                } else if constexpr (MODE == XiMode::PerSite) {
                    const uint64_t* w = ps.buffer(a.parity) + xrow + (row(m0 + m) << ps.lw);
                    xp[m][0] |= w[0];
                    if (HASQ) xq[m][0] |= w[ps.words];
                }
            }
        }
    }

    // Half-step of sublattice PI at MCS a.t; tile rows lo .. hi have to be
    // right, and `skip` (scalar): none of the wave's rows are among them.
    // `alone` (scalar): the wave holds all rows, and nothing else waits for it
    // at this half-step.
    template <int PI, class Edge>
    __device__ __forceinline__ void halfstep(SweepArgs a, uint64_t* ly, int lo, int hi, bool skip, Edge& edge,
                                             bool alone = false)
    {
        a.parity = PI;
        uint64_t xp[NX][I], xq[NX][I];
        if constexpr (MODE == XiMode::PerSite) ps.generate<HASQ>(a, lo, hi);
        if constexpr (PRE) {
            if (!skip) words(a, 0, xp, xq);
        }
        if (alone) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            __syncthreads();
        }
        if (skip) return;
        uint64_t* const lB = ly + PI * I * stride;        // y- slopes of the first row
        uint64_t* const lC = ly + (1 - PI) * I * stride;  // y+ slopes behind the last row
        uint64_t Cn[I];
#pragma unroll
        for (int k = 0; k < I; ++k) {
            y[0][PI][k] = lB[k * stride + own];
            Cn[k] = lC[k * stride + nxt];
        }
        edge.take(y[0][PI], Cn);
#pragma unroll
        for (int m = 0; m < N; ++m) {
            constexpr bool even_shifted = PI != 0;  // rows of even i are shifted in the odd half-step
            const int i = row(m);
            uint64_t mp0 = 0, mq0 = 0;
            if constexpr (!PRE)
                if (m % NX == 0) words(a, m, xp, xq);
            uint64_t(&C)[I] = i + 1 < N ? y[i + 1 < N ? i + 1 : 0][1 - PI] : Cn;
            if ((i & 1) == 0)
                tile_row<G, even_shifted, I, HASQ>(rl, x[i][PI], y[i][PI], C, x[i][1 - PI], xp[m % NX], xq[m % NX],
                                                   mp0, mq0);
            else
                tile_row<G, !even_shifted, I, HASQ>(rl, x[i][PI], y[i][PI], C, x[i][1 - PI], xp[m % NX], xq[m % NX],
                                                    mp0, mq0);
            // Pin the new slopes here, or the compiler interleaves the rows and
            // keeps the masks of all of them live.
            if constexpr (!PRE && MODE != XiMode::Ahead) {
#pragma unroll
                for (int k = 0; k < I; ++k)
                    asm volatile("" : "+v"(x[i][0][k]), "+v"(x[i][1][k]), "+v"(y[i][PI][k]), "+v"(C[k]));
            }
            if (PI == 0 && (i & 1) == 0) {
                lifts += (int32_t)((uint32_t)mp0 & org[i / 2]);
                if (HASQ) lifts -= (int32_t)((uint32_t)mq0 & org[i / 2]);
            }
            if (m == 0) edge.give_first(y[0][PI]);
            if (m == 1) edge.give_last(Cn);
        }
#pragma unroll
        for (int k = 0; k < I; ++k) {
            lB[k * stride + own] = y[0][PI][k];
            lC[k * stride + nxt] = Cn[k];
        }
    }
};

}  // namespace
}  // namespace sca
