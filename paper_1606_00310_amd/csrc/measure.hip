// measure.hip -- flat initial state, heights, exact height moments and
// two-time sums on gfx950.
//
// Heights are not stored; they follow from the slopes (Sec. II-A keeps two
// slope bits per site) and the tracked origin height h(0,0):
//   h(x,y) = c(y) + P_y(x),  c(y) = h(0,0) + sum_{j=1..y} (2 sy(0,j) - 1),
//   P_y(x) = sum_{i=1..x} (2 sx(i,y) - 1).
// Row y's x-slopes interleave two words per 128 sites: even x in the x-array
// of parity y&1, odd x in that of parity 1-(y&1), bit x>>1.
//
// Moments decompose exactly.  Eight consecutive sites are looked up at once: a
// table in LDS gives, for their eight slope bits, the running counts c_1..c_8
// of rises as eight nibbles, so that with the height K in front of them the
// heights are K + 2 c_i - i and every sum over them is a v_dot8_u32_u4 of
// nibbles:  sum c = c.(1..1),  sum c^2 = c.c,  sum i c = c.(1,2,..8), and for
// two states  sum c_t c_s = c_t.c_s.  Words, rows and blocks of rows then
// combine by
//   sum (B + d_i) = n B + sum d_i,   sum (B + d_i)^2 = n B^2 + 2 B sum d_i + sum d_i^2
// in int64, and the blocks in 128 bits.  Nothing is rounded at any stage.
#include "sca_internal.hpp"

namespace sca {
namespace {

constexpr int kBlock = 256;

__global__ void flat_init_kernel(uint64_t* S, int64_t plane, uint64_t valid, int64_t* h0)
{
    const int64_t n = 4 * plane;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int parity = (int)((i / plane) & 1);  // arrays ordered S[d][parity]
        S[i] = parity ? valid : 0ull;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *h0 = 0;
}

// The flat surface for many lattices at once: workgroups (i, 0), (i, 1), ..
// initialise items i, i + gridDim.x, ... (their states are small: one admission
// of an ensemble issues one launch instead of one per realization).  With one
// workgroup per item the largest, 1 MiB, set the time: 61 us for 512 of 2^6 to
// 2^11 squared, 30 us with eight.
__device__ __forceinline__ void flat_item_init(const FlatItem& f)
{
    const int64_t words = 4 * f.plane;
    for (int64_t i = (int64_t)blockIdx.y * kBlock + threadIdx.x; i < words; i += (int64_t)gridDim.y * kBlock) {
        const int parity = (int)((i / f.plane) & 1);  // arrays ordered S[d][parity]
        f.S[i] = parity ? f.valid : 0ull;
    }
    if (blockIdx.y == 0 && threadIdx.x == 0) *f.h0 = 0;
}

__global__ __launch_bounds__(kBlock) void flat_init_many_kernel(const FlatItem* items, int32_t n)
{
    for (int32_t it = blockIdx.x; it < n; it += gridDim.x) flat_item_init(items[it]);
}

// Up to 32 items as an argument: no table to copy first, which takes a small
// admission 4 us of 12.
struct FlatFew {
    FlatItem items[kFlatFew];
};
__global__ __launch_bounds__(kBlock) void flat_init_few_kernel(FlatFew f) { flat_item_init(f.items[blockIdx.x]); }

// ---------------------------------------------------------------- sums of one word pair
// Eight nibbles 1 and the nibbles 1..8.
constexpr uint32_t kOnes = 0x11111111u, kRamp = 0x87654321u;

// The running counts of rises over the eight sites whose even-x slopes are the
// low four bits of `byte` and whose odd-x slopes the high four.
__device__ __forceinline__ uint32_t running_counts(uint32_t byte)
{
    uint32_t c = 0, out = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        c += (byte >> k) & 1u;
        out |= c << (8 * k);
        c += (byte >> (4 + k)) & 1u;
        out |= c << (8 * k + 4);
    }
    return out;
}

__device__ __forceinline__ uint32_t dot8(uint32_t a, uint32_t b, uint32_t acc)
{
    return __builtin_amdgcn_udot8(a, b, acc, false);
}

// The table indices of a half word pair's eight chunks, in site order: byte m
// of `even` is chunk 2m, of `odd` chunk 2m+1.
struct ChunkBytes {
    uint32_t even, odd;
    __device__ __forceinline__ ChunkBytes(uint32_t e, uint32_t o)
        : even((e & 0x0f0f0f0fu) | ((o & 0x0f0f0f0fu) << 4)), odd(((e >> 4) & 0x0f0f0f0fu) | (o & 0xf0f0f0f0u))
    {
    }
    __device__ __forceinline__ uint32_t operator[](int j) const
    {
        return (((j & 1) ? odd : even) >> (8 * (j >> 1))) & 255u;
    }
};

// Sums over the 8 * chunks sites of a word pair (even-x word E, odd-x word O)
// of the heights d_i relative to the site in front of the first.
struct WordSums {
    int32_t tot;  // d of the last site
    int32_t s1;   // sum of d_i
    int32_t s2;   // sum of d_i^2, or of d_i d'_i for two states
};

// Eight sites behind height B: sum d = 8 B + 2 s - 36 and sum d^2 = 8 B^2 +
// 2 B (2 s - 36) + 4 c.c - 4 c.ramp + 204 with s = c.(1..1).
__device__ __forceinline__ WordSums word_sums(const uint32_t* lut, uint64_t E, uint64_t O, int chunks)
{
    int32_t B = 0, sB = 0, sBB = 0, sBs = 0;
    uint32_t S = 0, cc = 0, cr = 0;
    auto half = [&](uint32_t e, uint32_t o, int n) {
        const ChunkBytes idx(e, o);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (j >= n) break;
            const uint32_t c = lut[idx[j]];
            const uint32_t s = dot8(c, kOnes, 0);
            cc = dot8(c, c, cc);
            cr = dot8(c, kRamp, cr);
            S += s;
            sB += B;
            sBB += B * B;
            sBs += B * (int32_t)s;
            B += 2 * (int32_t)(c >> 28) - 8;
        }
    };
    if (chunks == 16) {
        half((uint32_t)E, (uint32_t)O, 8);
        half((uint32_t)(E >> 32), (uint32_t)(O >> 32), 8);
    } else {
        half((uint32_t)E, (uint32_t)O, chunks);
    }
    return {B, 8 * sB + 2 * (int32_t)S - 36 * chunks,
            8 * sBB + 4 * sBs - 72 * sB + 4 * (int32_t)cc - 4 * (int32_t)cr + 204 * chunks};
}

// Two states t and s: sum d_t d_s = 8 Bt Bs + Bt (2 ss - 36) + Bs (2 st - 36)
// + 4 ct.cs - 2 ct.ramp - 2 cs.ramp + 204.
__device__ __forceinline__ void word_sums2(const uint32_t* lut, uint64_t Et, uint64_t Ot, uint64_t Es, uint64_t Os,
                                           int chunks, WordSums& t, WordSums& s)
{
    int32_t Bt = 0, Bs = 0, sBt = 0, sBs = 0, m = 0;
    uint32_t St = 0, Ss = 0, cc = 0, cr = 0;
    auto half = [&](uint32_t et, uint32_t ot, uint32_t es, uint32_t os, int n) {
        const ChunkBytes it(et, ot), is(es, os);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (j >= n) break;
            const uint32_t ct = lut[it[j]], cs = lut[is[j]];
            const uint32_t st = dot8(ct, kOnes, 0), ss = dot8(cs, kOnes, 0);
            cc = dot8(ct, cs, cc);
            cr = dot8(cs, kRamp, dot8(ct, kRamp, cr));
            St += st;
            Ss += ss;
            sBt += Bt;
            sBs += Bs;
            m += Bt * (4 * Bs + (int32_t)ss) + Bs * (int32_t)st;
            Bt += 2 * (int32_t)(ct >> 28) - 8;
            Bs += 2 * (int32_t)(cs >> 28) - 8;
        }
    };
    if (chunks == 16) {
        half((uint32_t)Et, (uint32_t)Ot, (uint32_t)Es, (uint32_t)Os, 8);
        half((uint32_t)(Et >> 32), (uint32_t)(Ot >> 32), (uint32_t)(Es >> 32), (uint32_t)(Os >> 32), 8);
    } else {
        half((uint32_t)Et, (uint32_t)Ot, (uint32_t)Es, (uint32_t)Os, chunks);
    }
    t = {Bt, 8 * sBt + 2 * (int32_t)St - 36 * chunks,
         2 * m - 36 * (sBt + sBs) + 4 * (int32_t)cc - 2 * (int32_t)cr + 204 * chunks};
    s = {Bs, 8 * sBs + 2 * (int32_t)Ss - 36 * chunks, 0};
}

// Two sites per word (X = 4): too few for a table entry.
__device__ __forceinline__ void four_sites(uint64_t E, uint64_t O, int32_t (&d)[4])
{
    int32_t h = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        h += 2 * (int32_t)((((k & 1) ? O : E) >> (k >> 1)) & 1ull) - 1;
        d[k] = h;
    }
}

// Inclusive scan across the G lanes of a row group.
template <int G>
__device__ __forceinline__ int32_t group_incl_scan(int32_t v, int gl)
{
#pragma unroll
    for (int off = 1; off < G; off <<= 1) {
        const int32_t o = __shfl_up(v, off, G);
        if (gl >= off) v += o;
    }
    return v;
}

// ---------------------------------------------------------------- moments
constexpr int kSumBlock = 1024;              // threads of a block of rows
constexpr int kSumRows = 1024;               // rows of a block at most
constexpr int kPartial = kMomentsPartial;    // int64 per block

// Heights of column 0 for the R rows from y0 on, relative to the row in front
// of the block (to row 0's own height in the block with row 0), less the slope
// at x = 0: what a row's path from x = 0 on, that slope included, starts from.
// col: the last row's height of column 0.  One row per thread.
__device__ __forceinline__ void row_bases(const uint64_t* S, int64_t plane, int32_t W, int64_t y0, int R, int32_t* rb,
                                          int32_t* col, int32_t* waves)
{
    const int r = (int)threadIdx.x, lane = r & 63, wv = r >> 6;
    const int64_t y = y0 + (r < R ? r : 0);
    const int64_t base = (y & 1) * plane + y * W;
    const uint64_t x0 = S[base], yw = S[2 * plane + base];  // the even-x word holds x = 0
    const int32_t step = (y == 0 || r >= R) ? 0 : 2 * (int32_t)(yw & 1ull) - 1;
    const int32_t incl = group_incl_scan<64>(step, lane);
    if (lane == 63) waves[wv] = incl;
    __syncthreads();
    int32_t before = 0;
    for (int k = 0; k < wv; ++k) before += waves[k];
    if (r < R) rb[r] = before + incl - (2 * (int32_t)(x0 & 1ull) - 1);
    if (r == R - 1) *col = before + incl;
    __syncthreads();
}

struct Sums128 {
    __int128 v[3];
};

// Adds one block's sums (relative to its first row's predecessor) at the
// absolute heights Ct, Cs: {sum h, sum h^2, 0} or {sum h_t, sum h_t h_s, sum h_s}.
__device__ __forceinline__ void add_block(Sums128& t, const int64_t* p, int64_t n, int64_t Ct, int64_t Cs, bool two)
{
    const int64_t a1 = p[0], a2 = p[1], a3 = p[2];
    t.v[0] += (__int128)n * Ct + a1;
    if (!two) {
        t.v[1] += (__int128)n * Ct * Ct + (__int128)2 * Ct * a1 + a2;
    } else {
        t.v[1] += (__int128)n * Ct * Cs + (__int128)Ct * a3 + (__int128)Cs * a1 + a2;
        t.v[2] += (__int128)n * Cs + a3;
    }
}

// h0: where there is no second state, h(0,0) takes the place of its sum.
__device__ __forceinline__ void store_sums(Sums128& t, int64_t* res, const int32_t* flag, const int64_t* h0, bool two)
{
    if (!two) t.v[2] = *h0;
    for (int k = 0; k < 3; ++k) {
        res[2 * k] = (int64_t)(uint64_t)t.v[k];
        res[2 * k + 1] = (int64_t)(t.v[k] >> 64);
    }
    res[6] = flag ? *flag : 0;
}

constexpr int kCombine = 256;  // blocks of rows at most

// The blocks' sums at their absolute heights, in 128 bits: one block of rows
// per thread.
__global__ __launch_bounds__(kCombine) void combine_kernel(const int64_t* h0, const int64_t* snap_h0, bool two,
                                                          const int64_t* partials, int32_t blocks, int64_t sites,
                                                          int64_t* res, const int32_t* flag)
{
    __shared__ int32_t colsum[2][kCombine / 64];
    __shared__ __int128 red[kCombine / 64][3];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const bool on = (int)threadIdx.x < blocks;
    int64_t p[kPartial] = {0, 0, 0, 0, 0};
    if (on)
#pragma unroll
        for (int c = 0; c < kPartial; ++c) p[c] = partials[(int64_t)kPartial * threadIdx.x + c];
    Sums128 t{{0, 0, 0}};
    const int32_t it = group_incl_scan<64>((int32_t)p[3], lane), is = group_incl_scan<64>((int32_t)p[4], lane);
    if (lane == 63) {
        colsum[0][wv] = it;
        colsum[1][wv] = is;
    }
    __syncthreads();
    int64_t ct = *h0 + it - p[3], cs = (two ? *snap_h0 : 0) + is - p[4];
    for (int k = 0; k < wv; ++k) {
        ct += colsum[0][k];
        cs += colsum[1][k];
    }
    if (on) add_block(t, p, sites, ct, cs, two);
    for (int k = 0; k < 3; ++k) {
        __int128 v = t.v[k];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const uint64_t lo = __shfl_xor((uint64_t)v, off, 64);
            const int64_t hi = __shfl_xor((int64_t)(v >> 64), off, 64);
            v += ((__int128)hi << 64) | lo;
        }
        if (lane == 0) red[wv][k] = v;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int k = 0; k < 3; ++k) {
        t.v[k] = 0;
        for (int w = 0; w < kCombine / 64; ++w) t.v[k] += red[w][k];
    }
    store_sums(t, res, flag, h0, two);
}

// Bound by vector issue: about 13 instructions per eight sites (20 for two
// states) instead of some 60 in a loop over the sites, and the x-slopes read
// once.  2^14 x 2^14: two-time sums 202 us (87 us of it for the rows, the rest
// in one workgroup that combined them row by row) to 40 us; the moments of
// 128 x 128 in one launch of 4.6 us instead of two of 3.7 and 7.8 us.
//
// Sums over a block of R rows, with the workgroup's 16 waves on the rows'
// words: partials[5 * block + ..] = {sum P, sum P^2 or P_t P_s, sum P_s,
// column step of t, of s}, P the height over the row in front of the block.
// With one block the final sums go to res.  (Combining in the last block to
// finish, behind a device-scope counter, was slower than the second launch: the
// release writes back the L2 of its XCD, 137 instead of 130 us for all
// measurements of 2^13 x 2^13.)
template <bool TWO>
struct MomentsShared {
    uint32_t lut[256];
    int32_t rbt[kSumRows], rbs[TWO ? kSumRows : 1];
    int32_t col[2], waves[kSumBlock / 64];
    int64_t red[kSumBlock / 64][3];
};

template <int G, bool TWO>
__device__ __forceinline__ void block_moments(MomentsShared<TWO>& sh, int32_t block, int32_t blocks, const uint64_t* S,
                                              const int64_t* h0, const uint64_t* snap, const int64_t* snap_h0,
                                              int64_t Y, int32_t W, int32_t nb, int32_t R, int64_t* partials,
                                              int64_t* res, const int32_t* flag)
{
    uint32_t* const lut = sh.lut;
    const int32_t *const rbt = sh.rbt, *const rbs = sh.rbs;
    int64_t(&red)[kSumBlock / 64][3] = sh.red;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int gl = lane & (G - 1);
    const int64_t plane = Y * W, y0 = (int64_t)block * R;
    if (threadIdx.x < 256) lut[threadIdx.x] = running_counts(threadIdx.x);
    row_bases(S, plane, W, y0, R, sh.rbt, &sh.col[0], sh.waves);
    if (TWO) row_bases(snap, plane, W, y0, R, sh.rbs, &sh.col[1], sh.waves);

    const int chunks = nb >> 2, n = 2 * nb;
    int64_t a1 = 0, a2 = 0, a3 = 0;
    for (int r0 = wv * (64 / G); r0 < R; r0 += (kSumBlock / 64) * (64 / G)) {
        const int r_raw = r0 + lane / G;
        const bool active = r_raw < R;
        const int r = active ? r_raw : 0;
        const int64_t y = y0 + r;
        const int64_t pe = (y & 1) * plane + y * W, po = (1 - (y & 1)) * plane + y * W;
        int32_t ct = rbt[r], cs = TWO ? rbs[r] : 0;
        for (int w0 = 0; w0 < W; w0 += G) {
            const int w = w0 + gl;
            WordSums t, s{0, 0, 0};
            if (G == 1 && nb < 4) {
                int32_t d[4], ds[4];
                four_sites(S[pe + w], S[po + w], d);
                four_sites(TWO ? snap[pe + w] : S[pe + w], TWO ? snap[po + w] : S[po + w], ds);
                t = {d[3], d[0] + d[1] + d[2] + d[3], d[0] * ds[0] + d[1] * ds[1] + d[2] * ds[2] + d[3] * ds[3]};
                s = {ds[3], ds[0] + ds[1] + ds[2] + ds[3], 0};
            } else if constexpr (TWO) {
                word_sums2(lut, S[pe + w], S[po + w], snap[pe + w], snap[po + w], G == 1 ? chunks : 16, t, s);
            } else {
                t = word_sums(lut, S[pe + w], S[po + w], G == 1 ? chunks : 16);
            }
            const int32_t it = group_incl_scan<G>(t.tot, gl);
            const int32_t bt = ct + it - t.tot;
            int32_t bs = 0;
            if (TWO) {
                const int32_t is = group_incl_scan<G>(s.tot, gl);
                bs = cs + is - s.tot;
                if (w0 + G < W) cs += __shfl(is, (lane & ~(G - 1)) + G - 1);
            }
            if (w0 + G < W) ct += __shfl(it, (lane & ~(G - 1)) + G - 1);
            if (!active) continue;
            a1 += n * bt + t.s1;
            if (TWO) {
                a2 += (int64_t)bt * (n * bs + s.s1) + (int64_t)bs * t.s1 + t.s2;
                a3 += n * bs + s.s1;
            } else {
                a2 += (int64_t)bt * (n * bt + 2 * t.s1) + t.s2;
            }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        a1 += __shfl_xor(a1, off, 64);
        a2 += __shfl_xor(a2, off, 64);
        if (TWO) a3 += __shfl_xor(a3, off, 64);
    }
    if (lane == 0) {
        red[wv][0] = a1;
        red[wv][1] = a2;
        red[wv][2] = a3;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int k = 1; k < kSumBlock / 64; ++k)
        for (int c = 0; c < 3; ++c) red[0][c] += red[k][c];
    if (blocks == 1) {
        Sums128 tot{{0, 0, 0}};
        add_block(tot, red[0], (int64_t)n * W * R, *h0, TWO ? *snap_h0 : 0, TWO);
        store_sums(tot, res, flag, h0, TWO);
    } else {
        int64_t* p = partials + (int64_t)kPartial * block;
        for (int c = 0; c < 3; ++c) p[c] = red[0][c];
        p[3] = sh.col[0];
        p[4] = TWO ? sh.col[1] : 0;
    }
}

template <int G, bool TWO>
__global__ __launch_bounds__(kSumBlock) void moments_kernel(const uint64_t* S, const int64_t* h0, const uint64_t* snap,
                                                            const int64_t* snap_h0, int64_t Y, int32_t W, int32_t nb,
                                                            int32_t R, int64_t* partials, int64_t* res,
                                                            const int32_t* flag)
{
    __shared__ MomentsShared<TWO> sh;
    block_moments<G, TWO>(sh, (int32_t)blockIdx.x, (int32_t)gridDim.x, S, h0, snap, snap_h0, Y, W, nb, R, partials, res,
                          flag);
}

// The moments of many small lattices, one block each: a launch and a wait for
// each of them is what retiring an ensemble's realizations spends its time on
// (96 of 64 to 512 sites wide, served and collected: 5.4 to 2.6 ms).
__global__ __launch_bounds__(kSumBlock) void moments_many_kernel(const MomentsItem* items, const int32_t* flag)
{
    __shared__ MomentsShared<false> sh;
    const MomentsItem m = items[blockIdx.x];
    switch (m.W) {
#define SCA_ITEM(G) block_moments<G, false>(sh, 0, 1, m.S, m.h0, nullptr, nullptr, m.Y, m.W, m.nb, m.Y, nullptr, m.res, flag)
    case 1: SCA_ITEM(1); break;
    case 2: SCA_ITEM(2); break;
    case 4: SCA_ITEM(4); break;
    case 8: SCA_ITEM(8); break;
    case 16: SCA_ITEM(16); break;
    case 32: SCA_ITEM(32); break;
    default: SCA_ITEM(64); break;
#undef SCA_ITEM
    }
}

// ---------------------------------------------------------------- heights
constexpr int kColumn = 1024;

// Heights c(y) of column 0, and h(0,0) to h0_out (host memory).  Eight times
// 1024 rows at a time, row 1024 k + thread, so that the stores lie side by side
// and all loads of a round are in flight at once; the 128 wave sums are scanned
// by every wave for itself.  Bound by the lines one CU takes in, one per row of
// eight words or more: 8192 rows in 11.4 us (14.1 us with consecutive rows per
// thread).
__global__ __launch_bounds__(kColumn) void column_kernel(const uint64_t* S, const int64_t* h0, int64_t Y, int32_t W,
                                                         int64_t plane, int64_t* col, int64_t* h0_out)
{
    constexpr int K = 8, WAVES = kColumn / 64;
    static_assert(K * WAVES == 128, "two sums per lane");
    __shared__ int32_t sums[2][K * WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const uint64_t upto = (2ull << lane) - 1ull;  // this lane and those below
    int64_t c0 = *h0;
    int buf = 0;
    for (int64_t y0 = 0; y0 < Y; y0 += (int64_t)K * kColumn, buf ^= 1) {
        uint64_t w[K], ups[K], on[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int64_t y = y0 + k * kColumn + tid;
            w[k] = S[(2 + (tid & 1)) * plane + (y < Y ? y : (int64_t)(tid & 1)) * W];
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int64_t y = y0 + k * kColumn + tid;
            on[k] = __ballot(y < Y && y != 0);  // no step into row 0
            ups[k] = __ballot((w[k] & 1ull) != 0) & on[k];
            if (lane == 0) sums[buf][k * WAVES + wv] = 2 * __popcll(ups[k]) - __popcll(on[k]);
        }
        __syncthreads();
        const int32_t a = sums[buf][2 * lane], b = sums[buf][2 * lane + 1];
        const int32_t incl = group_incl_scan<64>(a + b, lane);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int i = k * WAVES + wv;  // sum i: the first or second of lane i / 2
            const int32_t before = __shfl((i & 1) ? incl - b : incl - a - b, i >> 1);
            const int64_t y = y0 + k * kColumn + tid;
            if (y < Y) col[y] = c0 + before + 2 * __popcll(ups[k] & upto) - __popcll(on[k] & upto);
        }
        c0 += __shfl(incl, 63);
    }
    if (tid == 0) *h0_out = *h0;
}

// Four heights of one store; the caller's buffer is aligned to an int32 only.
typedef int32_t Int4 __attribute__((ext_vector_type(4), aligned(4)));

// Heights of rows [y0, y0+ny), X >= 128.  A wave takes 64 consecutive words (of
// one row or of 64/G rows), parks them with the height in front of each in its
// part of LDS, and writes their 8192 sites as 32 stores of 64 lanes x four
// sites: every lane keeps its place within the word (chunk and half) in all of
// them, so the masks are loop-invariant, and gets its four heights from one
// table entry of running counts.  Bound by the write of 4 bytes per site.
template <int G>
__global__ __launch_bounds__(kBlock) void heights_kernel(const uint64_t* S, int64_t X, int32_t W, int64_t plane,
                                                         const int64_t* col, int64_t y0, int64_t ny, int32_t* out)
{
    __shared__ uint32_t lut[256];
    __shared__ uint64_t lE[kBlock], lO[kBlock];
    __shared__ int32_t lB[kBlock];
    const int lane = threadIdx.x & 63, gl = lane & (G - 1);
    const int first = threadIdx.x & ~63;  // LDS words of this wave
    lut[threadIdx.x] = running_counts(threadIdx.x);
    __syncthreads();
    const int64_t wave = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    const int64_t r0 = wave * (64 / G);
    if (r0 >= ny) return;
    const int64_t r_raw = r0 + lane / G;
    const int64_t y = y0 + (r_raw < ny ? r_raw : 0);
    const int64_t pe = (y & 1) * plane + y * W, po = (1 - (y & 1)) * plane + y * W;
    int32_t base = (int32_t)col[y] - (2 * (int32_t)(S[pe] & 1ull) - 1);
    const int j = (lane & 31) >> 1;  // this lane's chunk of eight sites within a word
    const uint32_t below = (1u << (4 * (j & 7))) - 1u;
    const uint32_t mlo = j < 8 ? below : ~0u, mhi = j < 8 ? 0u : below;
    const int64_t left = (ny - r0) * X;  // sites of this wave's rows
    for (int w0 = 0; w0 < W; w0 += G) {
        const uint64_t E = S[pe + w0 + gl], O = S[po + w0 + gl];
        const int32_t tot = 2 * (int32_t)(__popcll(E) + __popcll(O)) - 128;
        const int32_t incl = group_incl_scan<G>(tot, gl);
        lE[threadIdx.x] = E;
        lO[threadIdx.x] = O;
        lB[threadIdx.x] = base + incl - tot;
        if (w0 + G < W) base += __shfl(incl, 63);
        // the words are the wave's own: program order is enough
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        int32_t* const o = out + r0 * X + (int64_t)w0 * 128;
#pragma unroll 4
        for (int m = 0; m < 32; ++m) {
            const int e = first + 2 * m + (lane >> 5);
            const uint64_t we = lE[e], wo = lO[e];
            const uint32_t elo = (uint32_t)we, ehi = (uint32_t)(we >> 32), olo = (uint32_t)wo, ohi = (uint32_t)(wo >> 32);
            const int32_t ups = __popc(elo & mlo) + __popc(ehi & mhi) + __popc(olo & mlo) + __popc(ohi & mhi);
            const uint32_t eh = j < 8 ? elo : ehi, oh = j < 8 ? olo : ohi;
            const uint32_t byte = ((eh >> (4 * (j & 7))) & 15u) | (((oh >> (4 * (j & 7))) & 15u) << 4);
            const uint32_t c = lut[byte] >> (16 * (lane & 1));
            const int32_t h = lB[e] + 2 * ups - 8 * j - 4 * (lane & 1) - 1;
            const Int4 v = {h + 2 * (int32_t)(c & 15u), h - 1 + 2 * (int32_t)((c >> 4) & 15u),
                            h - 2 + 2 * (int32_t)((c >> 8) & 15u), h - 3 + 2 * (int32_t)((c >> 12) & 15u)};
            const int s = (m * 64 + lane) * 4;
            if (G == 64 || s < left) *reinterpret_cast<Int4*>(o + s) = v;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Heights of rows of less than 128 sites, one site per thread.
__global__ __launch_bounds__(kBlock) void heights_narrow_kernel(const uint64_t* S, int32_t lx, int64_t plane,
                                                               const int64_t* col, int64_t y0, int64_t sites,
                                                               int32_t* out)
{
    const int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (s >= sites) return;
    const int64_t y = y0 + (s >> lx);
    const int i = (int)(s & ((1 << lx) - 1));
    const uint64_t E = S[(y & 1) * plane + y], O = S[(1 - (y & 1)) * plane + y];
    const uint64_t me = (2ull << (i >> 1)) - 1ull, mo = (1ull << ((i + 1) >> 1)) - 1ull;  // sites 0 .. i, i < 64
    const int32_t ups = __popcll(E & me) + __popcll(O & mo) - (int32_t)(E & 1ull);
    out[s] = (int32_t)col[y] + 2 * ups - i;
}

template <bool TWO>
hipError_t launch_moments_g(const uint64_t* S, const int64_t* h0, const uint64_t* snap, const int64_t* snap_h0,
                            int64_t Y, int32_t W, int32_t nb, int32_t R, int64_t* partials, int64_t* res,
                            const int32_t* flag, hipStream_t stream)
{
    const dim3 grid((unsigned)(Y / R)), block(kSumBlock);
    switch (W) {
#define SCA_ROWS(G)                                                                                             \
    hipLaunchKernelGGL((moments_kernel<G, TWO>), grid, block, 0, stream, S, h0, snap, snap_h0, Y, W, nb, R, partials, \
                       res, flag)
    case 1: SCA_ROWS(1); break;
    case 2: SCA_ROWS(2); break;
    case 4: SCA_ROWS(4); break;
    case 8: SCA_ROWS(8); break;
    case 16: SCA_ROWS(16); break;
    case 32: SCA_ROWS(32); break;
    default: SCA_ROWS(64); break;
#undef SCA_ROWS
    }
    return hipGetLastError();
}

template <int G>
hipError_t launch_heights_g(const uint64_t* S, int64_t X, int32_t W, int64_t plane, const int64_t* col, int64_t y0,
                            int64_t ny, int32_t* out, hipStream_t stream)
{
    const int64_t rows_per_block = (kBlock / 64) * (64 / G);
    hipLaunchKernelGGL((heights_kernel<G>), dim3((unsigned)((ny + rows_per_block - 1) / rows_per_block)),
                       dim3(kBlock), 0, stream, S, X, W, plane, col, y0, ny, out);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_flat_init(uint64_t* S, int64_t Y, int32_t W, int32_t nb, int64_t* h0, hipStream_t stream)
{
    const int64_t plane = Y * W;
    const uint64_t valid = (nb == 64) ? ~0ull : ((1ull << nb) - 1ull);
    int64_t blocks = (4 * plane + kBlock - 1) / kBlock;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(flat_init_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, stream, S, plane, valid, h0);
    return hipGetLastError();
}

FlatItem flat_item(uint64_t* S, int64_t Y, int32_t W, int32_t nb, int64_t* h0)
{
    return FlatItem{S, h0, Y * W, (nb == 64) ? ~0ull : ((1ull << nb) - 1ull)};
}

hipError_t launch_flat_init_many(const FlatItem* items_dev, int32_t n, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    const int32_t grid = n < 4096 ? n : 4096;
    hipLaunchKernelGGL(flat_init_many_kernel, dim3((unsigned)grid, 8), dim3(kBlock), 0, stream, items_dev, n);
    return hipGetLastError();
}

hipError_t launch_flat_init_few(const FlatItem* items_host, int32_t n, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    if (n > kFlatFew) return hipErrorInvalidValue;
    FlatFew f{};
    for (int32_t i = 0; i < n; ++i) f.items[i] = items_host[i];
    hipLaunchKernelGGL(flat_init_few_kernel, dim3((unsigned)n, 8), dim3(kBlock), 0, stream, f);
    return hipGetLastError();
}

// Rows per block: the whole lattice in one block of up to two words per
// thread (2^10 x 2^9, four words per thread, took 13 us so), else 256 blocks,
// or fewer where that would leave waves of a block without rows.
static int32_t moments_rows(int64_t Y, int32_t W)
{
    if (Y <= kSumRows && Y * W <= 2 * kSumBlock) return (int32_t)Y;
    const int64_t sweep = (int64_t)kSumBlock / (W < 64 ? W : 64);  // rows the 16 waves take at once
    int64_t R = Y / kCombine > sweep ? Y / kCombine : sweep;
    if (R > kSumRows) R = kSumRows;
    return (int32_t)(R < Y ? R : Y);
}

hipError_t launch_moments(const uint64_t* S, const int64_t* h0, const uint64_t* snap, const int64_t* snap_h0,
                          int64_t X, int64_t Y, int32_t W, int32_t nb, int64_t* partials, int64_t* res,
                          const int32_t* flag, hipStream_t stream)
{
    const int32_t R = moments_rows(Y, W);
    const hipError_t e =
        snap ? launch_moments_g<true>(S, h0, snap, snap_h0, Y, W, nb, R, partials, res, flag, stream)
             : launch_moments_g<false>(S, h0, snap, snap_h0, Y, W, nb, R, partials, res, flag, stream);
    if (e != hipSuccess || R == Y) return e;
    hipLaunchKernelGGL(combine_kernel, dim3(1), dim3(kCombine), 0, stream, h0, snap_h0, snap != nullptr, partials,
                       (int32_t)(Y / R), X * (int64_t)R, res, flag);
    return hipGetLastError();
}

bool moments_in_one_block(int64_t Y, int32_t W) { return moments_rows(Y, W) == Y; }

hipError_t launch_moments_many(const MomentsItem* items, int32_t n, const int32_t* flag, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(moments_many_kernel, dim3((unsigned)n), dim3(kSumBlock), 0, stream, items, flag);
    return hipGetLastError();
}

hipError_t launch_column(const uint64_t* S, const int64_t* h0, int64_t Y, int32_t W, int64_t* col, int64_t* h0_out,
                         hipStream_t stream)
{
    hipLaunchKernelGGL(column_kernel, dim3(1), dim3(kColumn), 0, stream, S, h0, Y, W, Y * (int64_t)W, col, h0_out);
    return hipGetLastError();
}

hipError_t launch_heights(const uint64_t* S, int64_t X, int64_t Y, int32_t W, const int64_t* col, int64_t y0,
                          int64_t ny, int32_t* out, hipStream_t stream)
{
    const int64_t plane = Y * W;
    if (X < 128) {
        const int64_t sites = ny * X;
        hipLaunchKernelGGL(heights_narrow_kernel, dim3((unsigned)((sites + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                           stream, S, __builtin_ctzll((uint64_t)X), plane, col, y0, sites, out);
        return hipGetLastError();
    }
    switch (W) {
    case 1: return launch_heights_g<1>(S, X, W, plane, col, y0, ny, out, stream);
    case 2: return launch_heights_g<2>(S, X, W, plane, col, y0, ny, out, stream);
    case 4: return launch_heights_g<4>(S, X, W, plane, col, y0, ny, out, stream);
    case 8: return launch_heights_g<8>(S, X, W, plane, col, y0, ny, out, stream);
    case 16: return launch_heights_g<16>(S, X, W, plane, col, y0, ny, out, stream);
    case 32: return launch_heights_g<32>(S, X, W, plane, col, y0, ny, out, stream);
    default: return launch_heights_g<64>(S, X, W, plane, col, y0, ny, out, stream);
    }
}

}  // namespace sca
