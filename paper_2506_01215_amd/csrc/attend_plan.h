// How the bf16 forward pass of a problem is cut into workgroups.  Plain integer arithmetic without a device
// type, shared by the launcher, the kernels and a host program that replays it; P is AttnParams, or has
// its fields Hkv, G, D, M, Ct, n_row_blocks, by_head, shares, start, tiles and part_rows.  Sizes reach
// 2^30 keys and 2^31 query rows, so no product of keys and heads may be formed in 32 bits.
#pragma once

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define RF_PLAN __host__ __device__ __forceinline__
#else
#define RF_PLAN inline
#endif

namespace reform {

constexpr int kFwdWaves = 8;
constexpr int kFwdRows = kFwdWaves * 32;                       // query rows of a row block

// Key tiles of row block rb (64-key tiles up to the last key its last row sees): (M + (last row) / G) / 64 + 1.
template <class P>
RF_PLAN int fwd_row_block_tiles(const P &p, int rb)
{
    const int rows = p.G * p.Ct;
    const int last = (rb + 1 < p.n_row_blocks ? (rb + 1) * kFwdRows : rows) - 1;
    return (p.M + last / p.G) / 64 + 1;
}

// Share j holds the places [fwd_share_begin(j), fwd_share_begin(j + 1)) of the list.
template <class P>
RF_PLAN int fwd_share_begin(const P &p, int j) { return (int)((unsigned)j * (unsigned)p.tiles / (unsigned)p.shares); }

// Walks a KV head's list row block by row block without dividing: for a full row block the number of tiles is
// (a + rows / 64 * rb) / G + 1 with a = (M G + rows - 1) / 64, rows = kFwdRows being a multiple of 64; q
// and r are quotient and remainder of a + rows / 64 * rb by G.  M G itself may not fit 32 bits (32 heads
// over 2^26 keys): with M = 64 m + k, a = m G + (k G + rows - 1) / 64.
template <class P>
struct FwdWalk {
    int rb, pos, nt;                                     // row block, list position of its first tile, its tiles
    int q, r;

    RF_PLAN int count(const P &p) const
    {
        return rb + 1 < p.n_row_blocks ? q + 1 : (p.M + p.Ct - 1) / 64 + 1;
    }
    RF_PLAN explicit FwdWalk(const P &p) : rb(0), pos(p.start)
    {
        // 63 G fits: a split problem has at most four row blocks per compute unit, so G < 2^20
        const int a = (p.M % 64 * p.G + kFwdRows - 1) / 64;
        q = p.M / 64 + a / p.G;
        r = a % p.G;
        nt = count(p);
    }
    RF_PLAN void next(const P &p)
    {
        pos += nt + p.start;
        ++rb;
        for (r += kFwdRows / 64; r >= p.G; r -= p.G) ++q;
        nt = count(p);
    }
};

// Slot of the partial result of share j's tiles [t0, t1) of a row block of nt tiles, or -1 where the share covers
// the row block alone.  A share leaves at most two pieces: the end of a row block it begins in (slot 0
// of its two), and the beginning of the one it ends in (slot 1).
template <class P>
RF_PLAN long fwd_slot(const P &p, int j, int kvh, int t0, int t1, int nt)
{
    return t0 == 0 && t1 == nt ? -1 : (long)(j * p.Hkv + kvh) * 2 + (t0 == 0 ? 1 : 0);
}

// The pieces of the row block whose nt tiles begin at list position pos: those of the shares j0 .. j1.
template <class P>
struct FwdPieces {
    int j0, j1;
    bool begins;                                         // it begins inside share j0 (or with it)

    RF_PLAN FwdPieces(const P &p, int pos, int nt)
    {
        const unsigned T = p.tiles, S = p.shares;
        j0 = (int)(((unsigned)(pos + 1) * S - 1) / T);
        j1 = (int)(((unsigned)(pos + nt) * S - 1) / T);
        begins = fwd_share_begin(p, j0) <= pos;
    }
    RF_PLAN long slot(const P &p, int j, int kvh) const
    {
        return (long)(j * p.Hkv + kvh) * 2 + (begins && j == j0 ? 1 : 0);
    }
};

// How the forward pass of a problem is cut into workgroups: n_row_blocks and, if the key range is to be
// split, shares, tiles and part_rows.
template <class P>
inline void fwd_plan(P &p, int cus)
{
    const int rows = p.G * p.Ct;
    p.n_row_blocks = (int)(((long)rows + kFwdRows - 1) / kFwdRows);
    p.shares = 0;
    p.part_rows = rows < kFwdRows ? rows : kFwdRows;
    // Waves of one head are 0.6 % to 1.3 % faster where they are full (8192 rows over 8192 keys, 32768 over
    // 32768, 32/8 heads); with few chunk rows they would be nearly empty (one token: 20.6 instead of 18.3 us).
    p.by_head = kFwdWaves % p.G == 0 && p.Ct >= 32;
    const long whole = (long)p.Hkv * p.n_row_blocks;
    if (whole > 4l * cus || p.Hkv > cus) return;         // at least four well-filled rounds
    const long longest = (p.M + p.Ct - 1) / 64 + 1;
    p.start = p.n_row_blocks > 1 ? 4 : 0;
    long tiles = 0;
    for (int rb = 0; rb < p.n_row_blocks; ++rb) tiles += p.start + fwd_row_block_tiles(p, rb);
    // Time of either form, in key tiles of one workgroup (1.45 us at head_dim 128, 1.1 us at 64; one
    // workgroup is resident per compute unit).  Only ratios decide, and of these only the launches' would differ
    // (4 tiles are 5.8 us at 128 and 4.4 us at 64), so one set of constants serves both.  Whole row blocks run in rounds.  Equal shares pay the
    // launch that merges them and the partial results, written and read back, which grow with their
    // size, with the number of shares, and double where a share can begin and end inside row blocks.
    // Fitted to (us; whole, then with the number of shares per KV head): 60 rows over 8000 keys, 32/8
    // heads 183, 38 (8), 29 (16), 26 (32); 300 over 1500, 24/8 heads 48, 45 (8), 37 (13), 43 (32); 2000
    // over 4000, 8 heads 138, 95 (13), 66 (24), 61 (32); 60 over 8000, 14/2 heads, head_dim 64 136, 28
    // (16), 18.6 (64), 20.6 (128).  One token over 16640 keys (32/8 heads) 290 -> 18 us.
    const double rounds = (double)((whole + cus - 1) / cus);
    double best = whole <= cus ? 4.0 + (double)longest : rounds * (double)tiles * p.Hkv / (double)whole;
    const double slot = p.part_rows * p.D / (256.0 * 128.0) * (p.n_row_blocks > 1 ? 2.0 : 1.0);
    long shares = 0;
    for (long s = tiles / 2 < cus / p.Hkv ? tiles / 2 : cus / p.Hkv; s >= 2; s -= (s + 7) / 8) {
        const double t = (double)tiles / s + 4.0 + slot * (4.5 + 5.5 * (double)s * p.Hkv / cus);
        if (t < best) { best = t; shares = s; }
    }
    if (!shares || tiles * (shares + 1) >= (1l << 31)) return;
    p.shares = (int)shares;
    p.tiles = (int)tiles;
}

}  // namespace reform
