// How the bf16 forward pass and the score pass of a problem are cut into workgroups.  Plain arithmetic without a
// device type, shared by the launcher, the kernels and a host program that replays it; P is AttnParams, or
// has its fields Hkv, G, D, M, Ct, n, W, n_row_blocks, by_head, narrow, shares, start, tiles and part_rows, and for
// the score slices, slice_tiles, head_slices and slice_heads.  Sizes reach 2^30 keys and 2^31 query rows,
// so no product of keys and heads may be formed in 32 bits.
#pragma once

#include <limits.h>
#include <stddef.h>

#include <algorithm>

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define RF_PLAN __host__ __device__ __forceinline__
#else
#define RF_PLAN inline
#endif

namespace reform {

constexpr int kFwdWaves = 8;
constexpr int kFwdRows = kFwdWaves * 32;                       // query rows of a row block
constexpr int kFwdNarrowRows = 128;                            // those of the narrow form, four waves
template <int D> constexpr int kFwdNarrowResident = D == 64 ? 3 : 2;   // its workgroups on a compute unit

// Key tiles of row block rb (64-key tiles up to the last key its last row sees): (M + (last row) / G) / 64 + 1.
template <int ROWS = kFwdRows, class P>
RF_PLAN int fwd_row_block_tiles(const P &p, int rb)
{
    const int rows = p.G * p.Ct;
    const int last = (rb + 1 < p.n_row_blocks ? (rb + 1) * ROWS : rows) - 1;
    return (p.M + last / p.G) / 64 + 1;
}

// Share j holds the places [fwd_share_begin(j), fwd_share_begin(j + 1)) of the list.
template <class P>
RF_PLAN int fwd_share_begin(const P &p, int j) { return (int)((unsigned)j * (unsigned)p.tiles / (unsigned)p.shares); }

// Walks a KV head's list row block by row block without dividing: for a full row block the number of tiles is
// (a + rows / 64 * rb) / G + 1 with a = (M G + rows - 1) / 64, rows = ROWS being a multiple of 64; q
// and r are quotient and remainder of a + rows / 64 * rb by G.  M G itself may not fit 32 bits (32 heads
// over 2^26 keys): with M = 64 m + k, a = m G + (k G + rows - 1) / 64.
template <class P, int ROWS = kFwdRows>
struct FwdWalk {
    int rb, pos, nt;                                     // row block, list position of its first tile, its tiles
    int q, r;

    RF_PLAN int count(const P &p) const
    {
        return rb + 1 < p.n_row_blocks ? q + 1 : (p.M + p.Ct - 1) / 64 + 1;
    }
    RF_PLAN explicit FwdWalk(const P &p) : rb(0), pos(p.start)
    {
        // 63 G fits: a split problem has at most eight row blocks of 128 per compute unit, so G < 2^20
        const int a = (p.M % 64 * p.G + ROWS - 1) / 64;
        q = p.M / 64 + a / p.G;
        r = a % p.G;
        nt = count(p);
    }
    RF_PLAN void next(const P &p)
    {
        pos += nt + p.start;
        ++rb;
        for (r += ROWS / 64; r >= p.G; r -= p.G) ++q;
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

template <class P>
inline bool merge_with_score(const P &p, double *gain = nullptr);

// What the parts of a forward pass cost, in us on 256 compute units; fitted to 2900 timings of 143 problems of 8 to 5000
// rows over up to 37000 keys, with 32/8, 24/8, 16/4, 14/2 and 8/8 heads, each whole and with 7 to 12 numbers of shares: the
// fits miss by 3 to 6 % in the mean there.  Of 97 larger problems at 128, more than one round of row blocks, they fall short by
// 9 % whole and 12 % in shares, of 123 at 64 by 4 % and 2 %.  A key tile's time depends on how many workgroups share its compute
// unit.  (Three at 64: 1.47 in that fit, in which few problems have as many; 8 % too much for the 123.)
struct FwdCost {
    int resident;                                        // workgroups on a compute unit
    double whole, whole_begin, whole_tile[3];            // a launch; the start of a row block, in tiles; a tile with 1, 2, 3 on the unit
    double split, split_begin, split_tile[3], write, part;   // the same where keys are shared out; a MB of partial results; a whole slot of them
};
template <int ROWS>
inline FwdCost fwd_cost(int D)
{
    if (ROWS == kFwdRows)
        return D == 64 ? FwdCost{1, 2.0, 5.2, {1.02, 1.02, 1.02}, 8.6, 3.3, {1.07, 1.07, 1.07}, 0.52, 1.34}
                       : FwdCost{1, 3.0, 3.4, {1.46, 1.46, 1.46}, 7.5, 3.4, {1.46, 1.46, 1.46}, 0.36, 4.0};
    return D == 64 ? FwdCost{3, 5.3, 0.0, {0.78, 0.98, 1.35}, 9.6, 2.9, {0.88, 1.20, 1.75}, 0.49, 0.0}
                   : FwdCost{2, 3.1, 3.2, {1.19, 1.61, 1.66}, 8.8, 1.7, {1.29, 1.77, 1.77}, 0.46, 0.64};
}

// Bytes of the partial results of a planned forward pass: two slots to every share, fp32 sums, maximum and sum of each row.
template <class P>
inline size_t fwd_split_bytes(const P &p)
{
    return (size_t)p.shares * p.Hkv * 2 * p.part_rows * (p.D + 2) * sizeof(float);
}

// How the forward pass of a problem is cut into workgroups of ROWS query rows: n_row_blocks and, if the key range is to be
// split, shares, tiles and part_rows.  Returns the time estimated for it (0: whole row blocks, of which there are enough).
// scored: the call forms the score as well, so that the launch which merges shares may be the score's.
// scratch: bytes there are for partial results; the numbers of shares that fit are considered.
template <int ROWS = kFwdRows, class P>
inline double fwd_plan(P &p, int cus, bool scored = true, size_t scratch = (size_t)-1)
{
    const int rows = p.G * p.Ct;
    p.n_row_blocks = (int)(((long)rows + ROWS - 1) / ROWS);
    p.shares = 0;
    p.part_rows = rows < ROWS ? rows : ROWS;
    // Waves of one head are 0.6 % to 1.3 % faster where they are full (8192 rows over 8192 keys, 32768 over
    // 32768, 32/8 heads); with few chunk rows they would be nearly empty (one token: 20.6 instead of 18.3 us).
    p.by_head = ROWS / 32 % p.G == 0 && p.Ct >= 32;
    const long whole = (long)p.Hkv * p.n_row_blocks;
    const FwdCost cost = fwd_cost<ROWS>(p.D);
    if (whole > 4l * cus * kFwdRows / ROWS || p.Hkv > cus) return 0.0;   // at least four well-filled rounds
    p.start = p.n_row_blocks == 1 ? 0 : ROWS == kFwdRows ? 4 : 3;
    long tiles = 0;
    for (int rb = 0; rb < p.n_row_blocks; ++rb) tiles += p.start + fwd_row_block_tiles<ROWS>(p, rb);
    const long pure = tiles - (long)p.start * p.n_row_blocks;
    p.shares = 1;
    const size_t room = scratch / fwd_split_bytes(p);
    // a place in the list times the shares is formed in 32 bits
    const long most = std::min({tiles / 2, (long)cost.resident * cus / p.Hkv, INT_MAX / tiles - 1,
                                (long)std::min(room, (size_t)INT_MAX)});
    long shares = 0;
    double best;
    if (rows <= 16) {
        // attn_fwd_few, in key tiles: one token over 16640 keys (32/8 heads) 290 us whole, 18 us with 32 shares
        best = 4.0 + (double)((p.M + p.Ct - 1) / 64 + 1);
        const double slot = p.part_rows * p.D / (256.0 * 128.0);
        for (long s = most; s >= 2; s -= (s + 7) / 8) {
            const double t = (double)tiles / s + 4.0 + slot * (4.5 + 5.5 * (double)s * p.Hkv / cus);
            if (t < best) { best = t; shares = s; }
        }
    } else {
        // Whole row blocks, the longest first.  With one workgroup on a unit every second round pairs its longest with the
        // shortest of the round before; with several, the units fill up in that order and their tiles slow down.
        auto length = [&](long i) {
            return i < whole ? cost.whole_begin + fwd_row_block_tiles<ROWS>(p, p.n_row_blocks - 1 - (int)(i / p.Hkv)) : 0.0;
        };
        if (cost.resident == 1) {
            double t = 0.0;
            for (long r = 0; r < whole; r += 2l * cus) t += r + cus < whole ? 2.0 * length(r + cus) : length(r);
            best = cost.whole + cost.whole_tile[0] * (t < length(0) ? length(0) : t);
        } else {
            double t = 0.0;
            for (int r = 0; r < cost.resident; ++r)
                t += (cost.whole_tile[r] - (r ? cost.whole_tile[r - 1] : 0.0)) * length((long)r * cus);
            const double all = (pure + cost.whole_begin * p.n_row_blocks) * p.Hkv / cus / cost.resident;
            const double behind = cost.whole_tile[cost.resident - 1] * (all + 0.5 * length((long)cost.resident * cus));
            best = cost.whole + (whole > (long)cost.resident * cus && t < behind ? behind : t);
        }
        // Equal shares pay the launch that merges them and the partial results, written and read back, which double where
        // a share begins and ends inside row blocks.  They read K and V each at a place of its own, while whole row blocks
        // walk the same keys and find them in the L2; with more than one round of these that shows beyond the estimates at 128
        // (11419 rows, 16/4 heads 464 us whole, 485 with 64 shares).  Of 97 problems of eight waves at 128 and 123 at 64, timed in
        // both ways, a choice by the estimates takes 0.5 % and 0.2 % more than the faster way, at worst 7 % and 4 %; with the
        // whole blocks' times 0.94 0.05 % and 0.9 %, at worst 3 % and 13 % (12040 rows, 8/8 heads of 64 188 us in shares, 205 whole).
        const double whole_time = best;
        if (whole > cus && (p.D == 128 || ROWS != kFwdRows)) best *= 0.94;
        // (pieces of one row block are merged sooner: 132 rows over 5890 keys, 8/8 heads 20.8 us with 32 shares, 21.6 with 28)
        const double mb = p.part_rows * p.D * (p.n_row_blocks == 1 ? 3e-6 : 4e-6), full = p.part_rows * p.D / (256.0 * 128.0);
        for (long s = most; s >= 2; s -= (s + 7) / 8) {
            p.shares = (int)s;
            const double cut = p.n_row_blocks > s ? 1.0 : (p.n_row_blocks - 1.0) / s;
            const int on_unit = (int)((s * p.Hkv - 1) / cus);
            p.tiles = (int)tiles;
            double launch = 0.0;
            if (scored) merge_with_score(p, &launch);
            const double t = cost.split - launch + cost.split_tile[on_unit] * (pure + cost.split_begin * p.n_row_blocks) / s +
                             cost.write * mb * s * p.Hkv * (1.0 + cut) + cost.part * full;
            if (t < best) { best = t; shares = s; }
        }
        if (!shares) best = whole_time;
    }
    p.shares = (int)shares;
    p.tiles = (int)tiles;
    return best;
}

// Which form the forward pass takes.  Workgroups of four waves and 128 rows start sooner, wait for fewer waves at a barrier,
// leave less of a row block empty, and two of them (three at head_dim 64) overlap on a compute unit; but alone on it one
// reaches 0.6 of the rate, and each stages K and V for half the rows, so passes that fill the chip for long
// stay with eight waves.  us, eight / four, each with its best number of shares: 312 rows over 312 keys, 32/8 heads 16.2 /
// 12.1; 1998 over 1998 55.8 / 50.5; 1269 over 1808 48.9 / 45.5; 223 over 1518, 14/2 24.4 / 21.3; 78 over 8020, 16/4 27.4 /
// 23.2; 185 over 2775, 32/8 29.3 / 30.2; 1354 over 2834, 16/4 45.2 / 48.6; 335 over 12938, 32/8 82.9 / 96.6; 64 wide: 907 over
// 1423, 32/8 30.6 / 24.0; 4907 over 4907 131 / 115; 1767 over 1767, 24/8 34.6 / 29.2; 2592 over 14640, 8/8 96.4 / 98.5.
template <class P>
inline double fwd_choose_within(P &p, int cus, bool scored, size_t scratch)
{
    const double eight = fwd_plan(p, cus, scored, scratch);
    p.narrow = 0;
    if (eight == 0.0 || p.G * p.Ct <= 16) return eight;
    // Shares have to promise more: estimated 4 % ahead, 326 rows over 23729 keys, 8/8 heads take 62.7 us, not 53.2.  One row
    // block of many keys is bound by reading them, with half the loads in flight (96 over 30179, 8/8 29.7 us, with four 36.6).
    P q = p;
    const double four = fwd_plan<kFwdNarrowRows>(q, cus, scored, scratch);
    if (four >= (q.shares ? 0.95 : 0.98) * eight || (q.n_row_blocks == 1 && q.shares)) return eight;
    // Long shares are bound by what the estimate leaves out: every row block reads its K and V by itself, and there are up to
    // twice as many.  Problems for which the estimate is for shared-out four waves, time with four over that with eight (mean,
    // worst) by the tiles of a share, at 128: up to 7 0.88, 1.07 (660 problems); 7 to 9 0.94, 1.08 (121); 9 to 12 0.98, 1.10
    // (47); 12 to 18 1.07, 1.16 (15); beyond 1.18, 1.28 (26; 379 rows over 52252 keys, 8/8 heads 98.2 us, with four 115.0).  At 64,
    // with half the bytes, 0.90 with eight KV heads, 0.95 with four, 0.99 with two beyond 9 tiles, at worst 1.07.
    if (p.D == 128 && q.shares && q.tiles / q.shares >= 9) return eight;
    p = q;
    p.narrow = 1;
    return four;
}

// scratch: bytes there are for partial results.  What the plan wants of them does not depend on how much more there is.
// Returns the estimate of the plan that is made.
template <class P>
inline double fwd_choose(P &p, int cus, bool scored, size_t scratch = (size_t)-1)
{
    const double est = fwd_choose_within(p, cus, scored, (size_t)-1);
    return fwd_split_bytes(p) > scratch ? fwd_choose_within(p, cus, scored, scratch) : est;
}

constexpr int kFwdShortRows = 32;                        // query rows of a workgroup of attn_fwd_short

// 32-key tiles of row block rb of attn_fwd_short, up to the last key its last row sees.
template <class P>
RF_PLAN int fwd_short_tiles(const P &p, int rb)
{
    const int rows = p.G * p.Ct, end = (rb + 1) * kFwdShortRows;
    return (p.M + ((end < rows ? end : rows) - 1) / p.G) / 32 + 1;
}

// Of `tiles` share j holds [fwd_short_begin(j), fwd_short_begin(j + 1)).
template <class P>
RF_PLAN int fwd_short_begin(const P &p, int tiles, int j) { return (int)((long)tiles * j / p.shares); }

// The pieces of row block rb where attn_fwd_short's key tiles are shared out: each block's own, in equal parts.
template <class P>
struct ShortPieces {
    int j0, j1, rb;

    RF_PLAN ShortPieces(const P &p, int block) : j0(0), j1(p.shares - 1), rb(block) {}
    RF_PLAN long slot(const P &p, int j, int kvh) const { return ((long)rb * p.shares + j) * p.Hkv + kvh; }
};

// Bytes of the pieces of attn_fwd_short where its key tiles are shared out.
template <class P>
inline size_t fwd_short_bytes(const P &p)
{
    return p.shares ? (size_t)p.n_row_blocks * p.shares * p.Hkv * kFwdShortRows * (p.D + 2) * sizeof(float) : 0;
}

// Whether a forward pass is formed by attn_fwd_short instead of its plan, which is estimated at est us: the waves of a
// workgroup of that form (0: not; the plan stays), with n_row_blocks and, where every row block's key tiles are shared out
// over several workgroups, shares, part_rows and tiles.  Eight waves where every workgroup has a compute unit, else four, two
// workgroups to a unit (three at 64).  Time goes by 32-key tiles:
//   - With a unit to every workgroup by those of the longest, and 0.1 us a MB of K and V beyond 20, which the L2s of few row blocks
//     do not hold (76 rows over 7673 keys, 40/40 heads of 64 26.2 us by the plan, 35.2 so).  Fitted to 220 timings of 110
//     problems, mean error 3 to 4 %, and taken at less than 0.88 of the plan's estimate, or 0.84 where the score's launch merges the
//     plan's pieces at 128, since the form saves less there (20 rows over 2539 keys, 20/5 heads, 20 observing, whole calls 18.2, 19.1).  Of
//     4800 problems of 5 to 1500 rows over up to 30000 keys that the fit has not seen, with and without score, 3090 take this
//     form or the shares below, 0.81 of the plan's time in the mean, 20 more than 2 % longer, 2 more than 5 %, at worst 6 %.
//   - Beyond by the longest workgroup of each round of one to a unit, since just above one (two, three) to a unit some hold one
//     more than the mean: 206 rows over 5715 keys, 40/8 heads of 64 (1.03 to a unit) 29.1 us by the plan, 38.5 so; 418 over 1901,
//     40/8 of 128 (2.06) 34.2, 39.7.  The third round begins behind one of the first two.  Fitted to 1500 timings of 17 to 6700
//     rows over up to 23000 keys, standard error 4 to 5 %.  Of 1507 others of 116 to 25000 rows over up to 29000 keys, a choice
//     by estimates of less than 0.9 of the plan's takes 0.877 of the plans' time in the mean (the faster way of each 0.874), 28 more than
//     2 % longer, 11 more than 5 %, at worst 13 % (1471 over 2145, 16/16 of 128 37.9, 42.8); by a unit's mean load 0.883, 104, 68, 32 %.
//   - Shares pay their merge, 3 us (less with the score's launch, see merge_with_score), and need a tile for every wave.
//   - K and V have to come from memory once at least, and longer ones than an XCD's L2 holds come oftener: 23 rows over 26798
//     keys, 24/8 heads of 128 30.1 us by the plan, 35.3 so.  There row blocks that walk the same keys also have to meet on an
//     XCD, so shares come in multiples of what brings the next block back to it, or up to 3.8 MB of K and V a head less than one (109
//     rows over 24245 keys, 9/3 heads of 128 34.6 us by the plan, 53.0 with seven shares; 384 over 5971, 6/3, 3.1 MB 41.6, 38.9 with three).
//     Beyond 72 MB of K and V nothing is gained: 44 problems at 64 take 0.99 of the plan's time in the mean, at worst 1.04 (52 rows over
//     320718 keys, 5/1 heads 49.7 us by the plan, 51.7 so); 62 of 54 to 72 MB 0.93, below less; none at 128 is taken there.
//   - With a key tile or two of the plans and rows for one to three waves the estimates say too little for this form, whose waves
//     but one are idle and meet all the same.  Forward pass traced, us, plan / this: 8 rows over 8 keys, 32/8 heads of 128 5.6 / 6.6,
//     14/2 5.4 / 6.1, of 64 4.4 / 4.6; 20 over 20, 24/8 of 128 6.0 / 6.6, 14/2 (140 rows to a head) 7.0 / 6.6; 8 over 98, 32/8 of 128
//     6.5 / 7.0, 14/2 6.5 / 6.3; at 64 60 rows to a head over 20 5.1 / 5.0, 80 5.3 / 5.1.
// scratch: bytes there are for pieces.
template <class P>
inline int fwd_short(P &p, int cus, double est, bool scored, size_t scratch = (size_t)-1)
{
    const long rows = (long)p.G * p.Ct, blocks = (rows + kFwdShortRows - 1) / kFwdShortRows, groups = blocks * p.Hkv;
    if (rows <= 16 || est == 0.0 || groups > 4l * cus) return 0;
    if (p.n <= 64 && rows <= (p.D == 64 ? 64 : 96)) return 0;
    if (p.n <= 128 && rows <= 32 && p.D == 128) return 0;
    const double longest = (p.M + p.Ct - 1) / 32 + 1, first = p.M / 32 + 1;
    const double mb = 4e-6 * p.Hkv * (double)p.n * p.D;
    double best = (p.D == 64 ? 5.25 + 0.095 * longest : 6.5 + 0.195 * longest) + std::max(0.0, 0.1 * (mb - 20.0));
    if (groups > cus) {
        auto length = [&](long i) {                      // key tiles of the i-th workgroup
            const long end = std::min((blocks - i / p.Hkv) * kFwdShortRows, rows);
            return i < groups ? (double)((p.M + (end - 1) / p.G) / 32 + 1) : 0.0;
        };
        const double l1 = length(cus), l2 = length(2l * cus), l3 = length(3l * cus);
        best = p.D == 64 ? 4.6 + 0.15 * longest + 0.045 * l1 : 7.25 + 0.21 * longest + 0.13 * l1;
        if (l2 > 0.0)
            best = p.D == 64 ? std::max(best + 0.8, 6.8 + 0.165 * l1 + 0.1 * l2 + 0.15 * l3)
                             : std::max(best + 0.1, 12.65 + 0.3 * l1 + 0.285 * l2 + 0.11 * l3);
    }
    P q = p;
    q.n_row_blocks = (int)blocks;
    q.part_rows = kFwdShortRows;
    q.tiles = (p.M + p.Ct - 1) / 64 + 1;                 // of the longest row block, in the unit of the plans
    long shares = 0, step = 1;
    if (blocks > 1 && p.n * 4.0 * p.D > 3e6) while (step * p.Hkv % 8) step *= 2;
    const double stream = 7.0 + 0.29 * mb;
    for (long s = 2; mb <= 72.0 && s * groups <= cus && 8 * s <= (long)first; ++s) {
        if (s % step && (s > step || p.n * 4.0 * p.D > 3.8e6)) continue;
        q.shares = (int)s;
        if (fwd_short_bytes(q) > scratch) break;
        double launch = 0.0;
        if (scored) merge_with_score(q, &launch);
        const double t = std::max(p.D == 64 ? 5.25 + 0.095 * longest / s : 6.5 + 0.195 * longest / s, stream) + 3.0 + 0.05 * s - launch;
        if (t < best) { best = t; shares = s; }
    }
    const bool merged = p.D == 128 && scored && p.shares && merge_with_score(p);
    if (best >= (groups > cus ? 0.9 : merged ? 0.84 : 0.88) * est) return 0;
    q.shares = (int)shares;
    p = q;
    return groups <= cus ? 8 : 4;
}

// ------------------------------------------------------------------------------------------
// Forms of the tiled score pass (see attn_score_bf16): waves of a workgroup and keys of a wave.
constexpr int kScoreEight = 8;                           // eight waves of 64 keys
constexpr int kScoreFour = 4;                            // four of 64
constexpr int kScoreNarrow = 2;                          // four of 32

// Bytes of the slices' sums of a planned score pass.
template <class P>
inline size_t score_slice_bytes(const P &p) { return p.slices > 1 ? (size_t)p.slices * p.Hkv * p.n * sizeof(float) : 0; }

// How the score pass of a problem is cut into workgroups: form (returned), slices, slice_tiles, head_slices and
// slice_heads.  Time is estimated in query tiles that a compute unit takes against 512 keys (2.1 us at head_dim 128,
// 1.35 us at 64); two workgroups of four waves of 64 keys, three of 32 (four at head_dim 64) or one of eight are resident on it.
//   - Eight waves, uncut: the fewest Q bytes per key, the best form where its workgroups fill the chip
//     evenly.  Keys of the cache (and of the chunk before the window) cost the same each; those of
//     the window itself are triangular and fill up what the others leave.  Each round of them begins anew (8 us at 128).
//   - Four waves, cut: half or a quarter of the keys and 1/slices of the rows per workgroup, at the price of a start-up
//     of about 1.5 tiles each and of a launch that adds the slices up (2 tiles, 3 of the narrow form's).
//   - Which four-wave form: a workgroup of the narrow one starts and ends sooner, and with three or four on a compute unit
//     one's start and loads lie under the others' work; a long pass is bound by the power budget, and there twice the reads
//     of Q per key cost 5 %.  At 64 a pass is bound by its VALU work, and of the four-wave forms the
//     narrow one is the faster at every size; eight waves stay where one round of them fills the chip (they are up to 8 % faster
//     there than estimated: a window of 128 rows over 14086 keys, 24/8 heads 16.5, narrow 17.8).
// Measured at head_dim 128, us, eight waves / four of 64 keys / of 32, each with its best number of slices: 300 rows over
// 1300 keys, 32/8 heads 46 / 18 / 15.2; 500 over 4596, 8/8 25.5 / 19.9 / 16.1; 4000 over 4000, 16/4 467 / 78 / 62; 1000 over
// 3000, 32/8 132 / 46 / 37.8; 3000 over 3512, 8/8 94 / 36.6 / 28.7; 150 over 20150, 24/8 49 / 44.9 / 35.7; windows of 128 over
// 11193, 24/8 22.6 / 23.4 / 18.2, over 20000, 8/8 24.8 / 20.2 / 16.7, over 32000, 16/4 23.5 / 28.8 / 28.8; 4264 over 7945, 16/4
// 495 / 147 / 127; 5814 over 12828, 16/4 670 / 280 / 266 (114 tiles a compute unit); 2500 over 22500, 14/2 528 / 223 / 220 (92);
// from 146 on the other way: 6629 over 14487, 16/4 765 / 326 / 334; 6782 over 20108, 16/4 777 / 480 / 493; 1500 over
// 34268, 32/8 554 / 437 / 453; 8192 over 16384, 32/8 940 / 816 / 860; 16384 over 49152, 8/8 1416 / 1276 / 1373; 32768
// over 65536, 32/8 12.1 ms uncut, 12.3 ms in 4 or 8 slices.
// At 64, us, eight waves / narrow uncut / in 4 / 8 / 16 / 32 slices: 8192 rows over 16384 keys, 16/4 heads 752 / 500
// / 340 / 300 / 289 / 301; 16384 over 49152, 8/8 1123 / 893 / 893 / 909 / 944 / 1033; 12000 over 12000, 14/2 1904 / 994 /
// 362 / 255 / 224 / 205; 1000 over 4000, 32/8 111 / 55 / 36 / 36 / 38 / 38; a window of 128 rows over 11193, 24/8 19.6 /
// 15.0, over 32000, 16/4 19.8 / 20.8, over 20000, 8/8 19.0 / 10.7.
// scratch: bytes there are for the slices' sums; the cuts that fit are considered.
template <class P>
inline int score_plan_within(P &p, int cus, size_t scratch)
{
    const int tiles = (p.W + 63) / 64;
    const double iters = (double)p.G * tiles;
    const long full = (long)p.Hkv * ((p.n - p.W + 511) / 512), all = (long)p.Hkv * ((p.n + 511) / 512);
    const double total = (full + 0.5 * (double)(all - full)) * iters / cus;       // per compute unit
    // Uncut workgroups in the order they are dispatched: `whole` rounds of full ones, then on the units that a last,
    // partly filled round leaves (`room`) the triangular ones, the longest of which is a full one as well, and
    // with more than there is room for the longest left over behind the shortest.
    const long whole = full / cus, room = cus - full % cus, tri = all - full;
    double best = (double)(whole + (room < cus || tri > 0)) * iters;
    if (tri > room) {
        const double pair = (2.0 - 2.0 * (double)room / (double)tri) * iters;
        if (best < (double)whole * iters + pair) best = (double)whole * iters + pair;
    }
    if (best < total) best = total;
    best = p.D == 64 ? 1.2 * best + 2.0 : best + 4.0 * (double)((all + cus - 1) / cus);   // in the unit above, with the starts
    int form = kScoreEight;
    p.slices = p.head_slices = 1;
    p.slice_tiles = tiles;
    p.slice_heads = p.G;
    // slices of `per` tiles of `heads` heads, by workgroups of `keys` keys, `resident` of them on a compute unit; a full unit
    // takes `rate` a tile, a workgroup alone on one `alone`, the first tile `begin` more, the last ones leave `tail` of an item idle
    auto price = [&](int f, int keys, double resident, double rate, double tail, double alone, double begin, double fixed,
                     int per, int heads) {
        const int hs = (p.G + heads - 1) / heads, slices = (tiles + per - 1) / per * hs;
        if (slices > 1 && (size_t)slices * p.Hkv * p.n * sizeof(float) > scratch) return;
        const double item = (double)heads * per, items = 512.0 / keys * total * cus / item;
        double t = rate * total + tail * item;
        if (t < alone * item) t = alone * item;
        if (f == kScoreNarrow && p.D != 64 && slices == 1) {
            // a last round that is not full takes more than its part: 25 rows over 15606 keys, 32/8 heads (976 workgroups) 19.6 us, eight
            // waves 17.2
            double rounds = p.Hkv * (double)((p.n + keys - 1) / keys) / (resident * cus);
            if (rounds > 1.0) rounds = 0.5 * (rounds + (double)(long)rounds + 1.0);
            const double uncut = (rounds < 1.0 ? 1.0 : rounds) * (0.8 * item + begin) + 1.5 - begin * items / (resident * cus);
            if (t < uncut) t = uncut;
        }
        t += begin * items / (resident * cus) + fixed + (slices == 1 ? 0.0 : f == kScoreFour ? 2.0 : 3.0) + (p.D == 64 ? 0.1 * (hs - 1) : 0.0);
        if (t >= best) return;
        best = t;
        form = f;
        p.slices = slices;
        p.slice_tiles = per;
        p.head_slices = hs;
        p.slice_heads = heads;
    };
    const bool four = p.D != 64 && total >= 120.0;
    auto consider = [&](int per, int heads) {
        if (four) price(kScoreFour, 256, 2.0, 1.0, 0.5, 1.0, 1.5, 3.0, per, heads);
        else if (p.D == 64) price(kScoreNarrow, 128, 4.0, 1.0, 0.33, p.G == 1 ? 0.5 : 0.75, 1.6, 0.0, per, heads);
        else price(kScoreNarrow, 128, 3.0, 1.06, 0.35, 0.8, 1.6, 0.0, per, heads);
    };
    for (int want = 1; want <= (four ? 16 : 32); want *= 2) consider((tiles + want - 1) / want, p.G);
    // Where that leaves compute units without a workgroup the heads are cut as well: 60 rows over 8000 keys
    // with 14/2 heads of 64 (32 workgroups of 7 tiles) 38 -> 31 us for the call, 30 over 1000 with 14/2 of
    // 128 38 -> 28 us.  (On a chip that is busy it gives nothing: 2000 rows over 1000 keys, 32/8 heads, 18.9
    // -> 19.8 us.)  At 64 four workgroups share
    // a unit and one alone reaches a third of its rate (half with one head to a group: 520 rows over 2928 keys, 8/8 heads 11.8 us
    // uncut, 13.3 in three slices), so there with up to two to a unit as well: windows of 128 rows, 64/8
    // heads over 3211 keys 23.9 us uncut, 17.2 with the heads in two; 14/2 over 15117 20.5 and 15.7; 16/4 over 5292 16.2 and
    // 13.6.  Each set of heads costs the launch that adds up a little: 540 rows, 14/2 13.1 us in four sets, 14.3 in seven.
    const int keys = form == kScoreEight ? 512 : form == kScoreFour ? 256 : 128;
    if ((long)p.Hkv * ((p.n + keys - 1) / keys) * p.slices < (p.D == 64 ? 2l : 1l) * cus)
        for (int heads = (p.G + 1) / 2; heads >= 1; heads = heads > 1 ? (heads + 1) / 2 : 0) consider(1, heads);
    return form;
}

// The same, as cut as it is with room for all slices where those fit: a workspace kept from a smaller cut still serves
// for one like it.
template <class P>
inline int score_plan(P &p, int cus, size_t scratch = (size_t)-1)
{
    const int form = score_plan_within(p, cus, (size_t)-1);
    return score_slice_bytes(p) > scratch ? score_plan_within(p, cus, scratch) : form;
}

constexpr int kFewBlocks = 8;                            // row blocks over all heads of a group, at most (one wave)
constexpr int kFewKB = 2;                                // 16-key blocks of a wave of the register-only form

// Few observing rows over not too many keys: the register-only form.  Its waves (one per 32 keys of a KV
// head) fetch every query row themselves, so it loses its lead as rows or waves grow: 17 rows over 4113 keys of 8 heads
// 10 -> 6 us, 4 x 32 rows over 4128 keys 16.5 -> 12.3 us, 64 rows over 16064 keys 12 -> 18 us.
// Returns how many waves share their keys (RW in attn_score_few), 0 where this is not the form to take.
//
// Four of them for more row blocks: a workgroup per 32 keys of a KV head, which walks all rows.  At head_dim 128 its time
// goes by rounds of workgroups over the 256 compute units, each the longer the more blocks there are, about 3.5 + rounds
// (1.7 + blocks / 10) us, while the tiled form with its slices stays at 12 to 18 us.  Score alone, tiled / four waves, us,
// with one round: 12 blocks 10.4 / 6.3, 48 11.6 / 9.8, 64 11.7 / 11.4; two: 16 blocks 10.8 / 9.8, 28 13.1 / 13.0,
// 63 16.5 / 20.0; three: 9 blocks 14.0 / 11.3, 16 17.4 / 13.2, 24 13.8 / 15.1; five: 9 blocks 14.0 / 17.2; nine:
// 9 blocks 14.9 / 28.5.  In a round of few workgroups the tiled form is short as well, so more than 72 blocks need more of
// them.  Time with four waves over the tiled form's, one round: 68 to 72 blocks 0.85 to 1.01 from 20 workgroups on; 76 to 80
// blocks 1.04 to 1.10 at 50 to 88 (32 and 64 heads 0.90 to 0.94), 0.80 to 0.94 from 100 on; 84 to 90 blocks 1.11 to 1.15 at
// 50, 0.83 to 1.06 from 100 on (above 1 with 4 KV heads at 130 to 180 only, 0.5 us); 91 to 96 blocks 0.88 to 1.13 at 100 to
// 152, 0.90 to 0.96 at 180.
// At 64 a round costs half, tiled / four waves: 16 blocks, 210 workgroups 8.9 / 7.6; 20, 788 11.9 / 10.6; 32, 622 12.8 /
// 10.9; 56, 302 11.1 / 10.9; 40, 616 18.8 / 11.6; 72, 448 14.8 / 12.4; 91, 394 16.2 / 14.8; but 28, 856 10.3 / 11.8; 16, 1444
// 10.4 / 12.7; 37, 800 12.0 / 12.5; 64, 704 14.9 / 16.5; 80, 568 16.2 / 17.5; 12, 1592 8.2 / 15.3.
template <class P>
inline int score_few(const P &p)
{
    const long blocks = (long)p.G * ((p.W + 15) / 16);
    if (blocks <= 2 || (blocks <= kFewBlocks && (long)p.Hkv * p.n <= 65536)) return 1;
    if (blocks <= kFewBlocks || blocks > 96) return 0;
    const long groups = p.Hkv * ((p.n + 16l * kFewKB - 1) / (16 * kFewKB)), rounds = (groups + 255) / 256;
    if (p.D == 64) return groups * blocks <= (groups <= 640 ? 36000 : groups <= 1280 ? 20000 : 0) ? 4 : 0;
    if (rounds == 1) return blocks <= (groups < 100 ? 72 : groups <= 170 ? 90 : 96) ? 4 : 0;
    return rounds * (blocks + 14) <= 90 ? 4 : 0;
}

// Lanes that read the pieces of one observing row in attn_merge_score; entries: G W rows, 128 at most.
RF_PLAN int merge_score_lanes(int entries)
{
    int lanes = 64;
    while (lanes * entries > 256) lanes >>= 1;
    return lanes;
}

// Whether a split forward pass (planned) is merged by the launch that forms its score.  That saves a launch, 2 to 3 us, and
// costs every workgroup of the score, one per 128 keys of a KV head, the rows' normalisers from all their pieces.
// Whole calls, two launches / one, us:
//   - one token over 20000 keys, 14/2 heads of 64 17.0 / 13.3, 8/8 heads of 128 29.0 / 28.6 (1250 workgroups of the score);
//     16 rows over 14000, 8/8 of 128 28.9 / 27.1 (875), over 20000 34.8 / 35.8 (1250), over 60000 84.7 / 87.2; 16 over
//     30000, 8/8 of 64 29.4 / 28.0 (1875), one over 60000 41.1 / 42.6 (3750): not beyond four a compute unit, eight at 64.
//   - with many rows to merge, a workgroup each, fewer: 200 rows over 6000 keys, 8/8 of 64 29.8 / 27.9 (1975 workgroups
//     in all), 250 (17 observe) over 6000 27.1 / 26.8 (2375), over 10000 28.8 / 29.3 (2625), over 20000 34.5 / 36.5.
//   - a lane reads its row's pieces four at a time: 5 rows over 20000, 14/2 of 64 20.2 / 20.1 (eight times), 16 over 6000
//     17.7 / 16.4 (six), over 20000 24.4 / 27.3 (sixteen), of 128 33.5 / 36.6.
// gain: what it saves, us, if it does.
template <class P>
inline bool merge_with_score(const P &p, double *gain)
{
    const long n_merge = (long)p.Hkv * p.n_row_blocks * p.part_rows;
    const long n_score = p.Hkv * ((p.n + 64l * kFewKB - 1) / (64 * kFewKB));
    if (score_few(p) != 1 || n_merge > 2048 || n_merge + n_score > 2400 || n_score > (p.D == 64 ? 2048 : 1024)) return false;
    const long pieces = ((p.M + p.Ct - 1) / 64 + 1l) * p.shares / p.tiles;     // of the longest row block
    const int most = 8 * 4 * merge_score_lanes(p.G * p.W);
    if (gain && pieces < most) *gain = 3.0 * (1.0 - (double)pieces / most);
    return pieces <= most;
}

}  // namespace reform
