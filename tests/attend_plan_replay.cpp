// Replays the walk of every workgroup of the split forward pass and the piece ranges of the merge, as host
// code over the same header.  Returns 0 if every key tile of every row block is covered exactly once and the
// merge reads exactly the slots that were written for it, 1 if the problem is not split, else a number
// that tells what failed.  score_form: the form of the score pass.  merged: whether its launch merges a split
// forward pass.
#include "attend_plan.h"

#include <algorithm>
#include <vector>

using namespace reform;

struct Plan { int Hkv, G, D, M, Ct, n_row_blocks, by_head, narrow, shares, start, tiles, part_rows, n, W; };
struct ScorePlan { int Hkv, G, D, n, W, slices, slice_tiles, head_slices, slice_heads; };
struct Piece { long t0, t1, slot; };

extern "C" int replay(int Hkv, int G, int D, int M, int Ct, int cus)
{
    Plan p = {};
    p.Hkv = Hkv; p.G = G; p.D = D; p.M = M; p.Ct = Ct;
    fwd_plan(p, cus);
    if (!p.shares) return 1;
    if ((long)p.tiles * p.shares >= (1l << 31)) return 2;
    const long rows = (long)G * Ct, blocks = (rows + kFwdRows - 1) / kFwdRows;
    if (p.n_row_blocks != blocks) return 3;
    const int kvh = Hkv - 1;
    std::vector<std::vector<Piece>> got(blocks);
    for (int share = 0; share < p.shares; ++share) {
        const int begin = fwd_share_begin(p, share), end = fwd_share_begin(p, share + 1);
        if (begin != (long)share * p.tiles / p.shares) return 4;
        FwdWalk<Plan> w(p);
        while (w.pos + w.nt <= begin) {
            if (w.nt <= 0 || w.rb >= blocks) return 5;
            w.next(p);
        }
        while (w.pos < end) {
            if (w.nt <= 0 || w.rb >= blocks) return 6;
            const int t0 = std::max(begin - w.pos, 0), t1 = std::min(end - w.pos, w.nt);
            // a share may end in the empty places before a row block or begin in those before the next
            if (t0 < t1) got[w.rb].push_back({t0, t1, fwd_slot(p, share, kvh, t0, t1, w.nt)});
            w.next(p);
        }
    }
    int pos = 0;
    for (int rb = 0; rb < blocks; ++rb) {
        pos += p.start;
        const int nt = fwd_row_block_tiles(p, rb);
        const long last = std::min((rb + 1l) * kFwdRows, rows) - 1;
        if (nt != ((long)M + last / G) / 64 + 1) return 7;
        const FwdPieces<Plan> pieces(p, pos, nt);
        if (pieces.j1 - pieces.j0 + 1 != (long)got[rb].size()) return 8;
        long at = 0;
        for (size_t i = 0; i < got[rb].size(); ++i) {
            if (got[rb][i].t0 != at) return 9;
            at = got[rb][i].t1;
            const long slot = pieces.j0 == pieces.j1 ? -1 : pieces.slot(p, pieces.j0 + (int)i, kvh);
            if (got[rb][i].slot != slot) return 10;
        }
        if (at != nt) return 11;
        pos += nt;
    }
    return pos == p.tiles ? 0 : 12;
}

// Waves that share their keys in the register-only form (1 or 4); 0: the tiled form, uncut; 16 * slices: cut.
extern "C" int score_form(int Hkv, int G, int D, int M, int Ct, int W, int cus)
{
    ScorePlan p = {};
    p.Hkv = Hkv; p.G = G; p.D = D; p.n = M + Ct; p.W = W ? W : Ct;
    if (const int waves = score_few(p)) return waves;
    score_plan(p, cus);
    return p.slices > 1 ? 16 * p.slices : 0;
}

// Shares of the forward pass with that many bytes for partial results (negative: as many as it wants), bytes: what they take.
extern "C" int fwd_shares(int Hkv, int G, int D, int M, int Ct, int scored, int cus, long scratch, long *bytes)
{
    Plan p = {};
    p.Hkv = Hkv; p.G = G; p.D = D; p.M = M; p.Ct = Ct; p.n = M + Ct; p.W = Ct;
    fwd_choose(p, cus, scored, scratch < 0 ? (size_t)-1 : (size_t)scratch);
    *bytes = (long)fwd_split_bytes(p);
    return p.shares;
}

// Slices of the tiled score pass with that many bytes for their sums (negative: as many as it wants); -1 where they need more.
extern "C" int score_slices(int Hkv, int G, int D, int M, int Ct, int W, int cus, long scratch)
{
    ScorePlan p = {};
    p.Hkv = Hkv; p.G = G; p.D = D; p.n = M + Ct; p.W = W ? W : Ct;
    score_plan(p, cus, scratch < 0 ? (size_t)-1 : (size_t)scratch);
    const int tiles = (p.W + 63) / 64, sets = (tiles + p.slice_tiles - 1) / p.slice_tiles;
    if (p.slices != sets * p.head_slices || p.head_slices != (G + p.slice_heads - 1) / p.slice_heads) return -2;
    return scratch >= 0 && score_slice_bytes(p) > (size_t)scratch ? -1 : p.slices;
}

// Whether a call that wants both is split (bit 0), and merged by the launch that forms the score (bit 1).
extern "C" int merged(int Hkv, int G, int D, int M, int Ct, int W, int cus)
{
    Plan p = {};
    p.Hkv = Hkv; p.G = G; p.D = D; p.M = M; p.Ct = Ct; p.n = M + Ct; p.W = W ? W : Ct;
    fwd_plan(p, cus);
    return p.shares ? 1 + 2 * merge_with_score(p) : 0;
}
