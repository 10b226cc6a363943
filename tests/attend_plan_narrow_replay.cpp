// Replays the form that fwd_choose picks for a problem, as attend_plan_replay.cpp does for the form of 256-row blocks.
// Returns 0 if every key tile of every row block is covered exactly once and the merge reads exactly the slots that
// were written (for whole row blocks: if their tiles are counted right), else a number that tells what failed.
#include "attend_plan.h"

#include <algorithm>
#include <vector>

using namespace reform;

struct Plan { int Hkv, G, D, M, Ct, n_row_blocks, by_head, narrow, shares, start, tiles, part_rows, n, W; };
struct Piece { long t0, t1, slot; };

static Plan chosen(int Hkv, int G, int D, int M, int Ct, int W, int scored, int cus)
{
    Plan p = {};
    p.Hkv = Hkv; p.G = G; p.D = D; p.M = M; p.Ct = Ct; p.n = M + Ct; p.W = W ? W : Ct;
    fwd_choose(p, cus, scored != 0);
    return p;
}

template <int ROWS>
static int check(const Plan &p)
{
    const long rows = (long)p.G * p.Ct, blocks = (rows + ROWS - 1) / ROWS;
    if (p.n_row_blocks != blocks || p.part_rows != std::min(rows, (long)ROWS)) return 3;
    const int kvh = p.Hkv - 1;
    std::vector<std::vector<Piece>> got(blocks);
    for (int share = 0; share < p.shares; ++share) {
        const int begin = fwd_share_begin(p, share), end = fwd_share_begin(p, share + 1);
        if (begin != (long)share * p.tiles / p.shares) return 4;
        FwdWalk<Plan, ROWS> w(p);
        while (w.pos + w.nt <= begin) w.next(p);
        for (; w.pos < end; w.next(p)) {
            if (w.nt <= 0 || w.rb >= blocks) return 6;
            const int t0 = std::max(begin - w.pos, 0), t1 = std::min(end - w.pos, w.nt);
            if (t0 < t1) got[w.rb].push_back({t0, t1, fwd_slot(p, share, kvh, t0, t1, w.nt)});
        }
    }
    int pos = 0;
    for (int rb = 0; rb < blocks; ++rb) {
        const int nt = fwd_row_block_tiles<ROWS>(p, rb);
        const long last = std::min((rb + 1l) * ROWS, rows) - 1;
        if (nt != ((long)p.M + last / p.G) / 64 + 1) return 7;
        if (!p.shares) continue;
        pos += p.start;
        const FwdPieces<Plan> pieces(p, pos, nt);
        if (pieces.j1 - pieces.j0 + 1 != (long)got[rb].size()) return 8;
        long at = 0;
        for (size_t i = 0; i < got[rb].size(); ++i) {
            if (got[rb][i].t0 != at) return 9;
            at = got[rb][i].t1;
            if (got[rb][i].slot != (pieces.j0 == pieces.j1 ? -1 : pieces.slot(p, pieces.j0 + (int)i, kvh))) return 10;
        }
        if (at != nt) return 11;
        pos += nt;
    }
    return !p.shares || pos == p.tiles ? 0 : 12;
}

extern "C" int replay_chosen(int Hkv, int G, int D, int M, int Ct, int scored, int cus)
{
    const Plan p = chosen(Hkv, G, D, M, Ct, 0, scored, cus);
    if (p.shares && (long)p.tiles * p.shares >= (1l << 31)) return 2;
    return p.narrow ? check<kFwdNarrowRows>(p) : check<kFwdRows>(p);
}

// Bit 0: the narrow form; bit 1: shared out; bit 2: merged by the score's launch.
extern "C" int form(int Hkv, int G, int D, int M, int Ct, int W, int scored, int cus)
{
    const Plan p = chosen(Hkv, G, D, M, Ct, W, scored, cus);
    return p.narrow + (p.shares ? 2 : 0) + (p.shares && scored && merge_with_score(p) ? 4 : 0);
}
