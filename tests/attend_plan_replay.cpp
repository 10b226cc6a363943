// Replays the plans of the bf16 attention as host code over the header that the kernels use: the walk of every workgroup of
// a split forward pass against the pieces that the merge reads, and the form that each pass takes.
#include "attend_plan.h"

#include <algorithm>
#include <vector>

using namespace reform;

struct Plan {
    int Hkv, G, D, M, Ct, n_row_blocks, by_head, narrow, shares, start, tiles, part_rows, n, W;
    int slices, slice_tiles, head_slices, slice_heads;
};
struct Piece { long t0, t1, slot; };

static Plan problem(int Hkv, int G, int D, int M, int Ct, int W)
{
    Plan p = {};
    p.Hkv = Hkv; p.G = G; p.D = D; p.M = M; p.Ct = Ct; p.n = M + Ct; p.W = W ? W : Ct;
    return p;
}

static size_t room(long scratch) { return scratch < 0 ? (size_t)-1 : (size_t)scratch; }

// 0 if every key tile of every row block is covered exactly once and the merge reads exactly the slots that were written (for
// whole row blocks: if their tiles are counted right), else a number that tells what failed.
template <int ROWS>
static int check(const Plan &p)
{
    if (p.shares && (long)p.tiles * p.shares >= (1l << 31)) return 2;
    const long rows = (long)p.G * p.Ct, blocks = (rows + ROWS - 1) / ROWS;
    if (p.n_row_blocks != blocks || p.part_rows != std::min(rows, (long)ROWS)) return 3;
    const int kvh = p.Hkv - 1;
    std::vector<std::vector<Piece>> got(blocks);
    for (int share = 0; share < p.shares; ++share) {
        const int begin = fwd_share_begin(p, share), end = fwd_share_begin(p, share + 1);
        if (begin != (long)share * p.tiles / p.shares) return 4;
        FwdWalk<Plan, ROWS> w(p);
        while (w.pos + w.nt <= begin) {
            if (w.nt <= 0 || w.rb >= blocks) return 5;
            w.next(p);
        }
        for (; w.pos < end; w.next(p)) {
            if (w.nt <= 0 || w.rb >= blocks) return 6;
            const int t0 = std::max(begin - w.pos, 0), t1 = std::min(end - w.pos, w.nt);
            // a share may end in the empty places before a row block or begin in those before the next
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

// The check above of the form that is launched.
extern "C" int replay_chosen(int Hkv, int G, int D, int M, int Ct, int scored, int cus)
{
    Plan p = problem(Hkv, G, D, M, Ct, 0);
    fwd_choose(p, cus, scored != 0);
    return p.narrow ? check<kFwdNarrowRows>(p) : check<kFwdRows>(p);
}

// The same of the form of eight waves, launched or not; 1: it is not split.
extern "C" int replay_eight(int Hkv, int G, int D, int M, int Ct, int cus)
{
    Plan p = problem(Hkv, G, D, M, Ct, 0);
    fwd_plan(p, cus);
    return p.shares ? check<kFwdRows>(p) : 1;
}

// Plans the forward pass as the launcher does, with that much room for partial results; the waves of attn_fwd_short where that
// takes the plan's place, else 0.
static int place(Plan &p, int scored, int cus, size_t scratch)
{
    const double est = fwd_choose(p, cus, scored != 0, scratch);
    return fwd_short(p, cus, est, scored != 0, scratch);
}

static int form_bits(const Plan &p, int scored)
{
    return (p.shares ? 2 : 0) + (p.shares && scored && merge_with_score(p) ? 4 : 0);
}

// The plan of the forward pass by row blocks of 256 or 128, which attn_fwd_short may take the place of.  Bit 0: four waves; bit 1:
// shared out; bit 2: merged by the score's launch.  scored: the call wants both.
extern "C" int plan_form(int Hkv, int G, int D, int M, int Ct, int W, int scored, int cus)
{
    Plan p = problem(Hkv, G, D, M, Ct, W);
    fwd_choose(p, cus, scored != 0);
    return p.narrow + form_bits(p, scored);
}

// The forward pass as it is launched with that many bytes for partial results (negative: as many as it wants): as above, and
// 8 where attn_fwd_short forms it, with bits 1 and 2 for its shares.
extern "C" int form_in(int Hkv, int G, int D, int M, int Ct, int W, int scored, int cus, long scratch)
{
    Plan p = problem(Hkv, G, D, M, Ct, W);
    const int waves = place(p, scored, cus, room(scratch));
    return (waves ? 8 : p.narrow) + form_bits(p, scored);
}

extern "C" int form(int Hkv, int G, int D, int M, int Ct, int W, int scored, int cus)
{
    return form_in(Hkv, G, D, M, Ct, W, scored, cus, -1);
}

// Shares of the forward pass with that many bytes for partial results (negative: as many as it wants), bytes: what they take.
extern "C" int fwd_shares(int Hkv, int G, int D, int M, int Ct, int scored, int cus, long scratch, long *bytes)
{
    Plan p = problem(Hkv, G, D, M, Ct, 0);
    fwd_choose(p, cus, scored != 0, room(scratch));
    *bytes = (long)fwd_split_bytes(p);
    return p.shares;
}

// The score pass: 1 or 4 for the register-only form with that many waves to a set of keys, else 1000 times the tiled form
// (kScoreEight, kScoreFour or kScoreNarrow) and its slices.
extern "C" int score_form(int Hkv, int G, int D, int M, int Ct, int W, int cus)
{
    Plan p = problem(Hkv, G, D, M, Ct, W);
    if (const int waves = score_few(p)) return waves;
    const int tiled = score_plan(p, cus);
    return 1000 * tiled + p.slices;
}

// Slices of the tiled score pass with that many bytes for their sums (negative: as many as it wants); -1 where they need more.
extern "C" int score_slices(int Hkv, int G, int D, int M, int Ct, int W, int cus, long scratch)
{
    Plan p = problem(Hkv, G, D, M, Ct, W);
    score_plan(p, cus, room(scratch));
    const int tiles = (p.W + 63) / 64, sets = (tiles + p.slice_tiles - 1) / p.slice_tiles;
    if (p.slices != sets * p.head_slices || p.head_slices != (G + p.slice_heads - 1) / p.slice_heads) return -2;
    return score_slice_bytes(p) > room(scratch) ? -1 : p.slices;
}

// attn_fwd_short where that forms the forward pass instead of the plan above: its waves + 100 times the workgroups to a row
// block's keys, 10000 more where the score's launch merges them; else 0.
extern "C" int short_form(int Hkv, int G, int D, int M, int Ct, int W, int scored, int cus)
{
    Plan p = problem(Hkv, G, D, M, Ct, W);
    const int waves = place(p, scored, cus, (size_t)-1);
    if (!waves) return 0;
    return waves + 100 * std::max(p.shares, 1) + (p.shares && scored && merge_with_score(p) ? 10000 : 0);
}

// Bytes of its pieces with that much room for them (negative: as much as it wants).
extern "C" long short_bytes(int Hkv, int G, int D, int M, int Ct, int scored, int cus, long scratch)
{
    Plan p = problem(Hkv, G, D, M, Ct, 0);
    return place(p, scored, cus, room(scratch)) ? (long)fwd_short_bytes(p) : 0;
}

// 0 if the workgroups of attn_fwd_short, shared out, cover every key tile of every row block of every KV head exactly once, and
// leave their pieces in slots of their own inside its bytes, the ones that the merge reads; 1: it is not launched or not
// shared out; else a number that tells what failed.
extern "C" int replay_short(int Hkv, int G, int D, int M, int Ct, int scored, int cus, long scratch)
{
    Plan p = problem(Hkv, G, D, M, Ct, 0);
    if (!place(p, scored, cus, room(scratch)) || !p.shares) return 1;
    const long rows = (long)G * Ct, blocks = (rows + 31) / 32;
    if (kFwdShortRows != 32 || p.n_row_blocks != blocks || p.part_rows != 32) return 2;
    if (fwd_short_bytes(p) > room(scratch)) return 3;
    const long slots = (long)p.shares * Hkv * blocks;
    if (slots * 32 * (D + 2) * (long)sizeof(float) != (long)fwd_short_bytes(p)) return 4;
    std::vector<std::vector<Piece>> got(blocks * Hkv);
    for (long b = 0; b < slots; ++b) {                   // as the kernel reads blockIdx
        const int kvh = (int)(b % Hkv), group = (int)(b / Hkv), share = group % p.shares, rb = p.n_row_blocks - 1 - group / p.shares;
        if (rb < 0) return 5;
        const int all = fwd_short_tiles(p, rb);
        if (all != ((long)M + (std::min((rb + 1l) * 32, rows) - 1) / G) / 32 + 1) return 6;
        got[rb * Hkv + kvh].push_back({fwd_short_begin(p, all, share), fwd_short_begin(p, all, share + 1),
                                       ShortPieces<Plan>(p, rb).slot(p, share, kvh)});
    }
    std::vector<char> used(slots);
    for (int rb = 0; rb < blocks; ++rb)
        for (int kvh = 0; kvh < Hkv; ++kvh) {
            const ShortPieces<Plan> pieces(p, rb);
            const std::vector<Piece> &mine = got[rb * Hkv + kvh];
            if (pieces.j1 - pieces.j0 + 1 != (long)mine.size()) return 7;
            long at = 0;
            for (size_t i = 0; i < mine.size(); ++i) {
                if (mine[i].t0 != at || mine[i].t1 <= at) return 8;
                at = mine[i].t1;
                if (mine[i].slot != pieces.slot(p, pieces.j0 + (int)i, kvh)) return 9;
                if (mine[i].slot < 0 || mine[i].slot >= slots || used[mine[i].slot]++) return 10;
            }
            if (at != fwd_short_tiles(p, rb)) return 11;
        }
    return 0;
}
