// bf16 chunk attention over [cache || chunk] and the eviction score, for gfx950 MFMA.
//
// Two kernels per call (Sec. 3.1 / Fig. 1 step 1 of arXiv 2506.01215 for the attention; Sec. 3.1
// and Sec. 5 for the attention-based eviction score that the method wants fused next to it):
//
//   attn_fwd_bf16    row-owned flash-style pass: out and lse.
//   attn_score_bf16  column-owned pass: score_j = sum_h sum_i exp(s_ij - lse_i).  The exact score
//                    needs the final normaliser of every row, so QK^T is formed a second time; the
//                    probabilities are never stored.
//
// Problems that do not fill the chip have forms of their own (attn_fwd_few, attn_fwd_short, attn_score_few), and parts of
// shared-out ones meet in attn_fwd_merge, attn_merge_score and attn_score_sum; attend_plan.h says which when.
//
// Both kernels compute the TRANSPOSED logit tile  S^T = K Q^T: a lane then owns one query column
// and a few key rows, so the softmax row statistics are per-lane scalars (exchanged across the
// lane groups once), and the probabilities are already laid out as the B operand of
// O^T = V^T P^T  once the contraction index is permuted consistently on the V side (the V^T
// operands are fetched from a row-major V tile with gfx950's transposing LDS load, in that
// permuted key order).  Both kernels use v_mfma_f32_16x16x32_bf16 (wave64 operand layout:
// A[m][k]: lane l holds m = l%16, k = 8*(l/16)..+7;  B[k][n]: n = l%16, same k;
// C[m][n]: lane l holds n = l%16 and, in accumulator element e, m = 4*(l/16) + e).
#include "common.h"
#include "attend_plan.h"

#include <algorithm>
#include <atomic>

namespace reform {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// ------------------------------------------------------------------------------------------
// Global -> register -> LDS staging of one 64-key K/V tile by a workgroup of NT threads: K and V
// rows are copied as they are, 16 bytes per thread and piece.  V is NOT transposed on the way in:
// the V^T operands of O^T = V^T P^T are read with ds_read_b64_tr_b16, the transposing LDS load of
// gfx950 (see lds_read_tr16 below); two plain 16-byte stores per piece replace the transposing
// 4-byte stores and their packing VALU work (about 1 % of the kernel time, and 16 VGPRs).
//
// LDS layout, measured on gfx950: a ds_read_b128 is served half a wave at a time and is free of
// bank conflicts when the 32 lanes touch 32 different 16-byte slots modulo 512 bytes.  The K
// fragment reads have 16-lane row groups (lane%16 = row, lane/16 = 16-byte piece), so a half
// wave reads 16 rows x 2 adjacent pieces: the row pitch must be an odd multiple of 32 bytes
// (288 bytes for D = 128; 272 bytes showed 3.7x the bank-conflict cycles).  The transposing V
// reads touch 16 consecutive rows x 32 bytes per instruction; the same pitch keeps them apart.
template <int D, int NT>
struct TileStage {
    static constexpr int BN = 64;
    static constexpr int KROW = D + 16;      // row pitch of both tiles, elements
    static constexpr int C8 = D / 8;
    static constexpr int PIECES = BN * C8 / NT;
    static_assert(PIECES == 1 || PIECES == 2 || PIECES == 4, "tile/threads mismatch");
    v4u kpre[PIECES], vpre[PIECES];
    uint32_t goff;                // byte offset of this thread's first piece inside a tile (global)
    uint32_t loff;                // element offset inside an LDS tile
    int row0;                     // tile-relative row of the first piece (for the clamped tail path)

    __device__ __forceinline__ void init(int tid)
    {
        row0 = tid / C8;
        goff = (uint32_t)(row0 * D + (tid % C8) * 8) * 2u;
        loff = (uint32_t)(row0 * KROW + (tid % C8) * 8);
    }
    // Kt, Vt: tile base pointers (uniform); rows_left = n - j0 (>= 1).  Piece i sits NT/C8 rows
    // further down.
    __device__ __forceinline__ void load(const u16 *Kt, const u16 *Vt, int rows_left)
    {
        const char *kb = (const char *)Kt, *vb = (const char *)Vt;
        if (rows_left >= BN) {
#pragma unroll
            for (int i = 0; i < PIECES; ++i) {
                const uint32_t off = goff + (uint32_t)(i * (NT / C8) * D * 2);
                kpre[i] = *(const v4u *)(kb + off);
                vpre[i] = *(const v4u *)(vb + off);
            }
        } else {   // ragged last tile: rows past the end repeat the last valid row
#pragma unroll
            for (int i = 0; i < PIECES; ++i) {
                const int r = row0 + i * (NT / C8);
                const int back = r < rows_left ? 0 : r - (rows_left - 1);
                const uint32_t off = goff + (uint32_t)((i * (NT / C8) - back) * D * 2);
                kpre[i] = *(const v4u *)(kb + off);
                vpre[i] = *(const v4u *)(vb + off);
            }
        }
    }
    __device__ __forceinline__ void store(u16 *dk, u16 *dv) const
    {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            *(v4u *)(dk + loff + i * (NT / C8) * KROW) = kpre[i];
            *(v4u *)(dv + loff + i * (NT / C8) * KROW) = vpre[i];
        }
    }
};

// ds_read_b64_tr_b16 (gfx950).  Within each group of 16 lanes, lane r supplies the address of four
// consecutive 16-bit elements B[r][0..3]; lane i of the group receives, as element j,
// B[4*j + i/4][i%4] (established by writing element indices into LDS and reading them back).  With
// lane r = 4*j + q pointing at V[key_j][d0 + 4*q .. +3], lane i therefore receives
// V[key_0..3][d0 + i]: four keys of one d column, half of an MFMA A operand of V^T.
__device__ __forceinline__ v2u lds_read_tr16(const u16 *p)
{
    typedef short v4s __attribute__((ext_vector_type(4)));
    const v4s r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)p);
    return __builtin_bit_cast(v2u, r);
}

__device__ __forceinline__ f32x4 mfma16(v4u a, v4u b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a), as_bf16x8(b), c, 0, 0, 0);
}

// p = exp2(s*c - mc) for the 16 logits a lane holds of one query and one 64-key tile (four 16-key
// blocks x 4 keys), packed to bf16 as the two B operands of P.V (key pairs 0 and 1); returns the
// lane's partial row sum.  Plain v_add_f32 on purpose: v_dot2c_f32_bf16 was measured NOT to
// co-execute with another wave's MFMAs on gfx950, while v_fma / v_add / v_exp / v_cvt_pk do.
__device__ __forceinline__ float softmax_row(const f32x4 (&s)[4], float c, float mc, v4u (&pb)[2])
{
    float rs = 0.f;
#pragma unroll
    for (int kp = 0; kp < 2; ++kp) {
        float pv[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            pv[j] = __builtin_amdgcn_exp2f(fmaf(s[2 * kp + (j >> 2)][j & 3], c, -mc));
            rs += pv[j];
        }
        v4u w;
        w.x = pack_bf16x2(pv[0], pv[1]);
        w.y = pack_bf16x2(pv[2], pv[3]);
        w.z = pack_bf16x2(pv[4], pv[5]);
        w.w = pack_bf16x2(pv[6], pv[7]);
        pb[kp] = w;
    }
    return rs;
}

// Forward: out, lse.  One workgroup = 8 waves; a wave owns 32 query rows.  The query rows of a KV head
// are counted over its chunk rows and the G heads of its group together (row r is chunk row r / G
// of head r % G), and a workgroup takes 256 of them, so the K/V tiles staged in LDS (two K slots,
// three V slots, one barrier per 64-key tile) serve every wave and every head whatever G is, and
// only the last row block of a KV head is padded.  With one, two or four heads per row block, whichever
// divides G, and each head's chunk rows padded by themselves: four tokens over 60000 keys with 24/8
// heads 108 us, now 41; one over 20000 with 14/2 heads of 64 24 us, now 13.6; 300 rows over 1500 keys
// with 24/8 heads 66 us, now 56 (with the score).
//
// NW = 4 (the narrow form; where it is taken and what it gives: fwd_choose): 128 rows by four waves, two V slots and no wave
// lagging, as the other workgroups of the compute unit (two, at head_dim 64 three: 168 registers there) are out of step by
// themselves.  At 64 three waves per SIMD take 15 % fewer cycles on a large problem, at a clock that falls by 10 % (power).
// Shared out it spills in the set-up and the end of a segment, outside the loop over key tiles: 22 registers at 64 (5 where row
// blocks are whole), 11 at 128 (none); the forms of eight waves spill none.
//
// MFMA shape: v_mfma_f32_16x16x32_bf16 (A[m][k]: lane l holds m = l%16, k = 8*(l/16)..+7; B[k][n]:
// n = l%16, same k; C[m][n]: n = l%16, m = 4*(l/16) + e).  Measured on gfx950 with random bf16
// operands the matrix pipe is limited by the power budget, and this shape sustains 2.03 PFLOP/s
// against 1.83 PFLOP/s for 32x32x16 (both reach 2.36-2.39 with all-zero operands): it moves half
// the accumulator data per flop.  S^T = K Q^T is formed per 16-key block and 16-query block: a lane
// owns one query column (lane % 16) of each of the wave's two query blocks and, per key block, the
// four keys 4*(lane/16)..+3; row statistics are per-lane scalars reduced over lane/16 once at
// the end, and the probabilities are already the B operand of O^T = V^T P^T: key pair kp
// contracts the 32 keys of key blocks 2*kp and 2*kp+1, lane group g = lane/16 supplying keys
// 4g..4g+3 of each, and the transposing LDS reads fetch exactly those V rows.
//
// Wall time follows the energy of the launch (the shader clock falls to about 1.95 GHz under
// this kernel with random data), so the kernel keeps the instruction count and the data
// movement per tile small:
//   - no row maximum on the fast path: probabilities are formed against the current reference
//     m_run; if a row outgrew it by more than kBigSum (or m_run is still -inf) the tile sum of
//     that row is huge / inf / NaN, and only then the whole wave recomputes with the true maximum
//     and rescales its accumulators once;
//   - scale*log2(e) folded into one v_fma per logit, v_exp_f32 directly, packed bf16 converts;
//   - tile addresses are a uniform base plus per-thread constants computed once.
constexpr float kBigSum = 65536.0f;

template <int D, int NW>
constexpr size_t fwd_lds_bytes()
{
    return sizeof(u16) * (size_t)((NW == kFwdWaves ? 5 : 4) * 64 * (D + 16));      // two K slots, three V slots (two if no wave lags)
}

// One workgroup's pass of row block rb over the key tiles [t0, t1).  With
// SPLIT the result is either final (the range covers the whole row block) or goes, unnormalised,
// to partial slot `slot`; without it the range is the whole row block.
template <int D, int NW, bool SPLIT>
__device__ __forceinline__ void fwd_segment(const AttnParams &p, u16 *smem, int kvh, int rb, int t0, int t1, long slot)
{
    constexpr int NT = NW * 64, ROWS = NW * 32;
    constexpr bool LAG = NW == kFwdWaves;                // see below
    constexpr int VSLOTS = LAG ? 3 : 2;
    constexpr int KS = D / 32;           // MFMA k-steps of Q.K^T
    constexpr int DB = D / 16;           // 16-wide output blocks of P.V
    using Stage = TileStage<D, NT>;
    constexpr int BN = Stage::BN, KROW = Stage::KROW;
    constexpr int KTILE = BN * KROW, VTILE = BN * KROW;
    constexpr int kWin = 4;              // fragment prefetch distance (register quads)
    constexpr int NK = 4 * KS;           // K fragments per tile  (key block, k-step)
    constexpr int NV = 2 * DB;           // V^T fragments per tile (key pair, d block)

    u16 *ldsK = smem;                          // [2][KTILE]
    u16 *ldsV = smem + 2 * KTILE;              // [VSLOTS][VTILE]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int ln = lane & 15;
    const int lg = lane >> 4;

    const int rows = p.G * p.Ct;
    // Which 32 of the row block's rows the wave has: lane's row in 16-row block nb is row0 + rstep * (16 nb
    // + ln).  p.by_head (G divides the waves, so a full row block is ROWS / G chunk rows of every head): consecutive
    // chunk rows of one head; otherwise consecutive rows.
    const int slab = p.by_head ? wave / p.G : wave, rstep = p.by_head ? p.G : 1;
    const int row0 = rb * ROWS + slab * 32 * rstep + (p.by_head ? wave % p.G : 0);
    // Chunk row and head of this lane's row.  Formed where needed, from a G the compiler cannot relate to
    // the other uses: kept, the four values cost registers in the main loop.
    auto locate = [&](int nb, int &chunk_row, size_t &head) {
        int G = p.G;
        asm volatile("" : "+s"(G));
        const int r = min(row0 + rstep * (16 * nb + ln), rows - 1);
        chunk_row = r / G;
        head = kvh * G + r % G;
    };

    const int jbase = SPLIT ? t0 * BN : 0;               // first key of the range; tiles below count from it
    const u16 *Kg = (const u16 *)p.k + ((size_t)kvh * p.cap + jbase) * D;
    const u16 *Vg = (const u16 *)p.v + ((size_t)kvh * p.cap + jbase) * D;
    const int M = p.M - jbase, n = p.n - jbase;          // both relative to the range

    // Q^T operands of the wave's two 16-row query blocks stay in registers for the whole pass
    v4u qreg[2][KS];
    {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            int row;
            size_t head;
            locate(nb, row, head);
            const u16 *src = (const u16 *)p.q + head * p.q_hs + (size_t)row * p.q_rs + 8 * lg;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) qreg[nb][ks] = *(const v4u *)(src + ks * 32);
        }
    }

    const int ntiles = SPLIT ? t1 - t0 : fwd_row_block_tiles<ROWS>(p, rb);
    const int wave_first_row = row0 / p.G;
    const int wave_last_key = (row0 < rows) ? M + min(row0 + 31 * rstep, rows - 1) / p.G : -1;

    f32x4 o[2][DB];
    float m_run[2] = {-INFINITY, -INFINITY}, l_run[2] = {0.f, 0.f};
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int db = 0; db < DB; ++db) o[nb][db] = (f32x4){0.f, 0.f, 0.f, 0.f};

    const float c = p.scale * kLog2e;
    // per-lane fragment offsets (elements) inside a K tile / V^T tile
    const int k_frag0 = ln * KROW + 8 * lg;
    const int v_frag0 = (4 * lg + (ln >> 2)) * KROW + 4 * (ln & 3);   // see lds_read_tr16

    Stage st;
    st.init(tid);
    st.load(Kg, Vg, n);
    st.store(ldsK, ldsV);
    if (ntiles > 1) st.load(Kg + BN * D, Vg + BN * D, n - BN);
    __syncthreads();

    // Two waves share a SIMD (wave w and w + NW/2), and the barrier per tile keeps them in step.
    // To make one wave's MFMAs meet the other's softmax, the waves of the upper half run their
    // O^T += V^T P^T one tile late: iteration t does P.V of tile t-1 first, then Q.K^T and the
    // softmax of tile t, keeping the probabilities in registers across the barrier.  V therefore
    // lives in three LDS slots (tile u in slot u%3), K in two.  (Without lagging waves V has two: every wave
    // reads tile t between the barriers around it.)
    const bool lag = LAG && wave >= NW / 2;
    // last tile of the range this wave needs
    const int tl = SPLIT ? (wave_last_key >= 0 ? min(wave_last_key / BN, ntiles - 1) : -1)
                         : (wave_last_key >= 0 ? wave_last_key / BN : -1);
    v4u pb[2][2];
    int vslot = 0;                                                    // t mod VSLOTS

    auto mask_tile = [&](f32x4 (&s)[2][4], int j0) {
        if (j0 + BN - 1 > M + wave_first_row) {
            asm volatile("; mask path" ::: "memory");      // diagonal tiles only: keep out of line
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                int row;
                size_t head;
                locate(nb, row, head);
                const int lim = M + row - j0;                 // key offset <= lim is visible
#pragma unroll
                for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (kb * 16 + 4 * lg + e > lim) s[nb][kb][e] = -INFINITY;
            }
        }
    };
    // probabilities of one tile into pb, running sums; the rare rescale is kept out of line
    auto softmax_phase = [&](f32x4 (&s)[2][4]) {
        float rs0 = softmax_row(s[0], c, m_run[0] * c, pb[0]);
        float rs1 = softmax_row(s[1], c, m_run[1] * c, pb[1]);
        if (__builtin_amdgcn_ballot_w64(!(rs0 < kBigSum) || !(rs1 < kBigSum)) != 0ull) {
            asm volatile("; rescale path" ::: "memory");
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                float mx = s[nb][0][0];
#pragma unroll
                for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                    for (int e = 0; e < 4; ++e) mx = fmaxf(mx, s[nb][kb][e]);
                mx = fmaxf(mx, __shfl_xor(mx, 16));
                mx = fmaxf(mx, __shfl_xor(mx, 32));
                const float m_new = fmaxf(mx, m_run[nb]);
                // a range may begin on tiles in which a row sees no key yet: nothing to rescale then
                const float alpha = SPLIT && m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f((m_run[nb] - m_new) * c);
                m_run[nb] = m_new;
                l_run[nb] *= alpha;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[nb][db][e] *= alpha;
            }
            rs0 = softmax_row(s[0], c, SPLIT && m_run[0] == -INFINITY ? 0.f : m_run[0] * c, pb[0]);
            rs1 = softmax_row(s[1], c, SPLIT && m_run[1] == -INFINITY ? 0.f : m_run[1] * c, pb[1]);
        }
        l_run[0] += rs0;
        l_run[1] += rs1;
    };

    for (int t = 0; t < ntiles; ++t) {
        const int j0 = t * BN;
        const u16 *sk = ldsK + (t & 1) * KTILE + k_frag0;
        auto kfrag = [&](int i) -> v4u {         // i = 4*ks + kb: keys 16*kb + ln, d 32*ks + 8*lg..+7
            return *(const v4u *)(sk + (i & 3) * 16 * KROW + (i >> 2) * 32);
        };
        if (!lag) {
            if (t <= tl) {
                asm volatile("; in-step wave" ::: "memory");
                const u16 *sv = ldsV + vslot * VTILE + v_frag0;
                auto vfrag = [&](int i) -> v4u { // i = DB*kp + db: d 16*db + ln, key pair kp
                    const int kp = i / DB, db = i % DB;
                    const v2u lo = lds_read_tr16(sv + (32 * kp) * KROW + 16 * db);        // keys of block 2*kp
                    const v2u hi = lds_read_tr16(sv + (32 * kp + 16) * KROW + 16 * db);   // and of block 2*kp+1
                    return (v4u){lo.x, lo.y, hi.x, hi.y};
                };
                // ---- S^T = K Q^T; fragments stream through a rolling window of kWin register
                // quads, each feeding the MFMAs of both query blocks; the window is refilled with
                // the first V^T fragments while the last MFMAs run
                v4u fw[kWin];
#pragma unroll
                for (int i = 0; i < kWin; ++i) fw[i] = kfrag(i);
                f32x4 s[2][4];
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                    for (int kb = 0; kb < 4; ++kb) s[nb][kb] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int f = 0; f < NK; ++f) {
                    s[0][f & 3] = mfma16(fw[f % kWin], qreg[0][f >> 2], s[0][f & 3]);
                    s[1][f & 3] = mfma16(fw[f % kWin], qreg[1][f >> 2], s[1][f & 3]);
                    const int g = f + kWin;
                    fw[f % kWin] = g < NK ? kfrag(g) : vfrag(g - NK);
                }
                __builtin_amdgcn_sched_group_barrier(0x100, kWin, 0);
#pragma unroll
                for (int f = 0; f < NK - kWin; ++f) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                }
#pragma unroll
                for (int f = NK - kWin; f < NK; ++f) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);   // a V^T fragment is two reads
                }
                mask_tile(s, j0);
                softmax_phase(s);
                // ---- O^T += V^T P^T, rest of the V^T fragments
#pragma unroll
                for (int f = 0; f < NV; ++f) {
                    o[0][f % DB] = mfma16(fw[f % kWin], pb[0][f / DB], o[0][f % DB]);
                    o[1][f % DB] = mfma16(fw[f % kWin], pb[1][f / DB], o[1][f % DB]);
                    if (f + kWin < NV) fw[f % kWin] = vfrag(f + kWin);
                }
#pragma unroll
                for (int f = 0; f < NV; ++f) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
                    if (f + kWin < NV) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                }
            }
        } else {
            const bool do_pv = t >= 1 && t - 1 <= tl, do_qk = t <= tl;
            if (do_pv || do_qk) {
                asm volatile("; lagging wave" ::: "memory");
                const u16 *sv = ldsV + (vslot == 0 ? 2 : vslot - 1) * VTILE + v_frag0;   // tile t-1
                auto vfrag = [&](int i) -> v4u {
                    const int kp = i / DB, db = i % DB;
                    const v2u lo = lds_read_tr16(sv + (32 * kp) * KROW + 16 * db);
                    const v2u hi = lds_read_tr16(sv + (32 * kp + 16) * KROW + 16 * db);
                    return (v4u){lo.x, lo.y, hi.x, hi.y};
                };
                v4u fw[kWin];
                if (do_pv) {
                    // ---- O^T += V^T P^T of the previous tile; the window is refilled with the
                    // first K fragments of this tile while the last MFMAs run
#pragma unroll
                    for (int i = 0; i < kWin; ++i) fw[i] = vfrag(i);
#pragma unroll
                    for (int f = 0; f < NV; ++f) {
                        o[0][f % DB] = mfma16(fw[f % kWin], pb[0][f / DB], o[0][f % DB]);
                        o[1][f % DB] = mfma16(fw[f % kWin], pb[1][f / DB], o[1][f % DB]);
                        const int g = f + kWin;
                        fw[f % kWin] = g < NV ? vfrag(g) : kfrag(g - NV);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x100, 2 * kWin, 0);
#pragma unroll
                    for (int f = 0; f < NV - kWin; ++f) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
                        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                    }
#pragma unroll
                    for (int f = NV - kWin; f < NV; ++f) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < kWin; ++i) fw[i] = kfrag(i);
                }
                if (do_qk) {
                    f32x4 s[2][4];
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                        for (int kb = 0; kb < 4; ++kb) s[nb][kb] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int f = 0; f < NK; ++f) {
                        s[0][f & 3] = mfma16(fw[f % kWin], qreg[0][f >> 2], s[0][f & 3]);
                        s[1][f & 3] = mfma16(fw[f % kWin], qreg[1][f >> 2], s[1][f & 3]);
                        if (f + kWin < NK) fw[f % kWin] = kfrag(f + kWin);
                    }
#pragma unroll
                    for (int f = 0; f < NK; ++f) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
                        if (f + kWin < NK) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
                    mask_tile(s, j0);
                    softmax_phase(s);
                }
            }
        }
        // stage tile t+1 (already in registers), prefetch tile t+2
        if (t + 1 < ntiles) {
            const int vnext = vslot == VSLOTS - 1 ? 0 : vslot + 1;
            st.store(ldsK + ((t + 1) & 1) * KTILE, ldsV + vnext * VTILE);
            if (t + 2 < ntiles) {
                const size_t off = (size_t)(j0 + 2 * BN) * D;
                st.load(Kg + off, Vg + off, n - (j0 + 2 * BN));
            }
        }
        vslot = vslot == VSLOTS - 1 ? 0 : vslot + 1;
        __syncthreads();
    }
    if (lag && tl == ntiles - 1) {
        // the lagging waves (three V slots) still owe the P.V of their last tile (slot (ntiles-1) % 3)
        const u16 *sv = ldsV + (vslot == 0 ? 2 : vslot - 1) * VTILE + v_frag0;
#pragma unroll
        for (int f = 0; f < NV; ++f) {
            const int kp = f / DB, db = f % DB;
            const v2u lo = lds_read_tr16(sv + (32 * kp) * KROW + 16 * db);
            const v2u hi = lds_read_tr16(sv + (32 * kp + 16) * KROW + 16 * db);
            const v4u a = {lo.x, lo.y, hi.x, hi.y};
            o[0][db] = mfma16(a, pb[0][kp], o[0][db]);
            o[1][db] = mfma16(a, pb[1][kp], o[1][db]);
        }
    }

    if (SPLIT && slot >= 0) {
        // a partial result: every row of the slot is written (a wave that saw no key leaves m = -inf, l = 0)
        float *po = p.part_o + (size_t)slot * p.part_rows * D;
        float2 *pml = p.part_ml + (size_t)slot * p.part_rows;
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            const int row = row0 + rstep * (16 * nb + ln);
            float l_tot = l_run[nb] + __shfl_xor(l_run[nb], 16);
            l_tot += __shfl_xor(l_tot, 32);
            if (row >= rows) continue;
            const int pr = row - rb * ROWS;
#pragma unroll
            for (int db = 0; db < DB; ++db)
                *(f32x4 *)(po + (size_t)pr * D + db * 16 + 4 * lg) = o[nb][db];
            if (lg == 0) pml[pr] = make_float2(m_run[nb] * c, l_tot);
        }
        return;
    }
    if (!SPLIT && wave_last_key < 0) return;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        const int row = row0 + rstep * (16 * nb + ln);
        float l_tot = l_run[nb] + __shfl_xor(l_run[nb], 16);
        l_tot += __shfl_xor(l_tot, 32);
        if (row >= rows) continue;
        int chunk_row;
        size_t head;
        locate(nb, chunk_row, head);
        const float inv = 1.0f / l_tot;
        u16 *dst = (u16 *)p.out + head * p.o_hs + (size_t)chunk_row * p.o_rs;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            v2u w;
            w.x = pack_bf16x2(o[nb][db][0] * inv, o[nb][db][1] * inv);
            w.y = pack_bf16x2(o[nb][db][2] * inv, o[nb][db][3] * inv);
            *(v2u *)(dst + db * 16 + 4 * lg) = w;
        }
        if (lg == 0) p.lse[head * p.Ct + chunk_row] = (m_run[nb] * c + __builtin_amdgcn_logf(l_tot)) * kLn2;
    }
}

// SPLIT: for problems with few row blocks (a generated token has one per KV head) or a number of them
// that fills the last round of workgroups badly.  A KV head's key tiles, over all its row
// blocks, form one list, with p.start empty places before each row block's tiles for the time it
// takes to begin one (without a cache the first ones have a tile or two: 5000 rows, 14/2 heads, with the
// score 263 us without the empty places, 212 with four); `shares` workgroups take equal parts of it, whatever row
// blocks these cut through.  A row block that one workgroup covers alone is finished there, the pieces of the
// others are merged by attn_fwd_merge.  blockIdx % Hkv is the KV head in both forms, so with
// eight of them an XCD's L2 sees one head's K/V.
template <int D, int NW, bool SPLIT>
__global__ __launch_bounds__(NW * 64, NW == kFwdWaves ? 2 : kFwdNarrowResident<D>) void attn_fwd_bf16(AttnParams p)
{
    extern __shared__ __attribute__((aligned(16))) u16 smem[];
    const int bid = blockIdx.x;
    const int kvh = bid % p.Hkv;
    if constexpr (SPLIT) {
        const int share = bid / p.Hkv;
        const int begin = fwd_share_begin(p, share), end = fwd_share_begin(p, share + 1);
        FwdWalk<AttnParams, NW * 32> w(p);
        while (w.pos + w.nt <= begin) w.next(p);
        bool first = true;
        while (w.pos < end) {
            const int t0 = max(begin - w.pos, 0), t1 = min(end - w.pos, w.nt);      // t0 < nt, t1 > 0
            if (!first) __syncthreads();                 // lagging waves still read the last V tile
            first = false;
            fwd_segment<D, NW, true>(p, smem, kvh, w.rb, t0, t1, fwd_slot(p, share, kvh, t0, t1, w.nt));
            w.next(p);
        }
    } else {
        // block -> (kv head, row block); heavy (late) row blocks first
        fwd_segment<D, NW, false>(p, smem, kvh, p.n_row_blocks - 1 - bid / p.Hkv, 0, 0, -1);
    }
}

// The split pass of at most 16 query rows (a generated token), which is bound by reading K and V and,
// when they are short, by the time to start.  Nothing is shared between the waves: each takes every
// eighth 32-key tile of the share, K as A operands straight from global memory and V through LDS of
// its own (for the transposing loads), the next tile's loads in flight over this one's work, and no
// barrier until the waves' sums meet at the end.  In the general form all eight waves stage every
// tile and one of them computes: one token, 32/8 heads over 16640 keys (68 MB) 16.0 -> 13.8 us (4.9
// TB/s), 2048 keys 8.2 -> 5.9 us; with the merge, 16/4 heads of 64 over 65000 keys 21.3 -> 16.7 us.
// A form of 32 rows was slower than the general one (8 rows of 32/8 heads over 30000 keys 25.7 -> 27.4).
template <int D>
__global__ __launch_bounds__(kFwdWaves * 64) void attn_fwd_few(AttnParams p)
{
    constexpr int NW = kFwdWaves, KS = D / 32, DB = D / 16, C8 = D / 8, VP = D / 16;
    constexpr int VROW = D + 16, OROW = D + 4, R = 16;
    __shared__ __attribute__((aligned(16))) union { u16 v[NW][32 * VROW]; float o[NW / 2][R][OROW]; } sh;
    __shared__ float sm[NW][R], sl[NW][R];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ln = lane & 15, lg = lane >> 4;
    const int kvh = blockIdx.x % p.Hkv, share = blockIdx.x / p.Hkv;
    const int begin = fwd_share_begin(p, share), end = fwd_share_begin(p, share + 1);
    const int s1 = min(2 * end, (p.n + 31) / 32);
    const int rows = p.G * p.Ct;
    const u16 *Kg = (const u16 *)p.k + (size_t)kvh * p.cap * D;
    const u16 *Vg = (const u16 *)p.v + (size_t)kvh * p.cap * D;

    v4u kreg[2][KS], vreg[VP];
    auto load = [&](int s) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const u16 *src = Kg + (size_t)min(s * 32 + kb * 16 + ln, p.n - 1) * D + 8 * lg;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) kreg[kb][ks] = *(const v4u *)(src + ks * 32);
        }
#pragma unroll
        for (int i = 0; i < VP; ++i)
            vreg[i] = *(const v4u *)(Vg + (size_t)min(s * 32 + lane / C8 + i * (64 / C8), p.n - 1) * D + lane % C8 * 8);
    };
    int s = 2 * begin + wave;
    if (s < s1) load(s);
    v4u qreg[KS];
    const int row = min(ln, rows - 1), chunk_row = row / p.G, lim = p.M + chunk_row;   // last key the row sees
    {
        const u16 *src = (const u16 *)p.q + (size_t)(kvh * p.G + row % p.G) * p.q_hs + (size_t)chunk_row * p.q_rs + 8 * lg;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qreg[ks] = *(const v4u *)(src + ks * 32);
    }
    f32x4 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = (f32x4){0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;
    const float c = p.scale * kLog2e;
    u16 *sv = sh.v[wave];
    for (; s < s1; s += NW) {
        const int j0 = s * 32;
#pragma unroll
        for (int i = 0; i < VP; ++i) *(v4u *)(sv + (lane / C8 + i * (64 / C8)) * VROW + lane % C8 * 8) = vreg[i];
        f32x4 x[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) x[kb] = mfma16(kreg[kb][ks], qreg[ks], x[kb]);
        if (s + NW < s1) load(s + NW);
        float mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (j0 + (e >> 2) * 16 + 4 * lg + (e & 3) > lim) x[e >> 2][e & 3] = -INFINITY;
            mx = fmaxf(mx, x[e >> 2][e & 3]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m, mx);
        const float ref = m_new == -INFINITY ? 0.f : m_new * c;         // -inf: the row sees no key yet
        const float alpha = __builtin_amdgcn_exp2f(fmaf(m, c, -ref));
        m = m_new;
        float pv[8], sum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            pv[e] = __builtin_amdgcn_exp2f(fmaf(x[e >> 2][e & 3], c, -ref));
            sum += pv[e];
        }
        l = fmaf(l, alpha, sum);
#pragma unroll
        for (int db = 0; db < DB; ++db) o[db] *= alpha;
        const v4u pb = {pack_bf16x2(pv[0], pv[1]), pack_bf16x2(pv[2], pv[3]), pack_bf16x2(pv[4], pv[5]),
                        pack_bf16x2(pv[6], pv[7])};
        const u16 *vf = sv + (4 * lg + (ln >> 2)) * VROW + 4 * (ln & 3);      // see lds_read_tr16
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const v2u lo = lds_read_tr16(vf + 16 * db), hi = lds_read_tr16(vf + 16 * VROW + 16 * db);
            o[db] = mfma16((v4u){lo.x, lo.y, hi.x, hi.y}, pb, o[db]);
        }
    }
    // the waves' sums: scaled to the common maximum, the upper half's handed to the lower half's, and
    // those added up on the way out
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (lg == 0) { sm[wave][ln] = m; sl[wave][ln] = l; }
    __syncthreads();                                     // also: the last V tiles have been read
    float m_all = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) m_all = fmaxf(m_all, sm[w][ln]);
    const float f = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m - m_all) * c);
#pragma unroll
    for (int db = 0; db < DB; ++db) {
        o[db] *= f;
        if (wave >= NW / 2) *(f32x4 *)&sh.o[wave - NW / 2][ln][db * 16 + 4 * lg] = o[db];
    }
    __syncthreads();
    if (wave < NW / 2) {
#pragma unroll
        for (int db = 0; db < DB; ++db) *(f32x4 *)&sh.o[wave][ln][db * 16 + 4 * lg] += o[db];
    }
    __syncthreads();
    const size_t slot = (size_t)blockIdx.x * 2 + (begin == 0 ? 1 : 0);      // as in attn_fwd_bf16
    float *po = p.part_o + slot * p.part_rows * D;
    float2 *pml = p.part_ml + slot * p.part_rows;
    for (int t = threadIdx.x; t < rows * (D / 4); t += NW * 64) {
        const int r = t / (D / 4), c4 = t % (D / 4) * 4;
        f32x4 y = *(const f32x4 *)&sh.o[0][r][c4];
#pragma unroll
        for (int w = 1; w < NW / 2; ++w) y += *(const f32x4 *)&sh.o[w][r][c4];
        *(f32x4 *)(po + (size_t)r * D + c4) = y;
        if (c4 == 0) {
            float m_row = -INFINITY, l_row = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) m_row = fmaxf(m_row, sm[w][r]);
#pragma unroll
            for (int w = 0; w < NW; ++w)                 // multiplied, not left out: NaN logits alone leave -inf and a NaN sum
                l_row += sl[w][r] * (sm[w][r] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((sm[w][r] - m_row) * c));
            pml[r] = make_float2(m_row * c, l_row);
        }
    }
}

// The whole pass of 32 query rows by one workgroup, for problems of few rows and not too many keys: each wave takes every NW-th
// 32-key tile, as in attn_fwd_few, and their sums meet in LDS, so there are eight times as many workgroups as row
// blocks of attn_fwd_bf16, no barrier before the end, no pieces and no launch that merges them.  Bound: K and V, which every
// workgroup reads by itself, at what a compute unit gets from the L2 (32 keys of 256 bytes 0.2 us).  So both are read as
// whole rows and pass through LDS of the wave's own: with K as A operands straight from memory, 64 bytes of a row at a time, 739
// rows over 1691 keys, 8/8 heads 20.5 us, so 18.4.  Eight waves where every workgroup has a compute unit, else four (102 rows
// over 3078, 32/8 heads of 64 14.6, four 18.1; 302 over 346, 32/32 13.1, four 10.1).  Attention alone, attn_fwd_bf16's plan /
// this, us: 64 wide, 60 rows over 1060 keys, 32/8 heads 15.4 / 9.2; 767 over 841, 4/4 14.5 / 7.6; 600 over 600, 32/8 12.4 / 8.6;
// 128 wide, 130 over 1130, 32/8 19.9 / 13.6; 300 over 300, 32/8 12.2 / 9.9; 300 over 1300, 8/8 16.9 / 14.5, 14/2 19.1 / 14.9.
// SPLIT: each row block's key tiles in equal parts to p.shares workgroups, which leave pieces; with longer caches a block of 256
// rows shared out leaves eight times the bytes (attention alone: 137 rows over 2287, 14/2 heads of 128 19.2 -> 14.7 us, 90 over
// 9054, 16/4 of 64 19.7 -> 15.0, 150 over 4008, 24/8 of 128 26.7 -> 22.9).  Where it is taken: fwd_short.
template <int D, int NW, bool SPLIT>
__global__ __launch_bounds__(NW * 64, 2) void attn_fwd_short(AttnParams p)
{
    constexpr int NB = 2, KS = D / 32, DB = D / 16, C8 = D / 8, VP = D / 16;
    constexpr int VROW = D + 16, OROW = D + 4, R = kFwdShortRows, TILE = 32 * VROW;
    static_assert(R == 16 * NB, "two query blocks to a wave");
    __shared__ __attribute__((aligned(16))) union { u16 kv[NW][2 * TILE]; float o[NW / 2][R][OROW]; } sh;
    __shared__ float sm[NW][R], sl[NW][R];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ln = lane & 15, lg = lane >> 4;
    const int kvh = blockIdx.x % p.Hkv, rows = p.G * p.Ct;
    const int group = blockIdx.x / p.Hkv, share = SPLIT ? group % p.shares : 0;
    const int rb = p.n_row_blocks - 1 - (SPLIT ? group / p.shares : group);        // late (long) ones first
    const int row0 = rb * R, rows_here = min(R, rows - row0);
    const int all = fwd_short_tiles(p, rb);
    const int begin = SPLIT ? fwd_short_begin(p, all, share) : 0, tiles = SPLIT ? fwd_short_begin(p, all, share + 1) : all;
    const u16 *Kg = (const u16 *)p.k + (size_t)kvh * p.cap * D;
    const u16 *Vg = (const u16 *)p.v + (size_t)kvh * p.cap * D;

    // 16-byte pieces of a tile: piece i of a lane lies in row lane / C8 + i * (64 / C8)
    v4u kreg[VP], vreg[VP];
    const uint32_t off0 = (uint32_t)(lane / C8 * D + lane % C8 * 8) * 2u;
    auto load = [&](int s) {
        const char *kt = (const char *)(Kg + (size_t)s * 32 * D), *vt = (const char *)(Vg + (size_t)s * 32 * D);
        const int last = p.n - 1 - s * 32;
        if (last >= 31) {
#pragma unroll
            for (int i = 0; i < VP; ++i) {
                kreg[i] = *(const v4u *)(kt + (off0 + (uint32_t)(i * 128 / C8 * D)));
                vreg[i] = *(const v4u *)(vt + (off0 + (uint32_t)(i * 128 / C8 * D)));
            }
        } else {                                         // rows past the end repeat the last one
#pragma unroll
            for (int i = 0; i < VP; ++i) {
                const uint32_t off = (uint32_t)(min(lane / C8 + i * (64 / C8), last) * D + lane % C8 * 8) * 2u;
                kreg[i] = *(const v4u *)(kt + off);
                vreg[i] = *(const v4u *)(vt + off);
            }
        }
    };
    int s = begin + wave;
    if (s < tiles) load(s);
    v4u qreg[NB][KS];
    int lim[NB];                                         // last key the row sees
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int row = min(row0 + nb * 16 + ln, rows - 1), chunk_row = row / p.G;
        lim[nb] = p.M + chunk_row;
        const u16 *src = (const u16 *)p.q + (size_t)(kvh * p.G + row % p.G) * p.q_hs + (size_t)chunk_row * p.q_rs + 8 * lg;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qreg[nb][ks] = *(const v4u *)(src + ks * 32);
    }
    f32x4 o[NB][DB];
    float m[NB], l[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        m[nb] = -INFINITY;
        l[nb] = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db) o[nb][db] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    const float c = p.scale * kLog2e;
    u16 *sk = sh.kv[wave], *sv = sk + TILE;
    for (; s < tiles; s += NW) {
        const int j0 = s * 32;
#pragma unroll
        for (int i = 0; i < VP; ++i) {
            const int at = (lane / C8 + i * (64 / C8)) * VROW + lane % C8 * 8;
            *(v4u *)(sk + at) = kreg[i];
            *(v4u *)(sv + at) = vreg[i];
        }
        if (s + NW < tiles) load(s + NW);
        f32x4 x[NB][2];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) x[nb][0] = x[nb][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                const v4u a = *(const v4u *)(sk + (kb * 16 + ln) * VROW + 8 * lg + ks * 32);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) x[nb][kb] = mfma16(a, qreg[nb][ks], x[nb][kb]);
            }
        if (j0 + 31 > p.M + row0 / p.G) {
            asm volatile("; mask path" ::: "memory");
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (j0 + (e >> 2) * 16 + 4 * lg + (e & 3) > lim[nb]) x[nb][e >> 2][e & 3] = -INFINITY;
        }
        // as in attn_fwd_bf16: against the reference so far, and anew with the true maximum where a row outgrew it
        v4u pb[NB];
        float rs[NB];
        bool big = false;
        auto probabilities = [&](int nb, float ref) {
            float pv[8];
            rs[nb] = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                pv[e] = __builtin_amdgcn_exp2f(fmaf(x[nb][e >> 2][e & 3], c, -ref));
                rs[nb] += pv[e];
            }
            pb[nb] = (v4u){pack_bf16x2(pv[0], pv[1]), pack_bf16x2(pv[2], pv[3]), pack_bf16x2(pv[4], pv[5]),
                           pack_bf16x2(pv[6], pv[7])};
        };
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            probabilities(nb, m[nb] * c);
            big = big || !(rs[nb] < kBigSum);
        }
        if (__builtin_amdgcn_ballot_w64(big) != 0ull) {
            asm volatile("; rescale path" ::: "memory");
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                float mx = -INFINITY;
#pragma unroll
                for (int e = 0; e < 8; ++e) mx = fmaxf(mx, x[nb][e >> 2][e & 3]);
                mx = fmaxf(mx, __shfl_xor(mx, 16));
                mx = fmaxf(mx, __shfl_xor(mx, 32));
                const float m_new = fmaxf(m[nb], mx);
                const float ref = m_new == -INFINITY ? 0.f : m_new * c;     // -inf: the row sees no key yet
                const float alpha = __builtin_amdgcn_exp2f(fmaf(m[nb], c, -ref));
                m[nb] = m_new;
                l[nb] *= alpha;
#pragma unroll
                for (int db = 0; db < DB; ++db) o[nb][db] *= alpha;
                probabilities(nb, ref);
            }
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) l[nb] += rs[nb];
        const u16 *vf = sv + (4 * lg + (ln >> 2)) * VROW + 4 * (ln & 3);      // see lds_read_tr16
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const v2u lo = lds_read_tr16(vf + 16 * db), hi = lds_read_tr16(vf + 16 * VROW + 16 * db);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) o[nb][db] = mfma16((v4u){lo.x, lo.y, hi.x, hi.y}, pb[nb], o[nb][db]);
        }
    }
    // the waves' sums, as in attn_fwd_few
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        l[nb] += __shfl_xor(l[nb], 16);
        l[nb] += __shfl_xor(l[nb], 32);
        if (lg == 0) { sm[wave][nb * 16 + ln] = m[nb]; sl[wave][nb * 16 + ln] = l[nb]; }
    }
    __syncthreads();                                     // also: the last V tiles have been read
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        float m_all = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) m_all = fmaxf(m_all, sm[w][nb * 16 + ln]);
        const float f = m[nb] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m[nb] - m_all) * c);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            o[nb][db] *= f;
            if (wave >= NW / 2) *(f32x4 *)&sh.o[wave - NW / 2][nb * 16 + ln][db * 16 + 4 * lg] = o[nb][db];
        }
    }
    __syncthreads();
    if (wave < NW / 2) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int db = 0; db < DB; ++db) *(f32x4 *)&sh.o[wave][nb * 16 + ln][db * 16 + 4 * lg] += o[nb][db];
    }
    __syncthreads();
    for (int t = threadIdx.x; t < rows_here * (D / 4); t += NW * 64) {
        const int r = t / (D / 4), c4 = t % (D / 4) * 4;
        f32x4 y = *(const f32x4 *)&sh.o[0][r][c4];
#pragma unroll
        for (int w = 1; w < NW / 2; ++w) y += *(const f32x4 *)&sh.o[w][r][c4];
        float m_row = -INFINITY, l_row = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) m_row = fmaxf(m_row, sm[w][r]);
#pragma unroll
        for (int w = 0; w < NW; ++w)                     // multiplied, not left out: NaN logits alone leave -inf and a NaN sum
            l_row += sl[w][r] * (sm[w][r] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((sm[w][r] - m_row) * c));
        if constexpr (SPLIT) {
            const size_t at = (size_t)ShortPieces<AttnParams>(p, rb).slot(p, share, kvh) * R + r;
            *(f32x4 *)(p.part_o + at * D + c4) = y;
            if (c4 == 0) p.part_ml[at] = make_float2(m_row * c, l_row);
            continue;
        }
        const int chunk_row = (row0 + r) / p.G, head = kvh * p.G + (row0 + r) % p.G;
        const float inv = 1.0f / l_row;
        v2u w;
        w.x = pack_bf16x2(y[0] * inv, y[1] * inv);
        w.y = pack_bf16x2(y[2] * inv, y[3] * inv);
        *(v2u *)((u16 *)p.out + (size_t)head * p.o_hs + (size_t)chunk_row * p.o_rs + c4) = w;
        if (c4 == 0) p.lse[(size_t)head * p.Ct + chunk_row] = (m_row * c + __builtin_amdgcn_logf(l_row)) * kLn2;
    }
}

// List position of row block rb's first tile, by the 64 lanes of a wave.
template <int ROWS>
__device__ __forceinline__ int fwd_row_block_pos(const AttnParams &p, int rb)
{
    int pos = 0;
    for (int b = threadIdx.x & 63; b < rb; b += 64) pos += p.start + fwd_row_block_tiles<ROWS>(p, b);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) pos += __shfl_xor(pos, o);
    return pos + p.start;
}

template <int ROWS>
__device__ __forceinline__ auto row_block_pieces(const AttnParams &p, int rb)
{
    if constexpr (ROWS == kFwdShortRows) return ShortPieces<AttnParams>(p, rb);
    else return FwdPieces<AttnParams>(p, fwd_row_block_pos<ROWS>(p, rb), fwd_row_block_tiles<ROWS>(p, rb));
}

// Merges the pieces of the row blocks that several workgroups share: a group of D/4 lanes adds up
// pieces of one query row, four output columns per lane.  Each piece is a dependent load and an
// exponential, so with many pieces per row (MANY: a token's row has as many as its KV head has
// shares) all groups of a workgroup take one row together, and their sums meet in LDS: 33 pieces
// of one row 8 us with one group, 3 us with eight.  grid (KV head, rows of a row block / rows per workgroup, row block):
// the KV head is the fastest index, as in the pass that leaves the pieces, so with eight heads a head's pieces are in
// the L2 of the XCD that reads them (whole calls, us, KV head slowest / fastest, one state over and over: 300 rows over 1300
// keys, 32/8 heads 47.4 / 41.2; 40 over 2040 28.4 / 24.9; 130 over 1130, 8/8 22.7 / 21.3; 17 over 4113, 8/8 15.3 / 14.7; three
// states with a workspace each in turn: 43.3 / 42.4, 25.4 / 25.2, 22.7 / 21.3, 15.68 / 15.64).
// RPT: rows of a thread, whose pieces are asked for together; two where there are several workgroups to a unit all the same
// (attention alone, us, one / two / four rows: 3001 over 11193, 32/8 415 / 409 / 409, 1500 over 5500 120.8 / 119.2 /
// 119.3, 24/8 of 64 208.6 / 207.0 / 207.5, 2500 over 5500, 16/4 of 64 67.0 / 66.1 / 66.8; 1000 over 5000, 8/8 60.4 / - / 61.9).
template <int D, int ROWS, bool MANY, int RPT = 1>
__device__ __forceinline__ void fwd_merge(const AttnParams &p, int bx, int rb, int kvh)
{
    constexpr int L = D / 4, GROUPS = 256 / L;
    __shared__ f32x4 so[MANY ? GROUPS : 1][L];
    __shared__ float2 sml[GROUPS];
    const auto pieces = row_block_pieces<ROWS>(p, rb);
    const int j0 = pieces.j0, j1 = pieces.j1;
    if (j0 == j1) return;                                // finished by one workgroup
    const int grp = threadIdx.x / L, c4 = (threadIdx.x % L) * 4;
    // rows of this thread: pr0, pr0 + GROUPS, ...
    const int pr0 = MANY ? bx : bx * RPT * GROUPS + grp;
    const int rows_here = min(p.part_rows, p.G * p.Ct - rb * ROWS);
    if (pr0 >= rows_here) return;
    const int first = MANY ? j0 + grp : j0, step = MANY ? GROUPS : 1;
    float m[RPT], l[RPT];
    f32x4 o[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        m[i] = -INFINITY;
        l[i] = 0.f;
        o[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    auto add = [&](int i, float pm, float pl, f32x4 x) { // pm = -inf: a piece without a visible key
        const float m_new = fmaxf(m[i], pm);
        const float a = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m[i] - m_new);
        const float w = m_new == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(pm - m_new);
        m[i] = m_new;
        l[i] = fmaf(l[i], a, w * pl);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[i][e] = fmaf(o[i][e], a, w * x[e]);
    };
    constexpr int FLY = RPT == 1 ? 4 : 2;                // pieces in flight of each row
    for (int j = first; j <= j1; j += FLY * step) {
        float2 ml[FLY][RPT];
        f32x4 x[FLY][RPT];
#pragma unroll
        for (int u = 0; u < FLY; ++u) {
            const size_t at = (size_t)pieces.slot(p, min(j + u * step, j1), kvh) * p.part_rows;
#pragma unroll
            for (int i = 0; i < RPT; ++i) {
                const size_t r = at + min(pr0 + i * GROUPS, rows_here - 1);
                ml[u][i] = p.part_ml[r];
                x[u][i] = *(const f32x4 *)(p.part_o + r * D + c4);
            }
        }
#pragma unroll
        for (int u = 0; u < FLY; ++u)
            if (j + u * step <= j1) {
#pragma unroll
                for (int i = 0; i < RPT; ++i) add(i, ml[u][i].x, ml[u][i].y, x[u][i]);
            }
    }
    if constexpr (MANY) {
        so[grp][c4 / 4] = o[0];
        if (c4 == 0) sml[grp] = make_float2(m[0], l[0]);
        __syncthreads();
        if (grp) return;
        for (int g = 1; g < GROUPS; ++g) add(0, sml[g].x, sml[g].y, so[g][c4 / 4]);
    }
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        if (pr0 + i * GROUPS >= rows_here) break;
        const int r = rb * ROWS + pr0 + i * GROUPS, row = r / p.G, head = kvh * p.G + r % p.G;
        const float inv = 1.0f / l[i];
        v2u w;
        w.x = pack_bf16x2(o[i][0] * inv, o[i][1] * inv);
        w.y = pack_bf16x2(o[i][2] * inv, o[i][3] * inv);
        *(v2u *)((u16 *)p.out + (size_t)head * p.o_hs + (size_t)row * p.o_rs + c4) = w;
        if (c4 == 0) p.lse[(size_t)head * p.Ct + row] = (m[i] + __builtin_amdgcn_logf(l[i])) * kLn2;
    }
}

template <int D, int ROWS, bool MANY, int RPT>
__global__ __launch_bounds__(256) void attn_fwd_merge(AttnParams p)
{
    fwd_merge<D, ROWS, MANY, RPT>(p, blockIdx.y, blockIdx.z, blockIdx.x);
}

// ------------------------------------------------------------------------------------------
// Score: a workgroup owns NW*16*KB consecutive keys of one KV head (K^T tile held in registers
// as the A operand) and streams every observing query row of the G heads of the group through
// LDS.  Per-lane partial column sums are kept for the whole pass and reduced across the 16
// query lanes once at the end, in a fixed order: no atomics, bitwise reproducible, and two cache
// rows with identical keys get identical scores.
//
// Per logit the VALU does one v_fma (scale and -lse folded), one v_exp and one v_add; the mask is
// applied only on the tiles that straddle the causal diagonal (separate, rarely taken path), and
// rows past the chunk end are switched off through lse = +inf.
template <int D, int NT, int QT>
struct QStage {
    static constexpr int QROW = D + 16;
    static constexpr int C8 = D / 8;
    static constexpr int PIECES = QT * C8 / NT;
    static_assert(PIECES >= 1, "tile/threads mismatch");
    v4u qpre[PIECES];
    float lpre;
    bool lvalid;
    uint32_t goff, gstep;     // byte offset of this thread's first piece inside a tile, step per piece
    uint32_t loff;            // element offset inside the LDS tile
    int row0;

    __device__ __forceinline__ void init(int tid, long q_rs)
    {
        row0 = tid / C8;
        goff = (uint32_t)((long)row0 * q_rs * 2 + (tid % C8) * 16);
        gstep = (uint32_t)((long)(NT / C8) * q_rs * 2);
        loff = (uint32_t)(row0 * QROW + (tid % C8) * 8);
        lpre = 0.f;
        lvalid = false;
    }
    // Qt: first row of the tile (uniform); lse_t: lse of that row; rows_left = Ct - i0 (>= 1)
    __device__ __forceinline__ void load(const u16 *Qt, const float *lse_t, int rows_left, long q_rs, int tid)
    {
        // rows this far apart at most lie within 32 bits of the tile's first; a branch per tile, which is the same for all
        // waves and costs no registers, while 64-bit offsets would cost two to a piece
        constexpr long kFar = (0xffffffffl - 2 * D) / (2 * (QT - 1));
        const char *qb = (const char *)Qt;
        if (rows_left >= QT && q_rs <= kFar) {
#pragma unroll
            for (int i = 0; i < PIECES; ++i) qpre[i] = *(const v4u *)(qb + (goff + gstep * (uint32_t)i));
        } else {
#pragma unroll
            for (int i = 0; i < PIECES; ++i) {
                int r = row0 + i * (NT / C8);
                r = r < rows_left ? r : rows_left - 1;
                qpre[i] = *(const v4u *)(qb + ((size_t)r * q_rs * 2 + (tid % C8) * 16));
            }
        }
        // raw value only: multiplying here would wait for the load right after issuing it
        if (tid < QT) {
            lvalid = tid < rows_left;
            lpre = lvalid ? lse_t[tid] : 0.f;
        }
    }
    __device__ __forceinline__ void store(u16 *dq, float *dl, int tid) const
    {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) *(v4u *)(dq + loff + i * (NT / C8) * QROW) = qpre[i];
        if (tid < QT) dl[tid] = lvalid ? lpre * kLog2e : INFINITY;
    }
};

// A wave holds 64 keys (four 16-key blocks) as A operands for the whole pass; query rows stream
// through LDS as B operands, two 16-row blocks at a time; a lane owns one query column of each
// block and 4 keys per key block.  The MFMA shape and the operand order were chosen by
// measurement under the power cap (random bf16 operands): 16x16x32 sustains 2.03 PFLOP/s in a
// pure MFMA loop against 1.83 for 32x32x16, and an A operand that is held for two MFMAs while B
// alternates between two registers costs 4 % less than a new A operand on every MFMA.  The
// 32x32x16 form of this kernel (32 keys x 32 rows per MFMA, new key fragment every MFMA) was
// 1.2 % slower.
//
// KB = 2 (the narrow form): a wave holds 32 keys, in 107 registers at head_dim 64 and 158 at 128, so that four or three
// waves share a SIMD instead of two.  At 64 a logit costs half the MFMAs and the same VALU work, which then is the bound
// (v_fma, v_exp and v_add 17 cycles, its MFMAs 8, most of which do not overlap), so what counts is that some wave always has
// VALU work to issue (three waves per SIMD with 64 keys spill and gain half as much, five with 32 spill); six VALU instructions follow an
// MFMA there, not three.  At 128 it serves passes of up to some 250 us, whose starts it hides; longer ones are bound by the
// power budget.  Score alone, back to back: 64 wide, 8192 rows over 16384 keys, 16/4 heads 334 -> 289 us (VALU busy 0.60 ->
// 0.74 of the cycles); 16384 over 24576, 32/8 1697 -> 1423; 1000 over 4000, 32/8 44.6 -> 36.4; 128 of 3001 rows over 11193,
// 24/8 19.7 -> 15.0; 128 wide, 1000 over 3000, 32/8 48.7 -> 38.6; 500 over 4596, 8/8 23.3 -> 16.7.  See score_plan.
//
// WINDOW: not every row observes.  Without it the first observing row is 0 at compile time.
//
// QT: rows of a query tile, between two barriers.  A wave that waits at one leaves its SIMD to a single wave, which hides
// neither its exponentials nor its MFMAs, so long passes of eight waves take tiles of 192 rows (64, 128, 192: 12.13, 11.89, 11.76
// ms for 32768 rows over 65536 keys, 32/8 heads; 256 spill).  With two or more workgroups on a unit one computes while the other
// waits, and 128 rows give nothing (8192 over 16384 809, 822 us).
//
// SPREAD: the exponentials of both units of a loop trip lie between MFMAs.  Left alone the compiler finds the same flush of the
// pending unit on both sides of the diagonal branch and moves it in front, so that every other unit's VALU work runs by itself.
// us, moved / spread: 8192 rows over 16384, 32/8 heads 827 / 818, 16/4 of 64 298 / 295, 32768 over 65536, 32/8 of 64 8530 /
// 8430; but eight waves with tiles of 64 rows 12.01 / 12.13 ms, 25 over 15606 15.86 / 16.03, and windows at 64, of a few trips,
// 14.9 / 15.1: those keep the former.
template <int D, int KB, int NW, bool WINDOW, int QT>
__global__ __launch_bounds__(NW * 64, KB == 2 ? (D == 64 ? 4 : 3) : 2) void attn_score_bf16(AttnParams p)
{
    constexpr int NT = NW * 64;
    constexpr int KS = D / 32;                           // MFMA k-steps
    using Stage = QStage<D, NT, QT>;
    constexpr int QROW = Stage::QROW;
    constexpr int WKEYS = 16 * KB;
    constexpr bool SPREAD = D == 128 ? NW == 4 || QT > 64 : !WINDOW;
    constexpr int NQB = QT / 16;                         // 16-row query blocks per tile
    static_assert(NQB % 4 == 0, "the rotation below alternates two units of two query blocks");

    __shared__ __attribute__((aligned(16))) u16 ldsQ[2][QT * QROW];
    __shared__ float ldsL[2][QT];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int ln = lane & 15;
    const int lg = lane >> 4;

    const int kvh = blockIdx.x % p.Hkv;
    const int nkt = (p.n + NW * WKEYS - 1) / (NW * WKEYS);
    const int slice = p.slices - 1 - blockIdx.x / p.Hkv / nkt;
    const int tile_slice = slice / p.head_slices;
    const int g0 = slice % p.head_slices * p.slice_heads, heads = min(p.slice_heads, p.G - g0);
    const int kt = blockIdx.x / p.Hkv % nkt;
    const int j_wg = kt * (NW * WKEYS);
    const int jw = j_wg + wave * WKEYS;

    const int i_lo = WINDOW ? p.Ct - p.W : 0;            // first observing row
    const int i_first = max(i_lo, max(j_wg - p.M, 0));   // first row that both observes and sees j_wg
    // query tiles of this slice, counted from the first observing row for every key block: a window of 128 rows
    // is two tiles wherever it begins, not three (whole calls: 128 of 3001 rows over 11193 keys, 24/8 heads of 64 235.4
    // -> 229.2 us, 128 of 400 over 30400, 14/2 heads of 64 94.7 -> 85.3 us)
    const int s_lo = tile_slice * p.slice_tiles;
    const int qt0 = max((i_first - i_lo) / QT, s_lo);
    const int ntq = min(((WINDOW ? p.W : p.Ct) + QT - 1) / QT, s_lo + p.slice_tiles) - qt0;    // per head
    if (ntq <= 0) return;                                // the whole slice lies before the diagonal
    const int i_base = i_lo + qt0 * QT;

    const u16 *Kg = (const u16 *)p.k + (size_t)kvh * p.cap * D;
    v4u kreg[KB][KS];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        int key = jw + kb * 16 + ln;
        key = key < p.n ? key : p.n - 1;
        const u16 *src = Kg + (size_t)key * D + 8 * lg;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kreg[kb][ks] = *(const v4u *)(src + ks * 32);
    }

    f32x4 col[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) col[kb] = (f32x4){0.f, 0.f, 0.f, 0.f};

    const int iters = heads * ntq;
    const float c = p.scale * kLog2e;
    const int q_frag0 = ln * QROW + 8 * lg;

    Stage st;
    st.init(tid, p.q_rs);
    auto load_q = [&](int it) {
        const int head = kvh * p.G + g0 + it / ntq;
        const int i0 = i_base + it % ntq * QT;
        st.load((const u16 *)p.q + (size_t)head * p.q_hs + (size_t)i0 * p.q_rs,
                p.lse + (size_t)head * p.Ct + i0, p.Ct - i0, p.q_rs, tid);
    };
    load_q(0);
    st.store(ldsQ[0], ldsL[0], tid);
    if (iters > 1) load_q(1);
    __syncthreads();

    // Rotation inside a wave, in units of two adjacent 16-row query blocks: the 32 MFMAs of a unit
    // are interleaved, one MFMA to three VALU instructions, with the v_fma / v_exp / v_add work of
    // the PREVIOUS unit, which never waits for the MFMAs in flight.  Every key fragment (A
    // operand) is used for two MFMAs in a row, the B operand alternating between the unit's two
    // query blocks.  `sB` / `lsB0`, `lsB1` carry the unit whose VALU work is pending; lse = +inf
    // makes a block contribute exactly 0 (the empty state).
    f32x4 sA[2][KB], sB[2][KB];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) sB[h][kb] = (f32x4){0.f, 0.f, 0.f, 0.f};
    float lsB0 = INFINITY, lsB1 = INFINITY;
    auto issue_mfma2 = [&](f32x4 (&dst)[2][KB], const u16 *src) {
        v4u bq0[KS], bq1[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            bq0[ks] = *(const v4u *)(src + ks * 32);
            bq1[ks] = *(const v4u *)(src + 16 * QROW + ks * 32);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) dst[h][kb] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                dst[0][kb] = mfma16(kreg[kb][ks], bq0[ks], dst[0][kb]);
                dst[1][kb] = mfma16(kreg[kb][ks], bq1[ks], dst[1][kb]);
            }
    };
    auto accumulate2 = [&](const f32x4 (&src)[2][KB], float ls0, float ls1) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                col[kb][e] += __builtin_amdgcn_exp2f(fmaf(src[0][kb][e], c, -ls0));
                col[kb][e] += __builtin_amdgcn_exp2f(fmaf(src[1][kb][e], c, -ls1));
            }
    };
    f32x4 sD[KB];                          // diagonal path: one 16-row block at a time
    auto issue_mfma = [&](f32x4 (&dst)[KB], const u16 *src) {
        v4u bq[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) bq[ks] = *(const v4u *)(src + ks * 32);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) dst[kb] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) dst[kb] = mfma16(kreg[kb][ks], bq[ks], dst[kb]);
    };
    auto interleave_pattern = [&]() {
        __builtin_amdgcn_sched_group_barrier(0x100, 2 * KS, 0);
#pragma unroll
        for (int u = 0; u < 2 * KS * KB; ++u) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);     // one MFMA ...
            if constexpr (SPREAD) {
                __builtin_amdgcn_sched_group_barrier(0x400, 128 / D, 0);   // ... then its share of the exponentials
                __builtin_amdgcn_sched_group_barrier(0x002, 256 / D, 0);   // and of the other VALU work
            } else {
                __builtin_amdgcn_sched_group_barrier(0x402, 384 / D, 0);
            }
        }
    };
    for (int it = 0; it < iters; ++it) {
        const int buf = it & 1;
        const int i0 = i_base + it % ntq * QT;
        if (jw < p.n) {
            const u16 *sq = ldsQ[buf] + q_frag0;
            if (jw + WKEYS - 1 <= p.M + i0) {
                // ---- every row of the tile sees every key of this wave
#pragma unroll
                for (int qb = 0; qb < NQB; qb += 4) {
                    if (qb > 0 && 16 * qb >= p.Ct - i0) break;   // groups of 64 rows past the chunk's end
                    const float l0 = ldsL[buf][16 * qb + ln], l1 = ldsL[buf][16 * qb + 16 + ln];
                    const float l2 = ldsL[buf][16 * qb + 32 + ln], l3 = ldsL[buf][16 * qb + 48 + ln];
                    if constexpr (SPREAD) __builtin_amdgcn_sched_barrier(0);
                    issue_mfma2(sA, sq + 16 * qb * QROW);
                    accumulate2(sB, lsB0, lsB1);
                    interleave_pattern();
                    __builtin_amdgcn_sched_barrier(0);
                    issue_mfma2(sB, sq + (16 * qb + 32) * QROW);
                    accumulate2(sA, l0, l1);
                    interleave_pattern();
                    __builtin_amdgcn_sched_barrier(0);
                    lsB0 = l2;
                    lsB1 = l3;
                }
            } else {
                if constexpr (SPREAD) asm volatile("; diagonal path" : "+v"(lsB0), "+v"(lsB1) :: "memory");
                else asm volatile("; diagonal path" ::: "memory");
                accumulate2(sB, lsB0, lsB1);          // flush the pending unit first
                lsB0 = INFINITY;
                lsB1 = INFINITY;
#pragma unroll 1
                for (int qb = 0; qb < NQB; ++qb) {
                    const int r0 = i0 + qb * 16;                 // first row of this 16-row block
                    if (jw > p.M + r0 + 15) continue;            // no row of the block sees any key
                    issue_mfma(sD, sq + qb * 16 * QROW);
                    const float ls = ldsL[buf][qb * 16 + ln];
                    const int lim = p.M + r0 + ln - jw;          // key offset <= lim is visible
#pragma unroll
                    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int koff = kb * 16 + 4 * lg + e;
                            const float pv = __builtin_amdgcn_exp2f(fmaf(sD[kb][e], c, -ls));
                            col[kb][e] += koff > lim ? 0.f : pv;
                        }
                }
            }
        }
        if (it + 1 < iters) {
            st.store(ldsQ[buf ^ 1], ldsL[buf ^ 1], tid);
            if (it + 2 < iters) load_q(it + 2);
        }
        __syncthreads();
    }
    accumulate2(sB, lsB0, lsB1);               // flush the last pending unit

    if (jw >= p.n) return;
    const bool partial = p.slices > 1;
    float *dst = partial ? p.part_score + ((size_t)slice * p.Hkv + kvh) * p.n : p.score + (size_t)kvh * p.cap;
    const bool add = p.accumulate && !partial;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float x = col[kb][e];
#pragma unroll
            for (int off = 8; off >= 1; off >>= 1) x += __shfl_xor(x, off);    // over the 16 query lanes
            const int j = jw + kb * 16 + 4 * lg + e;
            if (ln == 0 && j < p.n) dst[j] = add ? dst[j] + x : x;
        }
}

// Adds up the slices of every key, in order; slices that lie before a key block's diagonal were
// not written.  keys: keys of one workgroup of the score pass.  As in that pass the KV head is blockIdx % Hkv (see fwd_merge).
__global__ __launch_bounds__(256) void attn_score_sum(AttnParams p, int keys)
{
    const int j = blockIdx.x / p.Hkv * 256 + threadIdx.x, kvh = blockIdx.x % p.Hkv;
    if (j >= p.n) return;
    const int i_lo = p.Ct - p.W, i_first = max(i_lo, max(j / keys * keys - p.M, 0));
    float x = 0.f;
#pragma unroll 4
    for (int s = (i_first - i_lo) / 64 / p.slice_tiles * p.head_slices; s < p.slices; ++s)
        x += p.part_score[((size_t)s * p.Hkv + kvh) * p.n + j];
    float *dst = p.score + (size_t)kvh * p.cap + j;
    *dst = p.accumulate ? *dst + x : x;
}

// Score of few observing rows (a ragged last chunk, or the observation window of 128 rows): the keys
// are read once and hardly anything is done with each, so nothing is staged.  A wave owns 16*KB
// keys as the A operand, as above, and takes the query rows 16 at a time straight from global
// memory (the waves of a compute unit walk the same rows, so all but the first find them in the
// cache), two blocks ahead of their use: no LDS, no barrier, and four times as many workgroups.
// Row blocks are counted from the first observing row, so all cache keys see the same blocks in
// the same order (identical keys, identical scores).
//
// RW: waves of a workgroup that share their keys and divide the row blocks among themselves; their sums meet in LDS, in
// wave order.  One where the blocks are few; four where there are more of them, which then need no slices
// and no launch that adds them up.
//
// PIECES: the attention of the same call left pieces that are not merged yet; the workgroup forms the rows'
// normalisers from the pieces' maxima and sums itself, in LDS (see attn_merge_score).
template <int D, int KB, int RW, int ROWS>
__device__ __forceinline__ void score_few_keys(const AttnParams &p, int bid)
{
    constexpr bool PIECES = ROWS > 0;
    static_assert(RW == 1 || (RW == 4 && !PIECES), "one wave or all waves of the workgroup to a set of keys");
    __shared__ float slse[PIECES ? kFewBlocks * 16 : 1];
    __shared__ float part[RW > 1 ? 4 : 1][16 * KB];
    const int w16 = (p.W + 15) / 16 * 16;                // rows of a head, filled up to whole blocks
    constexpr int KS = D / 32;
    constexpr int WKEYS = 16 * KB;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ln = lane & 15, lg = lane >> 4;
    const int kvh = bid % p.Hkv;
    const int jw = ((bid / p.Hkv) * (4 / RW) + wave / RW) * WKEYS, rw = wave % RW;
    if (!PIECES && jw >= p.n) return;                    // with RW = 4 no workgroup

    const u16 *Kg = (const u16 *)p.k + (size_t)kvh * p.cap * D;
    v4u kreg[KB][KS];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        const u16 *src = Kg + (size_t)min(jw + kb * 16 + ln, p.n - 1) * D + 8 * lg;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kreg[kb][ks] = *(const v4u *)(src + ks * 32);
    }
    f32x4 col[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) col[kb] = (f32x4){0.f, 0.f, 0.f, 0.f};

    const int i_lo = p.Ct - p.W;                         // first observing row
    // first row block with a row that sees key jw; row blocks per head (a wave behind the last key: one)
    const int b0 = min(max(jw - p.M - i_lo, 0) / 16, (p.W + 15) / 16 - 1), nb = (p.W + 15) / 16 - b0;
    const int iters = p.G * nb;
    const float c = p.scale * kLog2e;

    struct Block { v4u q[KS]; float lse; };
    auto load = [&](Block &b, int it) {
        it = min(it, iters - 1);
        const int head = kvh * p.G + it / nb;
        const int row = i_lo + (b0 + it % nb) * 16 + ln, r = min(row, p.Ct - 1);
        const u16 *src = (const u16 *)p.q + (size_t)head * p.q_hs + (size_t)r * p.q_rs + 8 * lg;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) b.q[ks] = *(const v4u *)(src + ks * 32);
        if (!PIECES) b.lse = p.lse[(size_t)head * p.Ct + r];
    };
    auto use = [&](const Block &b, int it) {
        if (it >= iters) return;
        const int r0 = i_lo + (b0 + it % nb) * 16;
        f32x4 s[KB];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) s[kb] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) s[kb] = mfma16(kreg[kb][ks], b.q[ks], s[kb]);
        const float ls = r0 + ln >= p.Ct ? INFINITY
                       : PIECES ? slse[it / nb * w16 + (b0 + it % nb) * 16 + ln] : b.lse * kLog2e;
        const int lim = p.M + r0 + ln - jw;              // key offset <= lim is visible
        if (p.M + r0 >= jw + WKEYS - 1) {
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int e = 0; e < 4; ++e) col[kb][e] += __builtin_amdgcn_exp2f(fmaf(s[kb][e], c, -ls));
        } else {
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float pv = __builtin_amdgcn_exp2f(fmaf(s[kb][e], c, -ls));
                    col[kb][e] += kb * 16 + 4 * lg + e > lim ? 0.f : pv;
                }
        }
    };
    Block x, y;
    load(x, rw);
    load(y, rw + RW);
    if constexpr (PIECES) {                              // while the keys and the first rows are on their way
        // the rows lie in row block rb0 and at most the next one (with blocks of 32 rows in up to five)
        constexpr bool SHORT = ROWS == kFwdShortRows;
        const int rb0 = (p.Ct - p.W) * p.G / ROWS, rb1 = min(rb0 + 1, p.n_row_blocks - 1);
        const int pos0 = SHORT ? 0 : fwd_row_block_pos<ROWS>(p, rb0), nt0 = SHORT ? 0 : fwd_row_block_tiles<ROWS>(p, rb0);
        const int pos1 = rb1 > rb0 ? pos0 + nt0 + p.start : pos0;
        const FwdPieces<AttnParams> pc0(p, pos0, nt0), pc1(p, pos1, SHORT ? 0 : fwd_row_block_tiles<ROWS>(p, rb1));
        // T threads to a row, each over every T-th piece
        const int entries = p.G * p.W, T = merge_score_lanes(entries);
        const int e = threadIdx.x / T, sub = threadIdx.x % T;
        if (e < entries) {                               // the same for all T lanes of a row
            const int row = p.Ct - p.W + e % p.W, gi = e / p.W, r = row * p.G + gi;
            const bool second = r / ROWS > rb0;
            const int j0 = SHORT ? 0 : second ? pc1.j0 : pc0.j0, j1 = SHORT ? p.shares - 1 : second ? pc1.j1 : pc0.j1, pr = r % ROWS;
            auto slot = [&](int j) -> size_t {
                if constexpr (SHORT) return ShortPieces<AttnParams>(p, r / ROWS).slot(p, j, kvh);
                else return (second ? pc1 : pc0).slot(p, j, kvh);
            };
            float m = -INFINITY, l = 0.f;
            if (j0 < j1)
                for (int j = j0 + sub; j <= j1; j += 4 * T) {        // four pieces in flight
                    float2 x[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        x[u] = p.part_ml[slot(min(j + u * T, j1)) * p.part_rows + pr];
                        if (j + u * T > j1) x[u] = make_float2(-INFINITY, 0.f);
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const float m_new = fmaxf(m, x[u].x);        // -inf: a piece without a visible key
                        const float a = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m - m_new);
                        const float w = m_new == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(x[u].x - m_new);
                        m = m_new;
                        l = fmaf(l, a, w * x[u].y);
                    }
                }
            for (int o = 1; o < T; o <<= 1) {
                const float om = __shfl_xor(m, o), ol = __shfl_xor(l, o);
                const float m_new = fmaxf(m, om);
                const float a = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m - m_new);
                const float w = m_new == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(om - m_new);
                m = m_new;
                l = fmaf(l, a, w * ol);
            }
            if (sub == 0)
                slse[gi * w16 + e % p.W] = j0 < j1 ? m + __builtin_amdgcn_logf(l) : p.lse[(size_t)(kvh * p.G + gi) * p.Ct + row] * kLog2e;
        }
        __syncthreads();
        if (jw >= p.n) return;
    }
    for (int it = rw; it < iters; it += 2 * RW) {
        Block z;
        load(z, it + 2 * RW);
        use(x, it);
        x = z;
        load(z, it + 3 * RW);
        use(y, it + RW);
        y = z;
    }

    float *dst = p.score + (size_t)kvh * p.cap;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float t = col[kb][e];
#pragma unroll
            for (int off = 8; off >= 1; off >>= 1) t += __shfl_xor(t, off);
            const int j = jw + kb * 16 + 4 * lg + e;
            if (ln != 0) continue;
            if (RW > 1) part[wave][j - jw] = t;
            else if (j < p.n) dst[j] = p.accumulate ? dst[j] + t : t;
        }
    if constexpr (RW > 1) {
        __syncthreads();
        const int at = threadIdx.x, j = jw + at;
        if (at >= WKEYS || j >= p.n) return;
        const float t = (part[0][at] + part[1][at]) + (part[2][at] + part[3][at]);
        dst[j] = p.accumulate ? dst[j] + t : t;
    }
}

template <int D, int KB, int RW>
__global__ __launch_bounds__(256) void attn_score_few(AttnParams p)
{
    score_few_keys<D, KB, RW, 0>(p, blockIdx.x);
}

// The merge of a split forward pass and the score of few rows in one launch: a ragged last chunk is a chain of
// short launches of 3 us and more, and the score only needs the pieces' maxima and sums, a few KB.
// The first n_score workgroups are the score's, the others merge as attn_fwd_merge<D, true> does, one row
// each.  Whole calls: 17 rows over 4113 keys of 8 heads 17.7 -> 16.0 us, 25 rows over 5025, 32/8 heads 29.0 -> 25.6
// us, 200 rows (128 observe) over 6200, 8 heads 37.9 -> 34.0 us.  With the normalisers formed before the keys are asked
// for, 30 over 30030, 8 heads took 55.5 instead of 50.8 us; with those of the rows that fill up a head's block of 16 formed
// as well, one token over 20000, 14/2 heads of 64 20.5 instead of 13.3 us.  Where it is taken: merge_with_score.
template <int D, int KB, int ROWS>
__global__ __launch_bounds__(256) void attn_merge_score(AttnParams p, int n_score)
{
    const int bid = blockIdx.x - n_score;
    if (bid < 0) score_few_keys<D, KB, 1, ROWS>(p, blockIdx.x);
    else fwd_merge<D, ROWS, true>(p, bid / p.Hkv % p.part_rows, bid / p.Hkv / p.part_rows, bid % p.Hkv);
}

// ------------------------------------------------------------------------------------------
// Host-side launchers (called from the C-ABI file).
static int compute_units() { return device_compute_units() > 0 ? device_compute_units() : 256; }

template <int D, int NW, bool SPLIT>
static hipError_t launch_fwd_form(const AttnParams &p, int grid, hipStream_t st)
{
    const size_t smem = fwd_lds_bytes<D, NW>();
    auto kern = attn_fwd_bf16<D, NW, SPLIT>;
    // the kernel needs more than the default 64 KB of LDS: raised once per device, not per launch
    static std::atomic<bool> lds_raised[64];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64 || !lds_raised[dev].load(std::memory_order_acquire)) {
        e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        if (dev >= 0 && dev < 64) lds_raised[dev].store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, dim3(grid), dim3(NW * 64), smem, st, p);
    return hipGetLastError();
}

// `part` (part_bytes): scratch for partial results; true if the key range is split.
template <int D>
static bool fwd_place(AttnParams &p, bool scored, void *part, size_t part_bytes)
{
    const size_t room = part ? part_bytes : 0;
    const double est = fwd_choose(p, compute_units(), scored, room);
    p.in_short = fwd_short(p, compute_units(), est, scored, room);
    if (!p.shares) return false;
    const long slots = (long)p.shares * p.Hkv * (p.in_short ? p.n_row_blocks : 2);
    p.part_o = (float *)part;
    p.part_ml = (float2 *)(p.part_o + (size_t)slots * p.part_rows * D);
    return true;
}

template <int D, bool SPLIT>
static hipError_t launch_fwd_short(const AttnParams &p, int grid, hipStream_t st)
{
    if (SPLIT || p.in_short == 8) hipLaunchKernelGGL((attn_fwd_short<D, 8, SPLIT>), dim3(grid), dim3(512), 0, st, p);
    else hipLaunchKernelGGL((attn_fwd_short<D, 4, false>), dim3(grid), dim3(256), 0, st, p);
    return hipGetLastError();
}

// f with the rows of a row block as a constant.
template <class F>
static void with_block_rows(const AttnParams &p, F f)
{
    if (p.in_short) f(std::integral_constant<int, kFwdShortRows>{});
    else if (p.narrow) f(std::integral_constant<int, kFwdNarrowRows>{});
    else f(std::integral_constant<int, kFwdRows>{});
}

// The split pass itself.
template <int D>
static hipError_t launch_fwd_pieces(const AttnParams &p, hipStream_t st)
{
    const int grid = p.shares * p.Hkv;
    if (p.in_short) return launch_fwd_short<D, true>(p, grid * p.n_row_blocks, st);
    if (p.narrow) return launch_fwd_form<D, 4, true>(p, grid, st);
    if (p.G * p.Ct > 16) return launch_fwd_form<D, kFwdWaves, true>(p, grid, st);
    hipLaunchKernelGGL(attn_fwd_few<D>, dim3(grid), dim3(kFwdWaves * 64), 0, st, p);
    return hipGetLastError();
}

template <int D>
static hipError_t launch_fwd(const AttnParams &p, bool split, hipStream_t st)
{
    if (!split) {
        const int grid = p.Hkv * p.n_row_blocks;
        if (p.in_short) return launch_fwd_short<D, false>(p, grid, st);
        return p.narrow ? launch_fwd_form<D, 4, false>(p, grid, st) : launch_fwd_form<D, kFwdWaves, false>(p, grid, st);
    }
    const hipError_t e = launch_fwd_pieces<D>(p, st);
    if (e != hipSuccess) return e;
    // pieces of the longest row block: two or three where row blocks are many, a head's shares for a token
    const long pieces = ((long)((p.M + p.Ct - 1) / 64 + 1) * p.shares) / p.tiles + 1;
    const int groups = 256 / (D / 4);
    // (11200 rows of up to 8 pieces at head_dim 64: 19 us with a workgroup per row, 6 us without)
    const long merged_rows = (long)p.Hkv * p.n_row_blocks * p.part_rows;
    if (pieces > 12 || (pieces > 6 && merged_rows <= 2048)) {
        const dim3 mgrid(p.Hkv, p.part_rows, p.n_row_blocks);
        with_block_rows(p, [&](auto rows) {
            hipLaunchKernelGGL((attn_fwd_merge<D, decltype(rows)::value, true, 1>), mgrid, dim3(256), 0, st, p);
        });
        return hipGetLastError();
    }
    auto launch = [&](auto rpt) {
        constexpr int RPT = decltype(rpt)::value;
        const dim3 mgrid(p.Hkv, (p.part_rows + RPT * groups - 1) / (RPT * groups), p.n_row_blocks);
        with_block_rows(p, [&](auto rows) {
            hipLaunchKernelGGL((attn_fwd_merge<D, decltype(rows)::value, false, RPT>), mgrid, dim3(256), 0, st, p);
        });
    };
    if (merged_rows > 16384) launch(std::integral_constant<int, 2>{});
    else launch(std::integral_constant<int, 1>{});
    return hipGetLastError();
}

template <int D, int KB, int NW>
static hipError_t launch_score_tiled(const AttnParams &p, hipStream_t st)
{
    constexpr int keys_wg = NW * 16 * KB;
    const int grid = p.Hkv * ((p.n + keys_wg - 1) / keys_wg) * p.slices;
    // Long tiles from 512 rows on: eight waves, 512 rows over 60512 keys, 32/8 heads 275 -> 272 us, 2100 over 64100 1028 -> 998,
    // but 25 over 15606 15.9 -> 25.8.  (Passes of eight waves are uncut, so slices do not meet tiles of another size.)
    constexpr int LONG = NW == 8 && D == 128 ? 192 : 64;
    if (p.W == p.Ct && p.Ct >= 512) hipLaunchKernelGGL((attn_score_bf16<D, KB, NW, false, LONG>), dim3(grid), dim3(NW * 64), 0, st, p);
    else if (p.W == p.Ct) hipLaunchKernelGGL((attn_score_bf16<D, KB, NW, false, 64>), dim3(grid), dim3(NW * 64), 0, st, p);
    else hipLaunchKernelGGL((attn_score_bf16<D, KB, NW, true, 64>), dim3(grid), dim3(NW * 64), 0, st, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.slices == 1) return e;
    hipLaunchKernelGGL(attn_score_sum, dim3((p.n + 255) / 256 * p.Hkv), dim3(256), 0, st, p, keys_wg);
    return hipGetLastError();
}

template <int D>
static hipError_t launch_score(AttnParams p, void *part, size_t part_bytes, hipStream_t st)
{
    if (const int rw = score_few(p)) {
        constexpr int KB = kFewKB;
        const int keys = rw == 1 ? 64 * KB : 16 * KB, grid = p.Hkv * ((p.n + keys - 1) / keys);
        if (rw == 1) hipLaunchKernelGGL((attn_score_few<D, KB, 1>), dim3(grid), dim3(256), 0, st, p);
        else hipLaunchKernelGGL((attn_score_few<D, KB, 4>), dim3(grid), dim3(256), 0, st, p);
        return hipGetLastError();
    }
    const int form = score_plan(p, compute_units(), part ? part_bytes : 0);
    p.part_score = (float *)part;
    if (form == kScoreEight) return launch_score_tiled<D, 4, 8>(p, st);
    if constexpr (D == 128)
        if (form == kScoreFour) return launch_score_tiled<D, 4, 4>(p, st);
    return launch_score_tiled<D, 2, 4>(p, st);
}

// Both passes.  Where the first is split and the second takes few rows, merging and the score are one launch.
template <int D>
static hipError_t launch_both(const AttnParams &p, void *part, size_t part_bytes, hipStream_t st)
{
    AttnParams f = p;
    const bool split = fwd_place<D>(f, true, part, part_bytes);
    if (!split || !merge_with_score(f)) {
        const hipError_t e = launch_fwd<D>(f, split, st);
        return e == hipSuccess ? launch_score<D>(p, part, part_bytes, st) : e;
    }
    const hipError_t e = launch_fwd_pieces<D>(f, st);
    if (e != hipSuccess) return e;
    const int n_score = f.Hkv * ((f.n + 64 * kFewKB - 1) / (64 * kFewKB));
    const int n_merge = f.part_rows * f.n_row_blocks * f.Hkv;
    with_block_rows(f, [&](auto rows) {
        hipLaunchKernelGGL((attn_merge_score<D, kFewKB, decltype(rows)::value>), dim3(n_score + n_merge), dim3(256), 0, st, f, n_score);
    });
    return hipGetLastError();
}

// Scratch of either pass (they run one after the other and share it).
size_t attend_bf16_scratch_bytes(const AttnParams &sizes)
{
    AttnParams p = sizes;
    size_t score = 0;
    if (!score_few(p)) {
        score_plan(p, compute_units());
        score = score_slice_bytes(p);
    }
    size_t bytes = score;
    for (const bool scored : {false, true}) {
        const double est = fwd_choose(p, compute_units(), scored);
        bytes = std::max(bytes, fwd_split_bytes(p));
        if (fwd_short(p, compute_units(), est, scored)) bytes = std::max(bytes, fwd_short_bytes(p));
    }
    return bytes;
}

template <int D>
static hipError_t launch_attention(AttnParams p, void *part, size_t part_bytes, hipStream_t st)
{
    const bool split = fwd_place<D>(p, false, part, part_bytes);
    return launch_fwd<D>(p, split, st);
}

hipError_t attend_bf16_forward(const AttnParams &p, void *part, size_t part_bytes, hipStream_t st)
{
    if (p.D == 128) return launch_attention<128>(p, part, part_bytes, st);
    return launch_attention<64>(p, part, part_bytes, st);
}

hipError_t attend_bf16_score(const AttnParams &p, void *part, size_t part_bytes, hipStream_t st)
{
    if (p.D == 128) return launch_score<128>(p, part, part_bytes, st);
    return launch_score<64>(p, part, part_bytes, st);
}

// Attention and score of one call.
hipError_t attend_bf16_both(const AttnParams &p, void *part, size_t part_bytes, hipStream_t st)
{
    if (p.D == 128) return launch_both<128>(p, part, part_bytes, st);
    return launch_both<64>(p, part, part_bytes, st);
}

}  // namespace reform
