// Gather stage (Sec. 3.3 "Identification of significant inputs" and App. C.6 "Similarity search"
// of arXiv 2506.01215): cosine similarity of query embeddings with every context embedding,
// per-query top-k with lowest-index ties, union with a +-radius neighbourhood, sorted unique.
//
//   sim_bf16_mfma   streams the [N][D] bf16 store once for up to 64 queries; 16 rows x 16 queries
//                   per v_mfma_f32_16x16x32_bf16; the row norms come from a second MFMA of the row
//                   tile with itself (Gram diagonal), so the VALU does no per-element work and
//                   the kernel stays HBM-bound.
//   sim_f32_mfma    fp32 inputs: the same on v_mfma_f32_16x16x4f32.
//   sim_generic     odd shapes, and short fp32 stores with few queries: one wave per row, fp32 FMA.
//   select_topk     (select.hip) radix select of the k-th largest per query and ordered emission,
//                   which also marks the dilated hits in a bitmap of N bits.
//   union_*         count and emit the bitmap's rows ascending.
#include "common.h"

namespace reform {

hipError_t select_topk(const SelParams &p, hipStream_t st);

// ------------------------------------------------------------------------------------------
// 16x16x32 operand layout (wave64): A[m][k]: lane l holds m = l%16, k = 8*(l/16)..+7;
// B[k][n]: lane l holds n = l%16, same k;  C[m][n]: lane l holds n = l%16, m = 4*(l/16) + e.
//
// The kernel is a pure HBM stream (1 flop/byte for the dot products of one query, 16 for 16), so
// what matters is bytes in flight: 8 waves per workgroup share one LDS copy of the queries, and
// every wave keeps two chunks of kChunk 16-byte loads per lane outstanding (2 x 8 KB per wave,
// 128 KB per CU: the prefetch registers leave room for one workgroup) while the MFMAs of the
// previous chunk run.  128 registers, so that two workgroups or sixteen waves fit, spill: 37
// queries over 262144 x 1024 167 -> 257 and 219 us.
//
// NG: blocks of 16 queries that share the pass, as many as fit the LDS (up to 4).  A store row costs
// its HBM time once for all of them; they add one LDS read and one MFMA per 16 x 32 tile each, which
// at NG = 4 is still less than half of either unit's time.  37 queries over 262144 x 1024: three passes
// of 108 us -> one of 119 us; with everything behind it the call takes 407 -> 167 us.
//
// A pass begins and ends without the stream, so both ends are kept short: several query loads in flight and
// the first store chunks right behind them (before: one load, one LDS store at a time, the norms read
// back from LDS, then the first chunk), and idle loads at the end that cost no traffic (33 MB over all
// waves before).  Whole calls: 131072 x 1024, one query 76.5 -> 72.4 us; 262144 x 1024, 37 queries 170 -> 162
// us; 1048576 x 2048, 16 queries 874 -> 861 us; 50000 x 2048, 64 queries 147 -> 124 us.
//
// MAX: the pooled gather only needs the maximum over the queries, so the row's largest similarity is
// stored instead of all of them (one value per row, the maximum with what an earlier pass over
// further queries left there): 39 MB less written and read back in that example.
constexpr int kSimThreads = 512;
constexpr int kChunk = 8;            // MFMA k-steps (of 32 elements) per prefetch chunk

__device__ __forceinline__ int sim_qrow(int D)   // LDS row pitch in elements: pitch % 256 B == 32 B
{
    const int rem = (2 * D) & 255;
    return D + (((32 - rem) & 255) >> 1);
}

// FULL: dim is a multiple of 32 * kChunk, so every prefetch chunk is whole and the loads and MFMAs of
// a loop trip are unconditional (the compiler can then count the loads in flight exactly).
template <bool FULL, int NG, bool MAX>
__global__ __launch_bounds__(kSimThreads) void sim_bf16_mfma(GatherParams p)
{
    extern __shared__ __attribute__((aligned(16))) u16 qs[];   // [16 * NG][QROW]
    __shared__ float qnorm[16 * NG];
    const int D = p.D, QROW = sim_qrow(D);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ln = lane & 15, lg = lane >> 4;
    if (p.sel.pre_zeroed && p.q0 == 0)        // the selection that follows finds its histograms cleared
        sel_clear(p.sel, (long)blockIdx.x * kSimThreads + tid, (long)gridDim.x * kSimThreads);

    const long ngroups_all = (p.N + 15) / 16;
    // A workgroup streams one contiguous range of row groups (its eight waves interleaved group
    // by group): measured 1.7 % faster than handing the groups out round-robin over the grid,
    // as long as the similarity rows are not a power of two apart (the workspace pitch is skewed;
    // with a dense 2^20-float pitch the round-robin order was the faster one by 3 %).
    // Where a wave has no more than one group (short stores) it takes single ones, not pairs.  Ranges are
    // whole pairs and no more: rounded to a pair for every wave they left up to half of the workgroups
    // without any.  Whole gathers, before and after: 4000 x 512 26.7 -> 18.8 us, 8000 x 2048 with 16
    // queries 57 -> 32 us, 30000 x 2048 58 -> 48 us, 70000 x 1024 58 -> 54 us, 131072 x 1024 unchanged; against that,
    // 100000 x 512 with 16 queries 63.7 -> 64.9 us.
    constexpr int NWAVES = kSimThreads / 64;
    const long share = (ngroups_all + gridDim.x - 1) / gridDim.x;
    const bool single = share <= NWAVES;
    const long per_wg = single ? share : (share + 1) / 2 * 2;
    const long ngroups = min(ngroups_all, (long)(blockIdx.x + 1) * per_wg);
    // a wave takes pairs of adjacent groups (32 rows): g, g+1, then 16 groups further on
    auto next_grp = [single](long g) -> long {
        return single ? g + NWAVES : (g & 1) ? g + 2 * NWAVES - 1 : g + 1;
    };
    const int nks = D / 32;                               // k-steps per row
    const int nchunks = (nks + kChunk - 1) / kChunk;
    const u16 *E = (const u16 *)p.emb;
    const u16 *qsrc = qs + ln * QROW + 8 * lg;

    long grp = (long)blockIdx.x * per_wg + (single ? wave : 2 * wave);
    auto row_ptr = [&](long g) -> const u16 * {
        long row = g * 16 + ln;
        row = row < p.N ? row : p.N - 1;
        return E + (size_t)row * D + 8 * lg;
    };
    // The wave's stream is (group, k-chunk) in row-major order over its groups grp, grp + stride,
    // ...; a load cursor runs two chunks ahead of the compute cursor, so two chunks beyond the
    // current one are always in flight.  Both cursors advance by increments only.
    v4u cur[kChunk], nx1[kChunk], nx2[kChunk];
    long l_grp = grp;                  // load cursor
    int l_ch = 0;
    // Past the wave's last group the cursor stays on one line of the store, so that the unconditional loads
    // there cost no traffic.
    const u16 *const idle = E + 8 * lg;
    const u16 *l_base = row_ptr(grp);
    auto load_next = [&](v4u (&dst)[kChunk]) {
        if (FULL) {
#pragma unroll
            for (int i = 0; i < kChunk; ++i) dst[i] = *(const v4u *)(l_base + (l_ch * kChunk + i) * 32);
            if (l_grp < ngroups && ++l_ch == nchunks) {
                const long g = next_grp(l_grp);
                l_grp = g;
                l_ch = 0;
                l_base = g < ngroups ? row_ptr(g) : idle;
            }
            return;
        }
        if (l_grp >= ngroups) return;
#pragma unroll
        for (int i = 0; i < kChunk; ++i) {
            const int ks = l_ch * kChunk + i;
            dst[i] = ks < nks ? *(const v4u *)(l_base + ks * 32) : (v4u){0u, 0u, 0u, 0u};
        }
        if (++l_ch == nchunks) {
            l_ch = 0;
            l_grp = next_grp(l_grp);
            if (l_grp < ngroups) l_base = row_ptr(l_grp);
        }
    };
    // Stage the queries of this pass, zero-padded, and their norms: a wave takes every eighth query, NQ * U
    // loads in flight, and forms the norms from the registers on the way.  The first chunks of the store
    // are asked for behind the last of these loads (loads return in order), so they arrive meanwhile.
    {
        constexpr int NQ = (16 * NG + NWAVES - 1) / NWAVES, U = NG == 1 ? 4 : 2;
        const u16 *Q = (const u16 *)p.qry + (size_t)p.q0 * D;
        const int pieces = D / 8;
        v4u v[NQ][U];
        float ss[NQ];
#pragma unroll
        for (int i = 0; i < NQ; ++i) ss[i] = 0.f;
        auto fetch = [&](int c0) {
#pragma unroll
            for (int i = 0; i < NQ; ++i) {
                const int r = wave + NWAVES * i;
#pragma unroll
                for (int u = 0; u < U; ++u) v[i][u] = (v4u){0u, 0u, 0u, 0u};
                if (r >= p.nq_grp) continue;
#pragma unroll
                for (int u = 0; u < U; ++u)
                    v[i][u] = *(const v4u *)(Q + (size_t)r * D + min(c0 + 64 * u + lane, pieces - 1) * 8);
            }
        };
        auto keep = [&](int c0) {
#pragma unroll
            for (int i = 0; i < NQ; ++i)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int c8 = c0 + 64 * u + lane;
                    if (c8 >= pieces || wave + NWAVES * i >= 16 * NG) continue;
                    *(v4u *)(qs + (wave + NWAVES * i) * QROW + c8 * 8) = v[i][u];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float lo = __uint_as_float(v[i][u][e] << 16), hi = __uint_as_float(v[i][u][e] & 0xffff0000u);
                        ss[i] = fmaf(hi, hi, fmaf(lo, lo, ss[i]));
                    }
                }
        };
        int c0 = 0;
        for (; c0 + 64 * U < pieces; c0 += 64 * U) {
            fetch(c0);
            keep(c0);
        }
        fetch(c0);
        if (grp < ngroups) {
            load_next(cur);
            load_next(nx1);
            keep(c0);
        } else {                           // a wave without a group (short stores): no loads in the others' way
            keep(c0);
        }
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const float t = wave_sum(ss[i]);
            if (lane == 0 && wave + NWAVES * i < 16 * NG) qnorm[wave + NWAVES * i] = sqrtf(t);
        }
    }
    __syncthreads();
    float un[NG];
#pragma unroll
    for (int y = 0; y < NG; ++y) un[y] = qnorm[16 * y + ln];
    if (grp >= ngroups) return;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 dot[NG], gram = zero;
#pragma unroll
    for (int y = 0; y < NG; ++y) dot[y] = zero;
    constexpr int NOUT = MAX ? 1 : NG;                     // result quads of a group of rows
    f32x4 held[NOUT];
    int ch = 0;                        // compute cursor
    while (grp < ngroups) {
        load_next(nx2);
        // MFMAs of the current chunk: dot products with the queries, Gram matrix of the row tile
#pragma unroll
        for (int i = 0; i < kChunk; ++i) {
            const int ks = ch * kChunk + i;
            if (FULL || ks < nks) {
                const bf16x8 a = as_bf16x8(cur[i]);
#pragma unroll
                for (int y = 0; y < NG; ++y) {
                    const bf16x8 b = as_bf16x8(*(const v4u *)(qsrc + 16 * y * QROW + ks * 32));
                    dot[y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, dot[y], 0, 0, 0);
                }
                gram = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, a, gram, 0, 0, 0);
            }
        }
        if (ch + 1 == nchunks) {
            // |e_r|^2 sits on the Gram diagonal: element (r, r) is in lane with ln == r, lg == r/4,
            // accumulator element r%4.  Lane (ln, lg) needs rows 4*lg + e.
            const long row0 = grp * 16;
            const float diag = (ln >> 2) == lg ? gram[ln & 3] : 0.f;
            f32x4 out[NOUT];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int r = 4 * lg + e;                 // row inside the group
                const float en2 = __shfl(diag, r + 16 * (r >> 2));
                float best = NAN;                         // fmaxf passes over NaN: padding takes no part
#pragma unroll
                for (int y = 0; y < NG; ++y) {
                    float den = sqrtf(en2) * un[y];
                    den = den < p.eps ? p.eps : den;
                    const float x = dot[y][e] / den;
                    if constexpr (MAX) best = 16 * y + ln < p.nq_grp ? fmaxf(best, x) : best;
                    else out[y][e] = x;
                }
                if constexpr (MAX) {
#pragma unroll
                    for (int o = 1; o < 16; o <<= 1) best = fmaxf(best, __shfl_xor(best, o));
                    out[0][e] = best;
                }
            }
            // The results of an even group wait for its odd neighbour, so that the wave writes the
            // 128 contiguous bytes of each query row back to back (whole cache lines).
            auto store_group = [&](long r0, const f32x4 (&o)[NOUT]) {
#pragma unroll
                for (int y = 0; y < NOUT; ++y) {
                    if (MAX ? ln > 0 : 16 * y + ln >= p.nq_grp) continue;
                    float *dst = (MAX ? p.sim : p.sim + (size_t)(p.q0 + 16 * y + ln) * p.sim_ld) + r0 + 4 * lg;
                    f32x4 x = o[y];
                    if (MAX && p.q0 > 0) {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (r0 + 4 * lg + e < p.N) x[e] = fmaxf(dst[e], x[e]);
                    }
                    if (r0 + 16 <= p.N && ((p.sim_ld & 3) == 0) && ((((uintptr_t)p.sim) & 15) == 0)) {
                        // one 16-byte store per lane (r0 and 4*lg are multiples of 4); four 4-byte
                        // stores cost the kernel 15 % of its time
                        *(f32x4 *)dst = x;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (r0 + 4 * lg + e < p.N) dst[e] = x[e];
                    }
                }
            };
            if (!single && !(grp & 1) && grp + 1 < ngroups) {
#pragma unroll
                for (int y = 0; y < NOUT; ++y) held[y] = out[y];
            } else {
                if (!single && (grp & 1)) store_group(row0 - 16, held);
                store_group(row0, out);
            }
#pragma unroll
            for (int y = 0; y < NG; ++y) dot[y] = zero;
            gram = zero;
        }
#pragma unroll
        for (int i = 0; i < kChunk; ++i) { cur[i] = nx1[i]; nx1[i] = nx2[i]; }
        if (++ch == nchunks) { ch = 0; grp = next_grp(grp); }
    }
}

// fp32 stores on v_mfma_f32_16x16x4f32 (operands and sums fp32; A[m][k] lane l holds m = l%16, k = l/16; B[k][n]
// n = l%16, k = l/16; C as above).  A workgroup takes 16 rows, its four waves every fourth 16 dims of them each: in
// step (chunk, i) the contraction is over the dims 16 * chunk + 4 * (l/16) + i, so every load is 16 bytes.  The
// waves' sums meet in LDS.  With a wave per row and a reduction over its lanes for every query the shuffles
// were the bound.  Whole gathers: 16000 x 512, 16 queries 107 -> 41.7 us, 16000 x 256, four 40.7 -> 31.0 us, 16000 x
// 512, one 33.9 -> 25.4 us, 3000 x 128, 16 queries 30.3 -> 24.5 us.  Sixteen chains of sums per wave, so that none is
// longer than there: relative error against 64 bits at 16000 x 512 1.04e-7 in both, with four chains 1.30e-7.
__device__ __host__ __forceinline__ int sim_f32_pitch(int D) { return D + (((32 - 4 * D) & 255) >> 2); }   // 32 mod 256 bytes

template <bool MAX>
__global__ __launch_bounds__(256) void sim_f32_mfma(GatherParams p)
{
    extern __shared__ __attribute__((aligned(16))) float qf[];   // [16][pitch]
    __shared__ float part[2][4][16][17], norm2[2][4][16];
    __shared__ float qnorm[16];
    constexpr int U = 4, AC = 4;                                 // chunks in flight, chains per k-step
    const int D = p.D, QP = sim_f32_pitch(D), nch = D / 16;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ln = lane & 15, lg = lane >> 4;
    if (p.sel.pre_zeroed && p.q0 == 0)
        sel_clear(p.sel, (long)blockIdx.x * 256 + tid, (long)gridDim.x * 256);
    const float *Q = (const float *)p.qry + (size_t)p.q0 * D, *E = (const float *)p.emb;
    const long ngroups = (p.N + 15) / 16;

    f32x4 a[U];
    auto load = [&](long g, int c) {
        const float *row = E + (size_t)min(g * 16 + ln, p.N - 1) * D + 4 * lg;
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = *(const f32x4 *)(row + min(c + 4 * u, nch - 1) * 16);
    };
    long g = blockIdx.x;
    {
        f32x4 v[4];
        float ss[4] = {0.f, 0.f, 0.f, 0.f};
        bool first = true;
        for (int c0 = 0; c0 < D / 4; c0 += 64) {
            const int c = c0 + lane;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
                if (wave + 4 * i < p.nq_grp) v[i] = *(const f32x4 *)(Q + (size_t)(wave + 4 * i) * D + min(c, D / 4 - 1) * 4);
            }
            if (first) load(g, wave);                            // behind the first query loads: loads return in order
            first = false;
            if (c >= D / 4) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                *(f32x4 *)(qf + (wave + 4 * i) * QP + 4 * c) = v[i];
#pragma unroll
                for (int e = 0; e < 4; ++e) ss[i] = fmaf(v[i][e], v[i][e], ss[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float t = wave_sum(ss[i]);
            if (lane == 0) qnorm[wave + 4 * i] = sqrtf(t);
        }
    }
    __syncthreads();
    int buf = 0;
    for (; g < ngroups; g += gridDim.x, buf ^= 1) {
        f32x4 acc[AC][4], sq = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < AC; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[u][i] = (f32x4){0.f, 0.f, 0.f, 0.f};
        for (int c = wave; c < nch; c += 4 * U) {
            f32x4 x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = a[u];
            // the next chunks: of this group, or the first of the next one
            if (c + 4 * U < nch) load(g, c + 4 * U);
            else if (g + gridDim.x < ngroups) load(g + gridDim.x, wave);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (c + 4 * u >= nch) continue;
                const f32x4 b = *(const f32x4 *)(qf + ln * QP + (c + 4 * u) * 16 + 4 * lg);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    acc[u % AC][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][i], b[i], acc[u % AC][i], 0, 0, 0);
                    sq[i] = fmaf(x[u][i], x[u][i], sq[i]);
                }
            }
        }
#pragma unroll
        for (int step = 1; step < AC; step *= 2)
#pragma unroll
            for (int u = 0; u + step < AC; u += 2 * step)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[u][i] += acc[u + step][i];
        const f32x4 sum = (acc[0][0] + acc[0][1]) + (acc[0][2] + acc[0][3]);
        float ss = (sq[0] + sq[1]) + (sq[2] + sq[3]);
        ss += __shfl_xor(ss, 16);
        ss += __shfl_xor(ss, 32);
#pragma unroll
        for (int e = 0; e < 4; ++e) part[buf][wave][4 * lg + e][ln] = sum[e];
        if (lg == 0) norm2[buf][wave][ln] = ss;
        __syncthreads();                                         // two buffers: the next one is written a barrier later
        const int r = MAX ? tid >> 4 : tid & 15, c = MAX ? tid & 15 : tid >> 4;
        const float dot = (part[buf][0][r][c] + part[buf][1][r][c]) + (part[buf][2][r][c] + part[buf][3][r][c]);
        const float en2 = (norm2[buf][0][r] + norm2[buf][1][r]) + (norm2[buf][2][r] + norm2[buf][3][r]);
        float den = sqrtf(en2) * qnorm[c];
        den = den < p.eps ? p.eps : den;
        const float y = dot / den;
        const long row = g * 16 + r;
        if constexpr (MAX) {
            float best = c < p.nq_grp ? y : NAN;                 // fmaxf passes over NaN
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) best = fmaxf(best, __shfl_xor(best, o));
            if (c == 0 && row < p.N) p.sim[row] = p.q0 > 0 ? fmaxf(p.sim[row], best) : best;
        } else if (c < p.nq_grp && row < p.N) {
            p.sim[(size_t)(p.q0 + c) * p.sim_ld + row] = y;
        }
    }
}

// One wave per context row; up to 16 queries of the group in LDS as fp32.  MAX as above.
template <typename T, bool MAX>
__global__ __launch_bounds__(256) void sim_generic(GatherParams p)
{
    extern __shared__ __attribute__((aligned(16))) float qf[];   // [nq_grp][D]
    __shared__ float qnorm[16];
    const int D = p.D;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (p.sel.pre_zeroed && p.q0 == 0)
        sel_clear(p.sel, (long)blockIdx.x * 256 + tid, (long)gridDim.x * 256);
    auto ld = [](const T *ptr, size_t i) -> float {
        if constexpr (sizeof(T) == 2) return bf16_bits_to_f32(((const u16 *)ptr)[i]);
        else return ((const float *)ptr)[i];
    };
    const T *Q = (const T *)p.qry + (size_t)p.q0 * D;
    for (int idx = tid; idx < p.nq_grp * D; idx += 256) qf[idx] = ld(Q, idx);
    __syncthreads();
    for (int qi = wave; qi < p.nq_grp; qi += 4) {
        float s = 0.f;
        for (int c = lane; c < D; c += 64) s = fmaf(qf[qi * D + c], qf[qi * D + c], s);
        s = wave_sum(s);
        if (lane == 0) qnorm[qi] = sqrtf(s);
    }
    __syncthreads();
    const long stride = (long)gridDim.x * 4;
    for (long row = (long)blockIdx.x * 4 + wave; row < p.N; row += stride) {
        const T *e = (const T *)p.emb + (size_t)row * D;
        float dot[16], en2 = 0.f;
#pragma unroll
        for (int qi = 0; qi < 16; ++qi) dot[qi] = 0.f;
        for (int c = lane; c < D; c += 64) {
            const float x = ld(e, c);
            en2 = fmaf(x, x, en2);
#pragma unroll
            for (int qi = 0; qi < 16; ++qi)
                if (qi < p.nq_grp) dot[qi] = fmaf(x, qf[qi * D + c], dot[qi]);
        }
        en2 = wave_sum(en2);
        float best = NAN;
#pragma unroll
        for (int qi = 0; qi < 16; ++qi) {
            if (qi < p.nq_grp) {
                const float dsum = wave_sum(dot[qi]);
                float den = sqrtf(en2) * qnorm[qi];
                den = den < p.eps ? p.eps : den;
                if constexpr (MAX) best = fmaxf(best, dsum / den);
                else if (lane == 0) p.sim[(size_t)(p.q0 + qi) * p.sim_ld + row] = dsum / den;
            }
        }
        if (MAX && lane == 0) p.sim[row] = p.q0 > 0 ? fmaxf(p.sim[row], best) : best;
    }
}

// ------------------------------------------------------------------------------------------
// Union through a bitmap of N bits, in which the selection marks its winners and their
// neighbourhoods as it writes them.  union_word: a word with the forced first / last rows added.
__device__ __forceinline__ uint32_t low_bits(long n) { return n >= 32 ? 0xffffffffu : n <= 0 ? 0u : (1u << n) - 1u; }

__device__ __forceinline__ uint32_t union_bits(const GatherParams &p, long w, uint32_t marked)
{
    const long b0 = w << 5;
    const uint32_t forced = low_bits(p.n_head - b0) | ~low_bits(p.N - p.n_tail - b0);
    return marked | (forced & low_bits(p.N - b0));
}

__device__ __forceinline__ uint32_t union_word(const GatherParams &p, long w)
{
    return w < p.nwords ? union_bits(p, w, p.bitmap[w]) : 0u;
}

// One bitmap word per thread, kUnionWordsPerBlock = 256 words (8192 rows) per workgroup.
__global__ __launch_bounds__(256) void union_count_words(GatherParams p)
{
    __shared__ int red[4];
    const int tid = threadIdx.x;
    int c = __popc(union_word(p, (long)blockIdx.x * kUnionWordsPerBlock + tid));
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) c += __shfl_xor(c, o);
    if ((tid & 63) == 0) red[tid >> 6] = c;
    __syncthreads();
    if (tid == 0) p.word_cnt[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// The set bits of the workgroup's words are expanded into an LDS staging array in ascending
// order and copied out as one contiguous, coalesced block of indices.  COUNTED: union_count_words
// has left the counts of the workgroups before this one; otherwise it counts their words itself.
template <bool COUNTED>
__global__ __launch_bounds__(256) void union_emit(GatherParams p)
{
    __shared__ int32_t stage[kUnionWordsPerBlock * 32];
    __shared__ int tmp[4];
    __shared__ int sh_base;
    const int tid = threadIdx.x, blk = blockIdx.x;
    int before = 0;
    if (COUNTED)
        for (int b = tid; b < blk; b += 256) before += p.word_cnt[b];
    else
#pragma unroll 8
        for (int w = 4 * tid; w < blk * kUnionWordsPerBlock; w += 4 * 256) {
            const v4u m = *(const v4u *)(p.bitmap + w);
#pragma unroll
            for (int j = 0; j < 4; ++j) before += __popc(union_bits(p, w + j, m[j]));
        }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) before += __shfl_xor(before, o);
    if (tid == 0) sh_base = 0;
    __syncthreads();
    if ((tid & 63) == 0) atomicAdd(&sh_base, before);
    const long w = (long)blk * kUnionWordsPerBlock + tid;
    uint32_t m = union_word(p, w);
    int tot;
    int pos = block256_excl_scan(__popc(m), tmp, tot);          // synchronises: sh_base is complete after it
    const int32_t first = (int32_t)(w << 5);
    while (m) {
        stage[pos++] = first + (__ffs(m) - 1);
        m &= m - 1;
    }
    __syncthreads();
    const int base = sh_base;
    for (int i = tid; i < tot; i += 256) p.union_idx[base + i] = stage[i];
    if (blk == gridDim.x - 1 && tid == 0) *p.union_count = base + tot;
}

// ------------------------------------------------------------------------------------------
#define RF_CHECK_LAUNCH()                     \
    do {                                      \
        hipError_t e_ = hipGetLastError();    \
        if (e_ != hipSuccess) return e_;      \
    } while (0)

template <bool MAX, int NG>
static auto sim_kernel(bool full) -> void (*)(GatherParams)
{
    return full ? sim_bf16_mfma<true, NG, MAX> : sim_bf16_mfma<false, NG, MAX>;
}

template <bool MAX>
static hipError_t similarity_passes(GatherParams p, bool bf16, hipStream_t st)
{
    const int cus = device_compute_units() > 0 ? device_compute_units() : 256;
    const size_t lds = 160 * 1024, block = (size_t)16 * (p.D + ((32 - 2 * p.D) & 255) / 2) * sizeof(u16);
    const bool mfma = bf16 && p.D % 32 == 0 && (size_t)16 * (p.D + 128) * 2 <= 150 * 1024;
    // Little work: a wave per row is as fast or faster, similarity alone, that / matrix form, us.  One query crosses between 260
    // and 700 thousand products of rows and dims: 1024 x 256 4.4 / 5.1, 2048 x 256 4.9 / 5.2, 2734 x 256 5.3 / 5.2, 2048 x 64
    // 4.1 / 4.9, 4096 x 128 5.2 / 5.1, but 1367 x 512 5.8 / 6.0; four queries at 150 to 350 thousand: 512 x 64 4.6 / 4.8,
    // 1562 x 64 5.1 / 4.9, 512 x 256 5.9 / 5.1.
    const bool f32_mfma = !bf16 && p.D % 16 == 0 && (size_t)16 * sim_f32_pitch(p.D) * sizeof(float) <= 140 * 1024 &&
                          (double)p.N * p.nq * p.D > 524288.0;
    // blocks of 16 queries: as few passes over the store as the LDS allows, evenly filled
    const int blocks = (p.nq + 15) / 16;
    const int fit = mfma ? (int)min((size_t)4, (lds - 1024) / block) : 1;
    const int passes = (blocks + fit - 1) / fit, ng = (blocks + passes - 1) / passes;
    // One workgroup is resident per compute unit.  A second round evens out a long stream and costs a
    // second start (staging the queries): one round / two, 16 queries or fewer, rows x dim: 131072 x
    // 1024 67.0 / 68.7 us, 262144 x 2048 240 / 254 us; 500000 x 1024 210 / 207 us, 1048576 x 2048
    // 868 / 857 us (whole gather, the same store again and again).
    const long rounds = (p.N + 15) / 16 >= 96l * cus ? 2 : 1;
    for (int q0 = 0; q0 < p.nq; q0 += 16 * ng) {
        p.q0 = q0;
        p.nq_grp = min(p.nq - q0, 16 * ng);
        void (*kern)(GatherParams);
        size_t smem;
        long grid;
        int threads;
        if (mfma) {
            smem = block * ng;
            threads = kSimThreads;
            grid = min((p.N + 15) / 16, cus * rounds);
            const bool full = p.D % (32 * kChunk) == 0;
            kern = ng == 1 ? sim_kernel<MAX, 1>(full) : ng == 2 ? sim_kernel<MAX, 2>(full)
                 : ng == 3 ? sim_kernel<MAX, 3>(full) : sim_kernel<MAX, 4>(full);
        } else if (f32_mfma) {
            smem = (size_t)16 * sim_f32_pitch(p.D) * sizeof(float);
            threads = 256;
            // Each workgroup stages the queries and starts its stream anew, so two per compute unit, one where the LDS holds
            // no more.  Similarity alone with one / two / three per unit, us: 110000 x 256, four queries 44.7 / 27.6 /
            // 35.2; 45000 x 16, one 15.7 / 10.2 / 13.3; 20000 x 2048, one 37.4 / 41.7 / 47.4.  With eight one query over
            // 30000 x 64 took 15.9 us, a wave per row 12.8, with two 9.6.
            grid = min((p.N + 15) / 16, (long)cus * (smem <= 70 * 1024 ? 2 : 1));
            kern = sim_f32_mfma<MAX>;
        } else {
            smem = (size_t)p.nq_grp * p.D * sizeof(float);
            threads = 256;
            grid = min((p.N + 3) / 4, (long)cus * 16);
            kern = bf16 ? sim_generic<u16, MAX> : sim_generic<float, MAX>;
        }
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(threads), smem, st, p);
        RF_CHECK_LAUNCH();
    }
    return hipSuccess;
}

hipError_t gather_similarity(const GatherParams &p, bool bf16, hipStream_t st)
{
    return similarity_passes<false>(p, bf16, st);
}

// The largest similarity of every row over all queries, into p.sim[N].
hipError_t gather_similarity_max(const GatherParams &p, bool bf16, hipStream_t st)
{
    return similarity_passes<true>(p, bf16, st);
}

constexpr int kUnionSelfCount = 16;

hipError_t gather_select_union(GatherParams p, hipStream_t st)
{
    hipError_t es = select_topk(p.sel, st);
    if (es != hipSuccess) return es;
    if (p.union_idx) {
        // Counting the words before its own costs a workgroup more as they grow; up to 16 workgroups that is
        // less than the launch it saves.  Whole calls, counted by themselves / by a launch of their own: 131072
        // rows 71.0 / 72.5 us, 262144 rows 95.1 / 94.6 us, 500000 rows 86.7 / 84.7 us, 1048576 rows 867 / 858 us.
        const int ub = (p.nwords + kUnionWordsPerBlock - 1) / kUnionWordsPerBlock;
        if (ub > kUnionSelfCount) {
            hipLaunchKernelGGL(union_count_words, dim3(ub), dim3(256), 0, st, p);
            RF_CHECK_LAUNCH();
            hipLaunchKernelGGL(union_emit<true>, dim3(ub), dim3(256), 0, st, p);
        } else {
            hipLaunchKernelGGL(union_emit<false>, dim3(ub), dim3(256), 0, st, p);
        }
        RF_CHECK_LAUNCH();
    }
    return hipSuccess;
}

}  // namespace reform
