// fp32 chunk attention + eviction score (Sec. 3.1 / Fig. 1 step 1 of arXiv 2506.01215).
//
// The fp32 configuration is the small verification workload: few rows, a few hundred keys, so what
// bounds it is latency, not arithmetic.  head_dim 32, 64 and 128 run on v_mfma_f32_16x16x4f32 (fp32
// operands and sums) with a row block's keys spread over the waves of a workgroup; any other
// head_dim takes the short formulation with one wave per attention row (two passes: row maximum,
// then probabilities and P.V) and one wave per key for the column sums.  Accurate expf/logf,
// fixed summation order, no atomics.
#include "common.h"

namespace reform {

constexpr int kMaxD32 = 256;

__device__ __forceinline__ float dot_row(const float *a_lds, const float *b_glb, int D)
{
    float s = 0.f;
    for (int c = 0; c < D; c += 4) {
        const float4 b = *(const float4 *)(b_glb + c);
        s = fmaf(a_lds[c + 0], b.x, s);
        s = fmaf(a_lds[c + 1], b.y, s);
        s = fmaf(a_lds[c + 2], b.z, s);
        s = fmaf(a_lds[c + 3], b.w, s);
    }
    return s;
}

// grid = Hq * Ct workgroups of one wave.
__global__ __launch_bounds__(64) void attn_fwd_f32(AttnParams p)
{
    __shared__ float qs[kMaxD32];
    __shared__ float ps[64];
    const int lane = threadIdx.x;
    const int h = blockIdx.x / p.Ct;
    const int i = blockIdx.x % p.Ct;
    const int g = h / p.G;
    const int D = p.D;
    const float *q = (const float *)p.q + (size_t)h * p.q_hs + (size_t)i * p.q_rs;
    const float *K = (const float *)p.k + (size_t)g * p.cap * D;
    const float *V = (const float *)p.v + (size_t)g * p.cap * D;
    for (int c = lane; c < D; c += 64) qs[c] = q[c];
    __syncthreads();
    const int nvis = p.M + i + 1;

    float m = -INFINITY;
    for (int j = lane; j < nvis; j += 64) m = fmaxf(m, p.scale * dot_row(qs, K + (size_t)j * D, D));
    m = wave_max(m);

    float l = 0.f;
    float o[kMaxD32 / 64] = {0.f, 0.f, 0.f, 0.f};
    for (int j0 = 0; j0 < nvis; j0 += 64) {
        const int j = j0 + lane;
        float pj = 0.f;
        if (j < nvis) pj = expf(p.scale * dot_row(qs, K + (size_t)j * D, D) - m);
        l += pj;
        __syncthreads();
        ps[lane] = pj;
        __syncthreads();
        const int cnt = min(64, nvis - j0);
        for (int jj = 0; jj < cnt; ++jj) {
            const float pw = ps[jj];
            const float *vr = V + (size_t)(j0 + jj) * D;
#pragma unroll
            for (int u = 0; u < kMaxD32 / 64; ++u) {
                const int c = lane + 64 * u;
                if (c < D) o[u] = fmaf(pw, vr[c], o[u]);
            }
        }
    }
    l = wave_sum(l);
    float *out = (float *)p.out + (size_t)h * p.o_hs + (size_t)i * p.o_rs;
#pragma unroll
    for (int u = 0; u < kMaxD32 / 64; ++u) {
        const int c = lane + 64 * u;
        if (c < D) out[c] = o[u] / l;
    }
    if (lane == 0) p.lse[(size_t)h * p.Ct + i] = m + logf(l);
}

// grid = Hkv * n workgroups of one wave: wave (g, j) sums p_ij over the observing rows of the G
// heads of the group.  Lane t takes items t, t+64, ... of the (head, row) list, so the order of
// additions depends only on (G, first row, Ct): identical keys in the cache give identical sums.
__global__ __launch_bounds__(64) void attn_score_f32(AttnParams p)
{
    __shared__ float ks[kMaxD32];
    const int lane = threadIdx.x;
    const int g = blockIdx.x / p.n;
    const int j = blockIdx.x % p.n;
    const int D = p.D;
    const float *kr = (const float *)p.k + ((size_t)g * p.cap + j) * D;
    for (int c = lane; c < D; c += 64) ks[c] = kr[c];
    __syncthreads();
    const int i_first = max(p.Ct - p.W, max(j - p.M, 0));
    const int rows = p.Ct - i_first;
    const int items = p.G * rows;
    float acc = 0.f;
    for (int it = lane; it < items; it += 64) {
        const int h = g * p.G + it / rows;
        const int i = i_first + it % rows;
        const float *q = (const float *)p.q + (size_t)h * p.q_hs + (size_t)i * p.q_rs;
        acc += expf(p.scale * dot_row(ks, q, D) - p.lse[(size_t)h * p.Ct + i]);
    }
    acc = wave_sum(acc);
    if (lane == 0) {
        float *dst = p.score + (size_t)g * p.cap + j;
        *dst = p.accumulate ? *dst + acc : acc;
    }
}

// ------------------------------------------------------------------------------------------
// Matrix-core forms.  v_mfma_f32_16x16x4f32: A[m][k] lane l holds m = l%16, k = l/16; B[k][n]: n = l%16,
// k = l/16; C[m][n]: n = l%16, m = 4*(l/16) + e.  As in the bf16 kernels the transposed tile
// S^T = K Q^T is formed, so a lane owns one query (ln) and the keys 4*lg + e of a 16-key block, and
// its probabilities are the B operands of O^T = V^T P^T as they stand (k-step e contracts the
// keys 4*lg + e).  Contraction and output order are free, so they are permuted to make every
// global load 16 bytes: k-step (j, i) of Q.K contracts the dims 16*j + 4*lg + i, and row m of
// output block db is dim D/16 * m + db.
template <int D>
__device__ __forceinline__ void f32_load_row(float (&dst)[D / 4], const float *row, int lg)
{
#pragma unroll
    for (int j = 0; j < D / 16; ++j) *(f32x4 *)&dst[4 * j] = *(const f32x4 *)(row + 16 * j + 4 * lg);
}

template <int D>
__device__ __forceinline__ f32x4 f32_logits(const float (&a)[D / 4], const float (&b)[D / 4])
{
    f32x4 s[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};    // two chains: an MFMA waits for its addend
#pragma unroll
    for (int i = 0; i < D / 4; ++i) s[i & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[i], s[i & 1], 0, 0, 0);
    return s[0] + s[1];
}

// Forward.  A workgroup owns 16 rows of one head; its NW waves take the 16-key blocks in turn, each
// with a running maximum of its own, and meet in LDS once at the end.  With one wave per row the
// keys of a row were a chain of dependent steps: 4 heads, 128 rows over 384 keys, head_dim 64
// 81 -> 11 us, and with the waves' factors formed once per row at the end, not per output element, 10 us.  Batches of
// two or three blocks that share the maximum and overlap their MFMA chains give nothing: the fp32 matrix pipe of a
// compute unit is what a row block waits for (2048 of the 2900 clocks of a step).
constexpr int kF32FwdWaves = 8;

// SPLIT: the fp32 matrix pipe of a compute unit is what a row block waits for, so few row blocks share their key blocks
// over p.shares workgroups each, whose sums go to the workspace: [share][head, row block, row].  They are merged by the
// launch that forms the score where there is one (attn_merge_score_f32), else by one of its own.  Attention and score:
// 128 rows over 384 keys, 4 heads of 64 13.4 -> 11.2 us, 16 over 1040, 8/2 heads 20.6 -> 13.2 us, 40 over 940, 4 heads
// of 128 31.3 -> 19.1 us.
constexpr int kF32MaxShares = 4;
__device__ __forceinline__ size_t f32_slot(const AttnParams &p, int nrb, int h, int i) { return ((size_t)h * nrb + i / 16) * 16 + i % 16; }

template <int D, bool SPLIT>
__global__ __launch_bounds__(kF32FwdWaves * 64) void attn_fwd_f32_mfma(AttnParams p)
{
    constexpr int NW = kF32FwdWaves, DB = D / 16, PITCH = D + 4;
    __shared__ __attribute__((aligned(16))) float so[NW / 2][16][PITCH];
    __shared__ float sm[NW][16], sl[NW][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ln = lane & 15, lg = lane >> 4;
    const int nrb = (p.Ct + 15) / 16;
    const int share = SPLIT ? blockIdx.x % p.shares : 0, bid = SPLIT ? blockIdx.x / p.shares : blockIdx.x;
    const int h = bid % p.Hq, i0 = (nrb - 1 - bid / p.Hq) * 16;                 // late row blocks first
    const int b0 = share * NW + wave, step = SPLIT ? p.shares * NW : NW;        // the wave's key blocks
    const int g = h / p.G;
    const float *K = (const float *)p.k + (size_t)g * p.cap * D;
    const float *V = (const float *)p.v + (size_t)g * p.cap * D;
    const int lim = p.M + i0 + ln;                       // last key this lane's row sees
    const int nblk = (p.M + min(i0 + 16, p.Ct) - 1) / 16 + 1;

    float q[D / 4], k[D / 4], v[4][DB];
    auto load_v = [&](int b) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float *src = V + (size_t)min(b * 16 + 4 * lg + e, p.n - 1) * D + DB * ln;
            if constexpr (DB % 4 == 0) {
#pragma unroll
                for (int c = 0; c < DB; c += 4) *(f32x4 *)&v[e][c] = *(const f32x4 *)(src + c);
            } else {
                *(float2 *)&v[e][0] = *(const float2 *)src;
            }
        }
    };
    auto key_row = [&](int b) { return K + (size_t)min(b * 16 + ln, p.n - 1) * D; };
    f32_load_row<D>(q, (const float *)p.q + (size_t)h * p.q_hs + (size_t)min(i0 + ln, p.Ct - 1) * p.q_rs, lg);
    f32_load_row<D>(k, key_row(b0), lg);
    load_v(b0);

    f32x4 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = (f32x4){0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;
    for (int b = b0; b < nblk; b += step) {
        const int j0 = b * 16;
        f32x4 s = f32_logits<D>(k, q);
        f32_load_row<D>(k, key_row(b + step), lg);         // past the end: the last key again
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = j0 + 4 * lg + e > lim ? -INFINITY : p.scale * s[e];
        float mx = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m, mx);
        if (m_new != -INFINITY) {                        // else: the row sees no key of this wave yet
            const float alpha = expf(m - m_new);
            m = m_new;
            l *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db) o[db] *= alpha;
        }
        float pr[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            pr[e] = x[e] == -INFINITY ? 0.f : expf(x[e] - m);
            l += pr[e];
        }
        bool finite = true;
        if (j0 + 15 > p.M + i0) {                        // some row does not see some key of the block:
#pragma unroll
            for (int e = 0; e < 4; ++e)                  // 0 * inf must not reach its sum
#pragma unroll
                for (int c = 0; c < DB; ++c) finite = finite && __builtin_isfinite(v[e][c]);
        }
        if (__all(finite)) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int db = 0; db < DB; ++db)
                    o[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[e][db], pr[e], o[db], 0, 0, 0);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                for (int u = 0; u < 4; ++u) {
                    const float w = __shfl(pr[e], ln + 16 * u);
                    const int j = j0 + 4 * u + e;
                    if (j > lim || j >= p.n) continue;
#pragma unroll
                    for (int db = 0; db < DB; ++db)
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            o[db][c] = fmaf(w, V[(size_t)j * D + DB * (4 * lg + c) + db], o[db][c]);
                }
        }
        load_v(b + step);
    }
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (lg == 0) sm[wave][ln] = m;
    __syncthreads();
    float m_tot = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) m_tot = fmaxf(m_tot, sm[w][ln]);
    const float f = m == -INFINITY ? 0.f : expf(m - m_tot);
    if (lg == 0) sl[wave][ln] = l * f;                   // scaled once, not for every output element
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] *= f;
    // the upper half of the waves hands its sums to the lower half, and that to the output
    float *mine = &so[wave % (NW / 2)][ln][DB * 4 * lg];
    if (wave >= NW / 2) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int db = 0; db < DB; ++db) mine[DB * c + db] = o[db][c];
    }
    __syncthreads();
    if (wave < NW / 2) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int db = 0; db < DB; ++db) mine[DB * c + db] += o[db][c];
    }
    __syncthreads();
    for (int t = threadIdx.x; t < 16 * (D / 4); t += NW * 64) {
        const int r = t / (D / 4), c = t % (D / 4) * 4;
        if (i0 + r >= p.Ct) break;
        float lt = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) lt += sl[w][r];
        f32x4 x = *(const f32x4 *)&so[0][r][c];
#pragma unroll
        for (int w = 1; w < NW / 2; ++w) x += *(const f32x4 *)&so[w][r][c];
        if constexpr (SPLIT) {
            const size_t at = (size_t)share * p.part_rows + f32_slot(p, nrb, h, i0 + r);
            *(f32x4 *)(p.part_o + at * D + c) = x;
            if (c == 0) {
                float mt = -INFINITY;                        // stays where the row has no finite logit in this share
#pragma unroll
                for (int w = 0; w < NW; ++w) mt = fmaxf(mt, sm[w][r]);
                p.part_ml[at] = make_float2(mt, lt);
            }
            continue;
        }
        *(f32x4 *)((float *)p.out + (size_t)h * p.o_hs + (size_t)(i0 + r) * p.o_rs + c) = x / lt;
        if (c == 0) {
            float mt = -INFINITY;
#pragma unroll
            for (int w = 0; w < NW; ++w) mt = fmaxf(mt, sm[w][r]);
            p.lse[(size_t)h * p.Ct + i0 + r] = mt + logf(lt);
        }
    }
}

// Score.  A workgroup owns 16 keys of one KV head as the A operand; its waves take the (head, 16-row
// block) items of the observing rows in turn and add up their columns in wave order.  Row blocks
// are counted from the first observing row, so all cache keys see the same items in the same
// order (identical keys, identical scores).  4 heads, 128 rows over 384 keys 7.8 -> 4 us.
constexpr int kF32ScoreWaves = 8;

// Weight of a share whose maximum is m_share.  A share without a visible key counts 0 times its sums of 0; one
// whose visible keys all have NaN logits has that maximum too (fmaxf passes over NaN), and 0 times its NaN sums
// is NaN, as without shares.  So sums are always multiplied, never left out.
__device__ __forceinline__ float f32_weight(float m_share, float m) { return m_share == -INFINITY ? 0.f : expf(m_share - m); }

// Largest maximum and the sum relative to it of a row's shares; places behind the last share hold (-inf, 0).
__device__ __forceinline__ float2 f32_total(const float2 (&ml)[kF32MaxShares])
{
    float m = -INFINITY, l = 0.f;
#pragma unroll
    for (int s = 0; s < kF32MaxShares; ++s) m = fmaxf(m, ml[s].x);
#pragma unroll
    for (int s = 0; s < kF32MaxShares; ++s) l += ml[s].y * f32_weight(ml[s].x, m);
    return make_float2(m, l);
}

template <int D, bool PIECES>
__device__ __forceinline__ void f32_score_keys(const AttnParams &p, int bid)
{
    constexpr int NW = kF32ScoreWaves;
    __shared__ float part[NW][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ln = lane & 15, lg = lane >> 4;
    const int g = bid % p.Hkv, j0 = bid / p.Hkv * 16;
    float k[D / 4], q[D / 4];
    f32_load_row<D>(k, (const float *)p.k + ((size_t)g * p.cap + min(j0 + ln, p.n - 1)) * D, lg);
    const int i_first = max(p.Ct - p.W, max(j0 - p.M, 0));     // first row that observes and sees key j0
    const int nb = (p.Ct - i_first + 15) / 16;                 // row blocks per head (>= 1 since j0 < n)
    const int items = p.G * nb;
    const int nrb = (p.Ct + 15) / 16;
    float lse = 0.f;
    float2 ml[kF32MaxShares];
    auto load_q = [&](int it) {
        it = min(it, items - 1);
        const int h = g * p.G + it / nb, i = min(i_first + it % nb * 16 + ln, p.Ct - 1);
        f32_load_row<D>(q, (const float *)p.q + (size_t)h * p.q_hs + (size_t)i * p.q_rs, lg);
        if constexpr (PIECES) {
#pragma unroll
            for (int s = 0; s < kF32MaxShares; ++s)
                ml[s] = s < p.shares ? p.part_ml[(size_t)s * p.part_rows + f32_slot(p, nrb, h, i)] : make_float2(-INFINITY, 0.f);
        } else {
            lse = p.lse[(size_t)h * p.Ct + i];
        }
    };
    load_q(wave);
    f32x4 col = {0.f, 0.f, 0.f, 0.f};
    for (int it = wave; it < items; it += NW) {
        const int i = i_first + it % nb * 16 + ln, lim = i < p.Ct ? p.M + i : -1;
        const f32x4 s = f32_logits<D>(k, q);
        float ls = lse;
        if constexpr (PIECES) {
            const float2 t = f32_total(ml);
            ls = t.x + logf(t.y);
        }
        load_q(it + NW);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float pv = expf(p.scale * s[e] - ls);
            col[e] += j0 + 4 * lg + e > lim ? 0.f : pv;
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float x = col[e];
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) x += __shfl_xor(x, off);
        if (ln == 0) part[wave][4 * lg + e] = x;
    }
    __syncthreads();
    const int j = j0 + threadIdx.x;
    if (threadIdx.x >= 16 || j >= p.n) return;
    float x = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) x += part[w][threadIdx.x];
    float *dst = p.score + (size_t)g * p.cap + j;
    *dst = p.accumulate ? *dst + x : x;
}

template <int D>
__global__ __launch_bounds__(kF32ScoreWaves * 64) void attn_score_f32_mfma(AttnParams p)
{
    f32_score_keys<D, false>(p, blockIdx.x);
}

// Output and lse of one row block of a head from its shares.
template <int D>
__device__ __forceinline__ void f32_merge_rows(const AttnParams &p, int bid)
{
    const int nrb = (p.Ct + 15) / 16, h = bid % p.Hq, i0 = bid / p.Hq * 16;
    for (int t = threadIdx.x; t < 16 * (D / 4); t += kF32ScoreWaves * 64) {
        const int i = i0 + t / (D / 4), c = t % (D / 4) * 4;
        if (i >= p.Ct) break;
        float2 ml[kF32MaxShares];
        f32x4 o[kF32MaxShares];
#pragma unroll
        for (int s = 0; s < kF32MaxShares; ++s) {
            const size_t at = (size_t)min(s, p.shares - 1) * p.part_rows + f32_slot(p, nrb, h, i);
            ml[s] = p.part_ml[at];
            o[s] = *(const f32x4 *)(p.part_o + at * D + c);
            if (s >= p.shares) {
                ml[s] = make_float2(-INFINITY, 0.f);
                o[s] = (f32x4){0.f, 0.f, 0.f, 0.f};
            }
        }
        const float2 tot = f32_total(ml);
        f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < kF32MaxShares; ++s) x += o[s] * f32_weight(ml[s].x, tot.x);
        *(f32x4 *)((float *)p.out + (size_t)h * p.o_hs + (size_t)i * p.o_rs + c) = x / tot.y;
        if (c == 0) p.lse[(size_t)h * p.Ct + i] = tot.x + logf(tot.y);
    }
}

template <int D>
__global__ __launch_bounds__(kF32ScoreWaves * 64) void attn_merge_f32(AttnParams p)
{
    f32_merge_rows<D>(p, blockIdx.x);
}

// Both in one launch: the first n_score workgroups form the score, with the normalisers from the shares.
template <int D>
__global__ __launch_bounds__(kF32ScoreWaves * 64) void attn_merge_score_f32(AttnParams p, int n_score)
{
    if ((int)blockIdx.x < n_score) f32_score_keys<D, true>(p, blockIdx.x);
    else f32_merge_rows<D>(p, blockIdx.x - n_score);
}

// Shares of a problem (1: whole) with and without a score behind it.  The four matrix pipes of a compute unit divide a row
// block's key blocks, so up to twelve of them (192 keys) shares save nothing and cost the score's launch the sums of
// all shares: whole / two shares, attention and score, us: 4 heads of 128, 16 rows over 140 keys 13.0 / 14.9, over 180
// 13.8 / 14.8, over 200 15.5 / 14.8; 4 of 64, 60 rows 9.5 / 10.2, 10.0 / 10.3, 10.7 / 10.3; 8/2 of 32, 60 rows 9.0 / 9.6,
// 9.2 / 9.6, 9.8 / 9.5.  At head_dim 32 with more than 16 row blocks over the heads of a group up to twenty (8/2, 128 rows
// over 290 keys 11.9 / 12.3, over 330 12.6 / 12.4).
// A launch of its own for the merge takes 3 us, a step of eight waves over their key blocks 1.2 us at head_dim 64, the measure
// here, 0.9 at 32 and 2.2 at 128: whole / four shares without the score, 60 rows over 400 keys, 4 heads of 32 6.9 / 6.8, of
// 64 9.5 / 8.2, of 128 16.1 / 11.7; over 330 keys they stay whole.
static int f32_shares(const AttnParams &p, bool score)
{
    if (p.D != 32 && p.D != 64 && p.D != 128) return 1;
    const long groups = (long)p.Hq * ((p.Ct + 15) / 16), cus = device_compute_units() > 0 ? device_compute_units() : 256;
    const int blocks = (p.n - 1) / 16 + 1, steps = (blocks - 1) / kF32FwdWaves + 1;
    if (blocks <= (p.D == 32 && (long)p.G * ((p.W + 15) / 16) > 16 ? 20 : 12)) return 1;
    int shares = (int)(cus / groups < kF32MaxShares ? cus / groups : kF32MaxShares);
    if (shares > steps) shares = steps;
    if (shares < 2 || (!score && (steps - (steps + shares - 1) / shares) * 1.2 < 3.0)) return 1;
    return shares;
}

static size_t f32_rows(const AttnParams &p) { return (size_t)p.Hq * ((p.Ct + 15) / 16) * 16; }

size_t attend_f32_scratch_bytes(const AttnParams &p)
{
    const int shares = f32_shares(p, true);                  // with a score at least as many as without
    return shares > 1 ? (size_t)shares * f32_rows(p) * (p.D * sizeof(float) + sizeof(float2)) : 0;
}

// Attention, and with `score` the score: in two launches of the same kind each, split or not.
template <int D>
static hipError_t launch_f32(AttnParams p, void *part, size_t part_bytes, bool score, hipStream_t st)
{
    const unsigned groups = (unsigned)p.Hq * ((p.Ct + 15) / 16), n_score = (unsigned)p.Hkv * ((p.n + 15) / 16);
    const dim3 fwd(kF32FwdWaves * 64), sc(kF32ScoreWaves * 64);
    p.shares = f32_shares(p, score);
    const size_t rows = f32_rows(p);
    if (p.shares < 2 || !part || part_bytes < p.shares * rows * (D * sizeof(float) + sizeof(float2))) {
        hipLaunchKernelGGL((attn_fwd_f32_mfma<D, false>), dim3(groups), fwd, 0, st, p);
        if (score && hipPeekAtLastError() == hipSuccess)
            hipLaunchKernelGGL(attn_score_f32_mfma<D>, dim3(n_score), sc, 0, st, p);
        return hipGetLastError();
    }
    p.part_rows = (int)rows;
    p.part_o = (float *)part;
    p.part_ml = (float2 *)(p.part_o + p.shares * rows * D);
    hipLaunchKernelGGL((attn_fwd_f32_mfma<D, true>), dim3(groups * p.shares), fwd, 0, st, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (score) hipLaunchKernelGGL(attn_merge_score_f32<D>, dim3(n_score + groups), sc, 0, st, p, (int)n_score);
    else hipLaunchKernelGGL(attn_merge_f32<D>, dim3(groups), sc, 0, st, p);
    return hipGetLastError();
}

template <int D>
static hipError_t launch_score_f32(const AttnParams &p, hipStream_t st)
{
    const unsigned grid = (unsigned)p.Hkv * ((p.n + 15) / 16);
    hipLaunchKernelGGL(attn_score_f32_mfma<D>, dim3(grid), dim3(kF32ScoreWaves * 64), 0, st, p);
    return hipGetLastError();
}

hipError_t attend_f32_score(const AttnParams &p, hipStream_t st);

// Attention and, with `score`, the score of one call.  part: scratch for the shares' sums.
hipError_t attend_f32_forward(const AttnParams &p, void *part, size_t part_bytes, bool score, hipStream_t st)
{
    if (p.D == 32) return launch_f32<32>(p, part, part_bytes, score, st);
    if (p.D == 64) return launch_f32<64>(p, part, part_bytes, score, st);
    if (p.D == 128) return launch_f32<128>(p, part, part_bytes, score, st);
    hipLaunchKernelGGL(attn_fwd_f32, dim3((unsigned)p.Hq * p.Ct), dim3(64), 0, st, p);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess && score ? attend_f32_score(p, st) : e;
}

hipError_t attend_f32_score(const AttnParams &p, hipStream_t st)
{
    if (p.D == 32) return launch_score_f32<32>(p, st);
    if (p.D == 64) return launch_score_f32<64>(p, st);
    if (p.D == 128) return launch_score_f32<128>(p, st);
    hipLaunchKernelGGL(attn_score_f32, dim3((unsigned)p.Hkv * p.n), dim3(64), 0, st, p);
    return hipGetLastError();
}

}  // namespace reform
