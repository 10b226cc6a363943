// Exact top-k selection per row with lowest-index ties, ascending output: the shared back end of
// the cache eviction (heavy hitters of the attention score, Sec. 3.1 of arXiv 2506.01215) and of
// the gather stage (highest similarities, Sec. 3.3).
//
//   sel_zero      clears the digit histograms (and, for a caller, a few more ints in the same launch)
//   select_hist   x3: 11 + 11 + 10 bit radix passes over the monotone uint32 image of the values;
//                 LDS histogram per workgroup of 4096 candidates, merged with integer atomics.
//                 From the second pass on every workgroup first re-derives the digit picked by
//                 the previous pass from the global histogram (8 KB of L2 reads, saves a launch).
//   select_count  final pick, then per workgroup the number of candidates above / equal to the
//                 threshold key
//   select_write  ordered emission: everything above the threshold, then the lowest-index ties
//   select_compact, select_*_rest
//                 the second pass and those behind it for rows that may be compacted in place
//   select_row    all of the above in one launch, keys held in LDS: one workgroup per row, or several that
//                 wait for each other where every workgroup of the launch fits on the chip at once.  Cosines go by
//                 a pass of finer bins first, and a pooled gather's row is max-pooled while it is read
// Candidates in the first n_sink or last n_recent slots get the maximal key (always selected).
#include "common.h"

#include <atomic>

namespace reform {

constexpr int kSelBlock = 4096;      // candidates per selection workgroup (256 threads x 16)
constexpr int kRestWorkgroups = 1024; // the passes over what remains of compacted rows
// Up to so many blocks in all these take one at a time with all waves, beyond four.  One / four, us: 80 queries, 33000 x
// 128 77 / 93, 40 queries, 90000 x 128 73 / 82 (920 blocks); 16 queries, 600000 x 512 193 / 187 (2352), 2^20 x 512 296 / 287.
constexpr int kRestFewBlocks = 2048;
constexpr int kHistWorkgroups = 2048; // the histogram passes use about this many workgroups at most

__device__ __forceinline__ uint32_t sel_key(const SelParams &p, const float *row, long t)
{
    if (t < p.n_sink || t >= p.N - p.n_recent) return 0xffffffffu;
    return ordered_key(row[t]);
}

__device__ __forceinline__ uint32_t sel_key_of(const SelParams &p, float v, long t)
{
    if (t < p.n_sink || t >= p.N - p.n_recent) return 0xffffffffu;
    return ordered_key(v);
}

// True when the rows of `vals` can be read as aligned 16-byte quads (row pitch and base).
__device__ __forceinline__ bool sel_rows_aligned(const SelParams &p)
{
    return ((p.ld & 3) == 0) && ((((uintptr_t)p.vals) & 15) == 0);
}

__global__ void sel_zero(SelParams p)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < (long)p.nq * 3 * 2048) p.hist[i] = 0;
    if (i < p.zero_extra_n) p.zero_extra[i] = 0;
    if (p.multi_groups && i < (long)p.nq * p.nblk * 2) p.blk_cnt[i] = 0;
    if (p.gave_up && i == 0) *p.gave_up = 0;
}

__device__ __forceinline__ int digit_of(uint32_t u, int pass)
{
    return pass == 0 ? (int)(u >> 21) : pass == 1 ? (int)((u >> 10) & 2047u) : (int)(u & 1023u);
}
__device__ __forceinline__ bool prefix_match(uint32_t u, uint32_t prefix, int pass)
{
    return pass == 0 ? true : pass == 1 ? (u >> 21) == prefix : (u >> 10) == prefix;
}

// Executed by all 256 threads of a workgroup: from the histogram of pass `pass` pick the digit
// that holds the k-th largest key; returns the extended prefix and the k remaining inside it.
// Every workgroup of the following kernel repeats this (8 KB of L2 reads) instead of paying a
// separate launch; workgroup 0 of each query also records the result for the kernels after it.
__device__ __forceinline__ void select_pick(const SelParams &p, int q, int pass, uint32_t &prefix,
                                            int &krem, int *part, int *sel)
{
    const int tid = threadIdx.x;
    const int *gh = p.hist + ((size_t)q * 3 + pass) * 2048;
    const uint32_t prev = pass ? p.sel_prefix[(pass - 1) * p.nq + q] : 0u;
    const int k_in = pass ? p.sel_krem[(pass - 1) * p.nq + q] : p.k;
    // thread t owns digits 8t..8t+7; suffix count of everything above its range
    int loc[8], sum = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) { loc[i] = gh[8 * tid + i]; sum += loc[i]; }
    int total;
    const int below = block256_excl_scan(sum, part, total);   // digits of lower threads
    int acc = total - below - sum;                             // count with digit above this thread's range
#pragma unroll
    for (int i = 7; i >= 0; --i) {
        const int hi = acc;           // count with digit > 8*tid+i
        acc += loc[i];
        if (hi < k_in && k_in <= acc) { sel[0] = 8 * tid + i; sel[1] = k_in - hi; }
    }
    __syncthreads();
    const int bits = pass == 2 ? 10 : 11;
    prefix = (prev << bits) | (uint32_t)sel[0];
    krem = sel[1];
    __syncthreads();
}

// grid (<= nblk, nq): histogram of the current digit over the candidates matching the prefix.
__global__ __launch_bounds__(256) void select_hist(SelParams p, int pass)
{
    __shared__ int h[2048];
    __shared__ int part[256];
    __shared__ int sel[2];
    const int q = blockIdx.y, tid = threadIdx.x;
    for (int i = tid; i < 2048; i += 256) h[i] = 0;
    uint32_t prefix = 0u;
    int krem = p.k;
    if (pass) {
        select_pick(p, q, pass - 1, prefix, krem, part, sel);
        if (blockIdx.x == 0 && tid == 0) {
            p.sel_prefix[(pass - 1) * p.nq + q] = prefix;
            p.sel_krem[(pass - 1) * p.nq + q] = krem;
        }
    }
    __syncthreads();
    const float *s = p.vals + (size_t)q * p.ld;
    // a workgroup takes every gridDim.x-th block of 4096 candidates (long rows: fewer, longer
    // workgroups, so the pick above and the merge below are paid less often)
    for (int blk = blockIdx.x; blk < p.nblk; blk += gridDim.x) {
        const long t0 = (long)blk * kSelBlock;
        if (sel_rows_aligned(p) && t0 + kSelBlock <= p.N) {
            // full, aligned block: 16-byte loads, four candidates per lane and step
#pragma unroll
            for (int it = 0; it < kSelBlock / 1024; ++it) {
                const long t = t0 + (it * 256 + tid) * 4;
                const float4 v = *(const float4 *)(s + t);
                const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t u = sel_key_of(p, x[j], t + j);
                    if (prefix_match(u, prefix, pass)) atomicAdd(&h[digit_of(u, pass)], 1);
                }
            }
        } else {
            for (int i = tid; i < kSelBlock; i += 256) {
                const long t = t0 + i;
                if (t < p.N) {
                    const uint32_t u = sel_key(p, s, t);
                    if (prefix_match(u, prefix, pass)) atomicAdd(&h[digit_of(u, pass)], 1);
                }
            }
        }
    }
    __syncthreads();
    int *gh = p.hist + ((size_t)q * 3 + pass) * 2048;
    for (int i = tid; i < 2048; i += 256)
        if (h[i]) atomicAdd(&gh[i], h[i]);
}

// grid (nblk, nq): per block, how many candidates are above / equal to the threshold key.
__global__ __launch_bounds__(256) void select_count(SelParams p)
{
    __shared__ int red[2][4];
    __shared__ int part[256];
    __shared__ int sel[2];
    const int q = blockIdx.y, tid = threadIdx.x;
    uint32_t T;
    int need_eq;
    select_pick(p, q, 2, T, need_eq, part, sel);
    if (blockIdx.x == 0 && tid == 0) {
        p.sel_prefix[2 * p.nq + q] = T;
        p.sel_krem[2 * p.nq + q] = need_eq;
    }
    const float *s = p.vals + (size_t)q * p.ld;
    const long t0 = (long)blockIdx.x * kSelBlock;
    int gt = 0, eq = 0;
    if (sel_rows_aligned(p) && t0 + kSelBlock <= p.N) {
#pragma unroll
        for (int it = 0; it < kSelBlock / 1024; ++it) {
            const long t = t0 + (it * 256 + tid) * 4;
            const float4 v = *(const float4 *)(s + t);
            const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t u = sel_key_of(p, x[j], t + j);
                gt += u > T;
                eq += u == T;
            }
        }
    } else {
        for (int i = tid; i < kSelBlock; i += 256) {
            const long t = t0 + i;
            if (t < p.N) {
                const uint32_t u = sel_key(p, s, t);
                gt += u > T;
                eq += u == T;
            }
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) { gt += __shfl_xor(gt, o); eq += __shfl_xor(eq, o); }
    if ((tid & 63) == 0) { red[0][tid >> 6] = gt; red[1][tid >> 6] = eq; }
    __syncthreads();
    if (tid == 0) {
        int *c = p.blk_cnt + ((size_t)q * p.nblk + blockIdx.x) * 2;
        c[0] = red[0][0] + red[0][1] + red[0][2] + red[0][3];
        c[1] = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    }
}

// ------------------------------------------------------------------------------------------
// Building blocks shared by the ordered emission of the multi-launch path and by the
// single-launch selection.  A wave owns a contiguous range of nit * 256 candidates starting at
// w_lo; in step `it` lane l holds the four consecutive candidates w_lo + it * 256 + 4 * l + (0..3).
// Every global access of a step is then one contiguous block per wave, and positions in index
// order follow from wave ballots (no cross-lane data movement) plus the running counts of the wave.
//
// The keys lie in LDS and every step is a trip of a short loop, so the code has one size for all
// rows (10 KB; with the keys in registers and every step unrolled up to 59 KB).
__device__ __forceinline__ int lanes_below(unsigned long long m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Keys of the wave's range into LDS, in batches whose loads are in flight together; slots at or
// beyond N get 0 and are masked by the users.
__device__ __forceinline__ void load_keys(const SelParams &p, const float *s, int N, int w_lo, int nit, v4u *keys)
{
    const int lane = threadIdx.x & 63;
    const bool quads = sel_rows_aligned(p);
    const int tail = N - p.n_recent;
#pragma unroll 1
    for (int it0 = 0; it0 < nit; it0 += 4) {
        float v[4][4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            if (it0 + b >= nit) continue;
            const int t = min(w_lo + (it0 + b) * 256 + 4 * lane, (N - 1) & ~3);
            if (quads) {                                      // a quad that begins inside the row ends inside its pitch
                *(f32x4 *)v[b] = *(const f32x4 *)(s + t);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) v[b][j] = s[min(t + j, N - 1)];
            }
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            if (it0 + b >= nit) continue;
            const int t = w_lo + (it0 + b) * 256 + 4 * lane;
            v4u u;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                u[j] = t + j >= N ? 0u : t + j < p.n_sink || t + j >= tail ? 0xffffffffu : ordered_key(v[b][j]);
            keys[(it0 + b) * 64 + lane] = u;
        }
    }
}

// Candidates of the wave's range above / equal to the threshold key (wave-uniform results).
__device__ __forceinline__ void range_count(const v4u *keys, int N, int w_lo, int nit, uint32_t T, int &gt, int &eq)
{
    const int lane = threadIdx.x & 63;
    gt = 0;
    eq = 0;
#pragma unroll 1
    for (int it = 0; it < nit; ++it) {
        const v4u u = keys[it * 64 + lane];
        const int t = w_lo + it * 256 + 4 * lane;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            gt += __popcll(__ballot(t + j < N && u[j] > T));
            eq += __popcll(__ballot(t + j < N && u[j] == T));
        }
    }
}

__device__ __forceinline__ void mark_range(uint32_t *bitmap, long lo, long hi)   // inclusive
{
    for (long w = lo >> 5; w <= (hi >> 5); ++w) {
        const uint32_t from_lo = lo > (w << 5) ? ~0u << (lo & 31) : ~0u;
        const uint32_t to_hi = hi < (w << 5) + 31 ? ~(~1u << (hi & 31)) : ~0u;
        atomicOr(&bitmap[w], from_lo & to_hi);
    }
}

// Ordered emission of the wave's range: dest_run = selected candidates before the range,
// eq_run = candidates equal to T before it (both wave-uniform).  A first loop replaces the keys by
// the indices of the kept candidates, dense (a step's keys are read before its indices are written,
// and those end before the next step's keys).  A second one writes them out, coalesced, together
// with their values, companion entries and marks, several loads in flight: inside the first loop
// every step would wait for the stores of the one before (5.6 us of a row's 11.6 us at 4113
// candidates, now 2.9 us).
__device__ __forceinline__ void range_emit(const SelParams &p, int q, v4u *keys, int N, int w_lo, int nit,
                                           uint32_t T, int need_eq, int dest_run, int eq_run)
{
    const int lane = threadIdx.x & 63;
    int32_t *orank = p.out_rank ? p.out_rank + (size_t)q * p.ld : nullptr;
    const bool rank_quads = ((p.ld & 3) == 0) && ((((uintptr_t)p.out_rank) & 15) == 0);
    int *found = (int *)keys;
    int n_found = 0;
#pragma unroll 1
    for (int it = 0; it < nit; ++it) {
        const int t = w_lo + it * 256 + 4 * lane;
        const v4u u = keys[it * 64 + lane];
        bool keep[4];
        int eq_seen = eq_run;                                 // ties: lowest index first
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const unsigned long long me = __ballot(t + j < N && u[j] == T);
            eq_seen += lanes_below(me);
            eq_run += __popcll(me);
        }
        int at = n_found;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool is_eq = t + j < N && u[j] == T;
            keep[j] = t + j < N && (u[j] > T || (is_eq && eq_seen < need_eq));
            eq_seen += is_eq;
            const unsigned long long mk = __ballot(keep[j]);
            at += lanes_below(mk);
            n_found += __popcll(mk);
        }
        if (orank) {
            const int r0 = dest_run + at, r1 = r0 + keep[0], r2 = r1 + keep[1], r3 = r2 + keep[2];
            if (rank_quads && t + 4 <= N) {
                *(int4 *)(orank + t) = make_int4(r0, r1, r2, r3);
            } else {
                if (t < N) orank[t] = r0;
                if (t + 1 < N) orank[t + 1] = r1;
                if (t + 2 < N) orank[t + 2] = r2;
                if (t + 3 < N) orank[t + 3] = r3;
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (keep[j]) found[at++] = t + j;
    }
    // dest_run and k bound the output whatever the keys were
    const int n_out = min(n_found, max(p.k - dest_run, 0));
    if (p.union_count && w_lo == 0 && lane == 0) *p.union_count = p.k;
    const int32_t *sv = (const int32_t *)(p.vals + (size_t)q * p.ld);
    int32_t *oi = p.out_idx + (size_t)q * p.out_ld + dest_run;
    int32_t *os = p.out_val ? (int32_t *)(p.out_val + (size_t)q * p.out_ld) + dest_run : nullptr;
    const int32_t *ss = p.side_src ? p.side_src + (size_t)q * p.ld : nullptr;
    int32_t *sd = p.side_src ? p.side_dst + (size_t)q * p.out_ld + dest_run : nullptr;
    constexpr int B = 4;
#pragma unroll 1
    for (int i0 = lane; i0 < n_out; i0 += 64 * B) {
        int t[B], val[B], side[B];
#pragma unroll
        for (int b = 0; b < B; ++b) t[b] = found[min(i0 + 64 * b, n_out - 1)];
        if (os) {
#pragma unroll
            for (int b = 0; b < B; ++b) val[b] = sv[t[b]];
        }
        if (ss) {
#pragma unroll
            for (int b = 0; b < B; ++b) side[b] = ss[t[b]];
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int i = i0 + 64 * b;
            if (i >= n_out) continue;
            oi[i] = t[b];
            if (p.union_idx) p.union_idx[dest_run + i] = t[b];
            if (os) os[i] = val[b];
            if (ss) sd[i] = side[b];
        }
    }
    // Neighbourhoods overlap where winners are dense, and atomics on one word queue: each winner marks only
    // what the one before it in the wave has not (16 rows of 8849, 1106 winners of
    // radius 64 each: 131 -> 60 us for the call).
    if (p.mark)
        for (int i = lane; i < n_out; i += 64) {
            const long t = found[i], before = i > 0 ? found[i - 1] + p.mark_radius + 1 : 0;
            mark_range(p.mark, max(t - p.mark_radius, before), min(t + p.mark_radius, N - 1L));
        }
}

// grid (nblk, nq): ordered emission of the selected indices (ascending), lowest-index ties.
// A workgroup covers 4096 candidates, a wave 1024 of them.
__global__ __launch_bounds__(256) void select_write(SelParams p)
{
    __shared__ v4u keys[kSelBlock / 4];
    __shared__ int wtot[2][4];
    __shared__ int sh_gt, sh_eq;
    const int q = blockIdx.y, tid = threadIdx.x, blk = blockIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const uint32_t T = p.sel_prefix[2 * p.nq + q];
    const int need_eq = p.sel_krem[2 * p.nq + q];
    const int N = (int)p.N;
    const int w_lo = blk * kSelBlock + wave * 1024;
    v4u *mine = keys + wave * 256;
    load_keys(p, p.vals + (size_t)q * p.ld, N, w_lo, 4, mine);
    // candidates above / equal to T in the blocks before this one
    const int *c = p.blk_cnt + (size_t)q * p.nblk * 2;
    int gt_b = 0, eq_b = 0;
    for (int b = tid; b < blk; b += 256) { gt_b += c[2 * b]; eq_b += c[2 * b + 1]; }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) { gt_b += __shfl_xor(gt_b, o); eq_b += __shfl_xor(eq_b, o); }
    if (tid == 0) { sh_gt = 0; sh_eq = 0; }
    __syncthreads();
    if (lane == 0) { atomicAdd(&sh_gt, gt_b); atomicAdd(&sh_eq, eq_b); }
    int gt_w, eq_w;
    range_count(mine, N, w_lo, 4, T, gt_w, eq_w);
    if (lane == 0) { wtot[0][wave] = gt_w; wtot[1][wave] = eq_w; }
    __syncthreads();
    int base_gt = sh_gt, base_eq = sh_eq;                         // above / equal to T before this wave's range
#pragma unroll
    for (int w = 0; w < 4; ++w)
        if (w < wave) { base_gt += wtot[0][w]; base_eq += wtot[1][w]; }
    range_emit(p, q, mine, N, w_lo, 4, T, need_eq, base_gt + min(base_eq, need_eq), base_eq);
}

// ------------------------------------------------------------------------------------------
// Rows that are the call's own scratch and of which at most 1/16 is selected: the second pass leaves of each block
// of 4096 candidates only those with at least the first pass's digit (2 to 4 % where 1/64 is selected),
// ascending, at the block's own place: their values and behind them their places in the block (16 bits
// each).  A block of which more than a quarter remains stays as it is.  blk_cnt[0] of a block holds 1 + the number that
// remain, shifted by 16, or 0 there.  The passes that follow read a few percent of the row.  16 rows of
// 2^20 of which 1/64 is selected: passes of 18 + 20 + 17 + 15 + 28 us -> 18 + 21 + 5 + 5 + 10 us.
//
// How much remains depends on the values: where most similarities share the first digit (cosines around 0.56) no block
// is compacted, and the passes read whole blocks as fast as the plain ones do.  Whole gathers, us, plain passes /
// these, spread similarities and such ones:
//     16 queries, 600000 x 512, 1/64    229 / 187    274 / 260        23 queries, 150000 x 256, 1/37    69 / 58    78 / 73
//     16 queries, 2^20 x 512, 1/64      331 / 287    373 / 365        80 queries, 33000 x 128, 1/20     86 / 77    92 / 87
//     5 queries, 600000 x 512, 1/33     180 / 167    187 / 176        40 queries, 90000 x 128, 1/16     86 / 73    95 / 86
// (with one wave to a whole block and 4-byte loads the last column was 320, 413, 253, 137, 194, 179).  The worst form seen
// is similar rows in runs of 3000 of 2^20, whose marks queue on few words: 632 / 651 us, within what two
// runs of one side differ.  At 1/16 itself: 200000 x 512, 16 queries 93.9 / 80.4 us, 90000 x 512, 23 82.3 / 66.3,
// 40000 x 256, 64 84.1 / 71.6.  At 1/8 spread similarities still gain (103.4 / 90.6, 93.5 / 81.5, 116.7 / 105.9 us), those
// that share a digit were not measured there.
constexpr int kCompactShare = 16;

struct Remaining {
    const float *val;
    const u16 *at;           // null: the block is as it was
    int n;
    __device__ __forceinline__ Remaining(const SelParams &p, int q, int blk, int word)
    {
        const long t0 = (long)blk * kSelBlock;
        val = p.vals + (size_t)q * p.ld + t0;
        n = (word >> 16) - 1;
        at = n < 0 ? nullptr : (const u16 *)(val + n);
    }
};

// grid (<= nblk, nq): histogram of the second digit, as select_hist, and the compaction.
__global__ __launch_bounds__(256) void select_compact(SelParams p)
{
    __shared__ int h[2048];
    __shared__ int part[4];
    __shared__ int sel[2];
    __shared__ int wtot[4];
    const int q = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < 2048; i += 256) h[i] = 0;
    uint32_t prefix;
    int krem;
    select_pick(p, q, 0, prefix, krem, part, sel);
    if (blockIdx.x == 0 && tid == 0) {
        p.sel_prefix[q] = prefix;
        p.sel_krem[q] = krem;
    }
    float *row = const_cast<float *>(p.vals) + (size_t)q * p.ld;
    for (int blk = blockIdx.x; blk < p.nblk; blk += gridDim.x) {
        const long t0 = (long)blk * kSelBlock;
        const int have = (int)min((long)kSelBlock, p.N - t0), w_lo = wave * 1024;
        float v[4][4];
#pragma unroll
        for (int it = 0; it < 4; ++it)                   // a quad that begins inside the row ends inside its pitch
            *(f32x4 *)v[it] = *(const f32x4 *)(row + t0 + min(w_lo + it * 256 + 4 * lane, (have - 1) & ~3));
        unsigned kept = 0;                               // bit 4 * it + j
        int mine = 0;
#pragma unroll
        for (int it = 0; it < 4; ++it)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t u = ordered_key(v[it][j]);
                const bool in = w_lo + it * 256 + 4 * lane + j < have && (u >> 21) >= prefix;
                if (in && (u >> 21) == prefix) atomicAdd(&h[digit_of(u, 1)], 1);
                kept |= in ? 1u << (4 * it + j) : 0u;
                mine += __popcll(__ballot(in));
            }
        if (lane == 0) wtot[wave] = mine;
        __syncthreads();                                 // also: every value of the block has been read
        int base = 0, c = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            base += w < wave ? wtot[w] : 0;
            c += wtot[w];
        }
        const bool fits = 4 * c <= have;                 // values and places then fill 3/8 of the block
        if (fits) {
            u16 *at = (u16 *)(row + t0 + c);
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                int to = base;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const unsigned long long m = __ballot(kept >> (4 * it + j) & 1u);
                    to += lanes_below(m);
                    base += __popcll(m);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (kept >> (4 * it + j) & 1u) {
                        row[t0 + to] = v[it][j];
                        at[to++] = (u16)(w_lo + it * 256 + 4 * lane + j);
                    }
            }
        }
        if (tid == 0) p.blk_cnt[((size_t)q * p.nblk + blk) * 2] = fits ? (c + 1) << 16 : 0;
        __syncthreads();                                 // wtot is rewritten by the next block
    }
    int *gh = p.hist + ((size_t)q * 3 + 1) * 2048;
    for (int i = tid; i < 2048; i += 256)
        if (h[i]) atomicAdd(&gh[i], h[i]);
}

// The passes over what remains.  A workgroup takes PER blocks of candidates at a time, a grid apart (winners that lie
// together fill neighbouring blocks, which then go to different workgroups), 4 / PER waves to a block that was
// compacted, and with all its waves every block that was not.
constexpr int kRestBatch = 4;                            // loads of a lane in flight

// Values of block blk that was not compacted, four consecutive ones per step and lane; at or beyond `have`: not the row's.
__device__ __forceinline__ int whole_block(const SelParams &p, int q, int blk, f32x4 (&v)[4])
{
    const long t0 = (long)blk * kSelBlock;
    const float *row = p.vals + (size_t)q * p.ld + t0;
    const int have = (int)min((long)kSelBlock, p.N - t0);
#pragma unroll
    for (int it = 0; it < 4; ++it) v[it] = *(const f32x4 *)(row + min(it * 1024 + 4 * (int)threadIdx.x, (have - 1) & ~3));
    return have;
}

// The words of a workgroup's blocks blk0 + i * gridDim.x, asked for together: this wave's (0 behind the last block), and
// which of the blocks were not compacted.
template <int PER>
__device__ __forceinline__ int rest_words(const SelParams &p, const int *cnt, int blk0, int i_mine, unsigned &whole)
{
    int mine = 0;
    whole = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int blk = blk0 + i * gridDim.x;
        const int word = blk < p.nblk ? cnt[2 * blk] : 0;
        if (i == i_mine) mine = word;
        whole |= blk < p.nblk && !(word >> 16) ? 1u << i : 0u;
    }
    whole = __builtin_amdgcn_readfirstlane(whole);
    return mine;
}

// grid (workgroups, nq): histogram of the last digit of what remains.
template <int PER>
__global__ __launch_bounds__(256) void select_hist_rest(SelParams p)
{
    __shared__ int h[1024];
    __shared__ int part[4];
    __shared__ int sel[2];
    const int q = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int sharing = 4 / PER;
    for (int i = tid; i < 1024; i += 256) h[i] = 0;
    uint32_t prefix;
    int krem;
    select_pick(p, q, 1, prefix, krem, part, sel);
    if (blockIdx.x == 0 && tid == 0) {
        p.sel_prefix[p.nq + q] = prefix;
        p.sel_krem[p.nq + q] = krem;
    }
    auto add = [&](float v, bool in) {
        const uint32_t u = ordered_key(v);
        if (in && (u >> 10) == prefix) atomicAdd(&h[u & 1023u], 1);
    };
    const int *cnt = p.blk_cnt + (size_t)q * p.nblk * 2;
    for (int blk0 = blockIdx.x; blk0 < p.nblk; blk0 += gridDim.x * PER) {
        unsigned whole;
        const int word = rest_words<PER>(p, cnt, blk0, wave / sharing, whole);
        const Remaining r(p, q, blk0 + wave / sharing * gridDim.x, word);
        if (r.at)
            for (int i0 = wave % sharing * 64 + lane; i0 < r.n; i0 += 64 * sharing * kRestBatch) {
                float v[kRestBatch];
#pragma unroll
                for (int b = 0; b < kRestBatch; ++b) v[b] = r.val[min(i0 + 64 * sharing * b, r.n - 1)];
#pragma unroll
                for (int b = 0; b < kRestBatch; ++b) add(v[b], i0 + 64 * sharing * b < r.n);
            }
        for (; whole; whole &= whole - 1) {
            const int i = __builtin_ctz(whole);
            f32x4 v[4];
            const int have = whole_block(p, q, blk0 + i * gridDim.x, v);
#pragma unroll
            for (int it = 0; it < 4; ++it)
#pragma unroll
                for (int j = 0; j < 4; ++j) add(v[it][j], it * 1024 + 4 * tid + j < have);
        }
    }
    __syncthreads();
    int *gh = p.hist + ((size_t)q * 3 + 2) * 2048;
    for (int i = tid; i < 1024; i += 256)
        if (h[i]) atomicAdd(&gh[i], h[i]);
}

// The same grid: per block, how many are above (low 16 bits of blk_cnt[0]) / equal to (blk_cnt[1]) the threshold.
template <int PER>
__global__ __launch_bounds__(256) void select_count_rest(SelParams p)
{
    __shared__ int part[4];
    __shared__ int sel[2];
    __shared__ int sum[PER][2];
    const int q = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int sharing = 4 / PER;
    uint32_t T;
    int need_eq;
    select_pick(p, q, 2, T, need_eq, part, sel);
    if (blockIdx.x == 0 && tid == 0) {
        p.sel_prefix[2 * p.nq + q] = T;
        p.sel_krem[2 * p.nq + q] = need_eq;
    }
    int *cnt = p.blk_cnt + (size_t)q * p.nblk * 2;
    for (int blk0 = blockIdx.x; blk0 < p.nblk; blk0 += gridDim.x * PER) {
        if (tid < PER * 2) sum[tid >> 1][tid & 1] = 0;
        __syncthreads();
        int gt = 0, eq = 0;
        auto add = [&](float v, bool in) {
            const uint32_t u = ordered_key(v);
            gt += __popcll(__ballot(in && u > T));
            eq += __popcll(__ballot(in && u == T));
        };
        auto total = [&](int i) {
            if (lane == 0) { atomicAdd(&sum[i][0], gt); atomicAdd(&sum[i][1], eq); }
            gt = eq = 0;
        };
        unsigned whole;
        const int word = rest_words<PER>(p, cnt, blk0, wave / sharing, whole);
        const Remaining r(p, q, blk0 + wave / sharing * gridDim.x, word);
        if (r.at) {
            for (int i0 = wave % sharing * 64; i0 < r.n; i0 += 64 * sharing * kRestBatch) {
                float v[kRestBatch];
#pragma unroll
                for (int b = 0; b < kRestBatch; ++b) v[b] = r.val[min(i0 + 64 * sharing * b + lane, r.n - 1)];
#pragma unroll
                for (int b = 0; b < kRestBatch; ++b) add(v[b], i0 + 64 * sharing * b + lane < r.n);
            }
            total(wave / sharing);
        }
        for (; whole; whole &= whole - 1) {
            const int i = __builtin_ctz(whole);
            f32x4 v[4];
            const int have = whole_block(p, q, blk0 + i * gridDim.x, v);
#pragma unroll
            for (int it = 0; it < 4; ++it)
#pragma unroll
                for (int j = 0; j < 4; ++j) add(v[it][j], it * 1024 + 4 * tid + j < have);
            total(i);
        }
        __syncthreads();
        const int blk = blk0 + tid * gridDim.x;
        if (tid < PER && blk < p.nblk) {
            cnt[2 * blk] |= sum[tid][0];                 // at most 4096
            cnt[2 * blk + 1] = sum[tid][1];
        }
        __syncthreads();                                 // sum is cleared for the next blocks
    }
}

// grid (nblk / PER, nq): ordered emission, as range_emit.
template <int PER>
__global__ __launch_bounds__(256) void select_write_rest(SelParams p)
{
    __shared__ v4u keys[kSelBlock / 4];
    __shared__ int red[2][4], wtot[2][4];
    const int q = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t T = p.sel_prefix[2 * p.nq + q];
    const int need_eq = p.sel_krem[2 * p.nq + q];
    const int *cnt = p.blk_cnt + (size_t)q * p.nblk * 2;
    const int step = gridDim.x, first = blockIdx.x;      // blocks first + i * step
    constexpr int sharing = 4 / PER;
    const int blk = first + wave / sharing * step;
    unsigned whole;
    const int word = rest_words<PER>(p, cnt, first, wave / sharing, whole);
    const Remaining r(p, q, blk, word);                  // at most 1024: a quarter of them is one batch
    const int share = ((r.n + sharing - 1) / sharing + 63) & ~63;
    const int i_lo = wave % sharing * share, i_hi = min(i_lo + share, r.n);
    float vals[kRestBatch];
    int places[kRestBatch];
    auto fetch = [&](int i0) {
#pragma unroll
        for (int b = 0; b < kRestBatch; ++b) {
            const int i = max(min(i0 + 64 * b + lane, r.n - 1), 0);
            vals[b] = r.val[i];
            places[b] = r.at[i];
        }
    };
    if (r.at) fetch(i_lo);                               // on their way during the sums
    // candidates above / equal to T in the blocks before, a wave for those between two blocks of this workgroup
    // (PER = 1: for a quarter of those before it)
    const int lo = PER == 1 ? first * wave / 4 : wave ? first + (wave - 1) * step : 0;
    const int hi = PER == 1 ? first * (wave + 1) / 4 : min(first + wave * step, p.nblk);
    int gt = 0, eq = 0;
    for (int b = lo + lane; b < hi; b += 64) { gt += cnt[2 * b] & 0xffff; eq += cnt[2 * b + 1]; }
    gt = __builtin_amdgcn_readlane(wave_incl_scan(gt), 63);
    eq = __builtin_amdgcn_readlane(wave_incl_scan(eq), 63);
    if (lane == 0) { red[0][wave] = gt; red[1][wave] = eq; }
    __syncthreads();
    auto before_block = [&](int i) {                     // the i-th of this workgroup
        gt = eq = 0;
        for (int w = 0; w <= (PER == 1 ? 3 : i); ++w) { gt += red[0][w]; eq += red[1][w]; }
    };
    if (r.at) {
        before_block(wave / sharing);
        if (PER == 1) {                                  // and in the waves before: all four are here
            int gt_w = 0, eq_w = 0;
#pragma unroll
            for (int b = 0; b < kRestBatch; ++b) {
                const bool in = i_lo + 64 * b + lane < i_hi;
                const uint32_t u = ordered_key(vals[b]);
                gt_w += __popcll(__ballot(in && u > T));
                eq_w += __popcll(__ballot(in && u == T));
            }
            if (lane == 0) { wtot[0][wave] = gt_w; wtot[1][wave] = eq_w; }
            __syncthreads();
            for (int w = 0; w < wave; ++w) { gt += wtot[0][w]; eq += wtot[1][w]; }
        }
        int dest = gt + min(eq, need_eq);
        const long t0 = (long)blk * kSelBlock;
        int32_t *oi = p.out_idx + (size_t)q * p.out_ld;
        float *os = p.out_val ? p.out_val + (size_t)q * p.out_ld : nullptr;
        long before = 0;                                 // first place that the wave's winners so far have not marked
        for (int i0 = i_lo; i0 < i_hi; i0 += 64 * kRestBatch) {
            if (i0 > i_lo) fetch(i0);
#pragma unroll
            for (int b = 0; b < kRestBatch; ++b) {
                const bool in = i0 + 64 * b + lane < i_hi;
                const float v = vals[b];
                const int t = (int)t0 + places[b];
                const uint32_t u = ordered_key(v);
                const unsigned long long me = __ballot(in && u == T);
                const bool keep = in && (u > T || (u == T && eq + lanes_below(me) < need_eq));
                const unsigned long long mk = __ballot(keep);
                const int to = dest + lanes_below(mk);
                if (keep && to < p.k) {                  // always, whatever the keys were
                    oi[to] = t;
                    if (os) os[to] = v;
                }
                if (p.mark && mk) {                      // each winner marks what the one before it has not
                    const unsigned long long below = mk & ((1ull << lane) - 1ull);
                    const int prev = __shfl(t, below ? 63 - __clzll(below) : lane);
                    const long from = below ? prev + p.mark_radius + 1 : before;
                    if (keep) mark_range(p.mark, max(t - p.mark_radius, from), min(t + p.mark_radius, p.N - 1));
                    before = __builtin_amdgcn_readlane(t, 63 - __clzll(mk)) + p.mark_radius + 1;
                }
                dest += __popcll(mk);
                eq += __popcll(me);
            }
        }
    }
    for (; whole; whole &= whole - 1) {
        const int i = __builtin_ctz(whole), N = (int)p.N;
        const int w_lo = (first + i * step) * kSelBlock + wave * 1024;
        v4u *mine = keys + wave * 256;
        load_keys(p, p.vals + (size_t)q * p.ld, N, w_lo, 4, mine);
        int gt_w, eq_w;
        range_count(mine, N, w_lo, 4, T, gt_w, eq_w);
        __syncthreads();                                 // wtot may still be read for the block before
        if (lane == 0) { wtot[0][wave] = gt_w; wtot[1][wave] = eq_w; }
        __syncthreads();
        before_block(i);
        for (int w = 0; w < wave; ++w) { gt += wtot[0][w]; eq += wtot[1][w]; }
        range_emit(p, q, mine, N, w_lo, 4, T, need_eq, gt + min(eq, need_eq), eq);
    }
}

// ------------------------------------------------------------------------------------------
// The whole selection of a row in ONE launch, by `parts` workgroups of 1024 threads (16 waves, each
// owning nit * 256 candidates, nit <= 8).  The row is read once; its keys stay in LDS through the
// radix passes (LDS histogram, pick by a workgroup scan) and the ordered emission.  As soon as the
// bins or digits picked so far are shared by at most kSelList candidates (nearly always after one or two passes:
// the rest is ties) these go into a list, whose k-th largest list_pick finds.  Results are identical to
// the multi-launch path; the per-pass selection state is not written back.
//
// One workgroup per row (MULTI = false) serves short rows and many rows: its compute unit does all the
// work of a row, so a few long ones are faster with more of them.
//
// MULTI: several workgroups per row, when the whole grid can be resident at once.  Per radix pass
// a workgroup merges its LDS histogram into the row's
// global histogram (cleared by the launch before) with integer atomics and then polls that
// histogram until its total equals the number of candidates the pass must see -- all N in the
// first pass, afterwards the count of the bin picked by the pass before -- so the merged histogram
// is its own completion signal and no separate barrier is paid.  Every workgroup of a row takes
// the same pick from the same numbers.  The list is a global one of (key, index) words, polled for in
// the same way, and goes out together with the workgroups' counts of the candidates beyond it
// (published as count + 1 into cleared words, which the later workgroups of the row poll for); from
// both each workgroup derives where its share of the ascending output starts.  Without a list (more
// ties than fit) a third pass and the counts above / equal to the threshold take its place.
//
// Everything that crosses workgroups inside the launch goes through agent-scope atomics (adds,
// loads, stores), which are performed beyond the per-XCD L2s.  The host launches this kernel with at
// most kMultiMaxGroups workgroups, which fit the chip's 256 compute units together even where
// the keys leave room for one on each (nit = 8), so every workgroup that is waited for is running or will be
// dispatched as soon as unrelated work drains.  Several such launches on different streams may fill the
// chip with workgroups that wait for others which find no room; so may other programs.  The
// waits are therefore bounded, and a workgroup whose wait expires goes on alone: the row lies in memory
// as the launch before left it, so it selects from the whole row by itself (select_alone) and then
// emits its own part like the others.  A row that is pooled on the way in does not: the workgroups of this launch write it
// (p.vals) without an order between them, so there it is pooled anew from the similarities, which the launch before left
// (select_alone_pooled), and p.vals is not read.  The outcome is the same, only late.  It also sets *gave_up, on which
// the other waits of the call end as well: what they wait for will not come.
template <bool BINS> constexpr int kSelList = BINS ? 508 : 256;
// Entries of a list shared between workgroups that take their places one by one.  Atomics on one word queue, so of more each
// workgroup takes its places together, a round trip behind its own barrier (190 of 131072 similarities 63.7 -> 62.0 us for the call; but
// 20 of 15000 scores 50.2 -> 51.3).
constexpr int kSelDirect = 64;

// Where the size of the largest values is known (cosines), a pass of bins of 1/64 of an octave over the sixteen octaves up to
// `top` (sign and exponent of an ordered key) comes first; what lies below and above falls into the first and the last bin.
// Digits of a key's first eleven bits are a quarter of an octave, and a threshold's holds several percent of the row, so they need a
// second pass and, between workgroups, a second exchange of 3 us; one of these holds some hundreds of 10^5.  A
// threshold in the first or last bin (not positive, or sixteen octaves below) sends the row through the plain digits.  Whole
// calls, us: gather of 131072 x 1024 63.3 -> 62.0, of 20000 x 1024, 16 queries 34.8 -> 32.6, of 6000 x 256 14.3 -> 12.9; pooled and
// rows, 30000 x 512 30.2 -> 28.5.  Scores, whose size a sample of the row has to tell, gained nothing (8 heads, 32768
// of 65536 113.5 -> 114.3, 12000 of 15000 50.5 -> 49.8, 4096 of 4113 30.7 -> 31.4).
constexpr int kBinShift = 17, kBins = 1024;

__device__ __forceinline__ int bin_base(uint32_t top) { return (int)(top << 6 | 63u) - (kBins - 1); }

__device__ __forceinline__ int bin_of(uint32_t u, int base) { return min(max((int)(u >> kBinShift) - base, 0), kBins - 1); }

// Histogram of the bins over the wave's keys.
__device__ __forceinline__ void bin_hist(const v4u *keys, int N, int w_lo, int nit, int base, int *h)
{
    const int lane = threadIdx.x & 63;
    int low = 0;                                              // what falls into the first bin is counted without its atomics
#pragma unroll 1
    for (int it = 0; it < nit; ++it) {
        const v4u u = keys[it * 64 + lane];
        const int t = w_lo + it * 256 + 4 * lane;
        int d[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            d[j] = t + j < N ? bin_of(u[j], base) : -1;
            low += __popcll(__ballot(d[j] == 0));
        }
        if (d[0] > 0 && d[0] == d[1] && d[0] == d[2] && d[0] == d[3]) {
            const int first = __builtin_amdgcn_readfirstlane(d[0]);
            const unsigned long long like = __ballot(d[0] == first);
            if (d[0] != first) atomicAdd(&h[d[0]], 4);        // a plateau: pooled scores mostly are
            else if (lane == __builtin_ctzll(like)) atomicAdd(&h[first], 4 * __popcll(like));
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (d[j] > 0) atomicAdd(&h[d[j]], 1);
        }
    }
    if (lane == 0 && low) atomicAdd(&h[0], low);
}

// Histogram of the digit at `shift` over the wave's keys whose higher bits equal the prefix.
__device__ __forceinline__ void radix_hist(const v4u *keys, int N, int w_lo, int nit, int shift, int bits,
                                           uint32_t prefix, int *h)
{
    const int lane = threadIdx.x & 63;
#pragma unroll 1
    for (int it = 0; it < nit; ++it) {
        const v4u u = keys[it * 64 + lane];
        const int t = w_lo + it * 256 + 4 * lane;
        bool m[4];
        bool same = true;                                     // all four count and share one digit
        const uint32_t low = (1u << bits) - 1u, d0 = (u[0] >> shift) & low;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            m[j] = t + j < N && (u[j] >> shift) >> bits == prefix;
            same = same && m[j] && ((u[j] >> shift) & low) == d0;
        }
        // a wave whose 256 candidates all fall into one bin adds them at once (constant or
        // narrowly spread rows would otherwise serialise 64 lanes on one LDS address)
        const uint32_t dref = __builtin_amdgcn_readfirstlane(d0);
        if (__all(same && d0 == dref)) {
            if (lane == 0) atomicAdd(&h[dref], 256);
        } else if (same) {                                    // a plateau: pooled scores mostly are
            atomicAdd(&h[d0], 4);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (m[j]) atomicAdd(&h[(u[j] >> shift) & low], 1);
        }
    }
}

// Sum of 16 waves' totals, and of those before this wave, by every wave for itself.
__device__ __forceinline__ int waves_total(const int *wtot, int &before)
{
    const int wave = threadIdx.x >> 6, incl = row_incl_scan(wtot[threadIdx.x & 15]);
    const int upto = __builtin_amdgcn_readlane(incl, (wave + 15) & 15);
    before = __builtin_amdgcn_readfirstlane(wave) ? upto : 0;
    return __builtin_amdgcn_readlane(incl, 15);
}

// Where the time of a selection by digits goes (time stamps, 131072 similarities in 32 workgroups, 13.8 us; similarities have since
// gone by bins, see kBins, which leaves out the second histogram and its exchange):
// load 1.5, histogram 0.6, exchange 2.8, pick 0.5 (0.85 with shuffles in place of data-parallel primitives), second
// histogram 0.5 and exchange 2.5, pick 0.5, list 1.4, its pick 0.9, count 0.6, emission 1.6.  Whole calls: 37
// queries pooled over 262144 x 1024 162.4 -> 155.7 us (its plateaus queued on few histogram words), 2048
// rows fp32 13.5 -> 12.3 us, 65536 slots of 8 heads 115.6 -> 113.8 us.
//
// Executed by all 1024 threads: pick the digit of the histogram that holds the krem-th largest
// key (thread t owns digits 2t and 2t+1), extend the prefix by it and report how many candidates
// the digit holds.
__device__ __forceinline__ void bin_pick(int bits, uint32_t &prefix, int &krem, int &in_bin, const int *h, int *wtot,
                                         int *sel)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l0 = h[2 * tid], l1 = h[2 * tid + 1], sum = l0 + l1;
    const int incl = wave_incl_scan(sum);
    if (lane == 63) wtot[wave] = incl;
    __syncthreads();
    int below;
    const int total = waves_total(wtot, below);
    const int above = total - below - incl;                   // candidates with a digit above 2t+1
    if (above < krem && krem <= above + l1) { sel[0] = 2 * tid + 1; sel[1] = krem - above; sel[2] = l1; }
    else if (above + l1 < krem && krem <= above + sum) { sel[0] = 2 * tid; sel[1] = krem - above - l1; sel[2] = l0; }
    __syncthreads();
    prefix = (prefix << bits) | (uint32_t)sel[0];
    krem = sel[1];
    in_bin = sel[2];
    __syncthreads();
}

// All 1024 threads: the krem-th largest of the m <= kSelList<BINS> keys in `list` (padded with zeros), which agree from bit
// `shift` up.  A short list: four threads per key count how many are larger, 0.5 us at 20 keys and 2.3 us at 256.  A
// longer one: the first wave holds it all and settles a bit at a time by counting, 0.8 us for 10 bits and
// 1.3 us for 21 whatever the length.
constexpr int kCountedList = 96;

template <bool BINS>
__device__ __forceinline__ void list_pick(const v4u *list, int m, int krem, int shift, uint32_t &T, int &need_eq, int *sel)
{
    if (m <= kCountedList) {
        const int at = threadIdx.x >> 2;
        const uint32_t mine = ((const uint32_t *)list)[at];
        int gt = 0, eq = 0;
#pragma unroll 4
        for (int i = threadIdx.x & 3; i < (m + 3) / 4; i += 4) {
            const v4u x = list[i];
#pragma unroll
            for (int j = 0; j < 4; ++j) { gt += x[j] > mine; eq += x[j] == mine; }
        }
        gt += __builtin_amdgcn_update_dpp(0, gt, 0xb1, 0xf, 0xf, false);      // lanes 1 0 3 2 of each four
        gt += __builtin_amdgcn_update_dpp(0, gt, 0x4e, 0xf, 0xf, false);      // lanes 2 3 0 1
        eq += __builtin_amdgcn_update_dpp(0, eq, 0xb1, 0xf, 0xf, false);
        eq += __builtin_amdgcn_update_dpp(0, eq, 0x4e, 0xf, 0xf, false);
        if (at < m && gt < krem && krem <= gt + eq) { sel[0] = (int)mine; sel[1] = krem - gt; }   // equal keys write the same
    } else if (threadIdx.x < 64) {
        constexpr int X = BINS ? 8 : 4;
        uint32_t x[X];
#pragma unroll
        for (int j = 0; j < X; j += 4) {
            const int i = threadIdx.x + 16 * j;
            const v4u u = i < kSelList<BINS> / 4 ? list[i] : (v4u){0u, 0u, 0u, 0u};
#pragma unroll
            for (int c = 0; c < 4; ++c) x[j + c] = u[c];
        }
        uint32_t t = __builtin_amdgcn_readfirstlane(x[0]) >> shift << shift;  // the shared bits
        for (int b = shift - 1; b >= 0; --b) {
            const uint32_t up = t | 1u << b;
            int ge = 0;
#pragma unroll
            for (int j = 0; j < X; ++j)
                if (j < 4 || m > 256) ge += __popcll(__ballot(x[j] >= up));
            if (ge >= krem) t = up;
        }
        int gt = 0;
#pragma unroll
        for (int j = 0; j < X; ++j) gt += __popcll(__ballot(x[j] > t));
        if (threadIdx.x == 0) { sel[0] = (int)t; sel[1] = krem - gt; }
    }
    __syncthreads();
    T = (uint32_t)sel[0];
    need_eq = sel[1];
}

// Whether a wait of this call has to end: after spin_limit polls, or soon after another one has.
__device__ __forceinline__ bool multi_give_up(const SelParams &p, int spins)
{
    const bool over = spins >= p.spin_limit ||
        ((spins & 63) == 63 && __hip_atomic_load(p.gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0);
    if (over) atomicExch(p.gave_up, 1);
    return over;
}

// All 1024 threads: poll the row's histogram of a pass (thread t owns digits 2t, 2t+1) until it
// holds `expected` candidates, then leave that snapshot in h.  False (for all of them) if the wait
// had to end; a spin_limit of 0 ends every wait.
__device__ __forceinline__ bool multi_wait_hist(const SelParams &p, const int *gh, int ndigits, int expected, int *h,
                                                int *wtot, int *stop)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int v0 = 0, v1 = 0;
    for (int spins = 0;; ++spins) {
        if (2 * tid < ndigits) {
            v0 = __hip_atomic_load(&gh[2 * tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            v1 = __hip_atomic_load(&gh[2 * tid + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        const int incl = wave_incl_scan(v0 + v1);
        if (lane == 63) wtot[wave] = incl;
        __syncthreads();
        int below;
        const int total = waves_total(wtot, below);
        if (total == expected && p.spin_limit > 0) break;     // uniform: every thread saw the same total
        if (tid == 0) *stop = multi_give_up(p, spins);
        __syncthreads();                                      // also: wtot is rewritten by the next poll
        if (*stop) return false;
        __builtin_amdgcn_s_sleep(1);
    }
    h[2 * tid] = v0;
    h[2 * tid + 1] = v1;
    __syncthreads();
    return true;
}

// Wait for a word that another workgroup sets to a value other than 0; 0, and *stop set, if the wait had to end.
template <typename T>
__device__ __forceinline__ T multi_wait_word(const SelParams &p, const T *word, int *stop)
{
    for (int spins = 0;; ++spins) {
        const T v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (v != 0 && p.spin_limit > 0) return v;
        if (multi_give_up(p, spins)) {
            *stop = 1;
            return 0;
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

// Largest window in whole quads on one side, and one more for what it begins or ends in.
constexpr int kPoolHaloQuads = (kPoolMaxWindow - 1) / 8 + 1;

// What a selection that pools its row reads and, beside the selection, writes.
struct PoolSrc {
    const float *best;
    float *pooled;
    int window;
};

// LDS of the pooling of nit * 4096 tokens: their quads with the halo, and the quads' maxima twice.
__host__ __device__ constexpr size_t pool_lds_bytes(int nit) { return (size_t)(nit * 1024 + 2 * kPoolHaloQuads) * (16 + 2 * 4); }

// All 1024 threads: keys of the max-pooled tokens [lo, lo + nit * 4096), nit <= 2, quad by quad, from the similarities, and the
// pooled values in registers.  With h = 4 a + b tokens to each side (a > 0) the window of a token in quad t is the quads
// between t - a and t + a, whose maxima come from spans of a power of two (each the larger of two half as long), and up to two
// quads at either end in part.  Bound: the launch and its barriers, so it saves a launch (pool_window, tiles of 512 tokens that
// double over single ones) for four or five barriers.  Calls with their gather of rows, us: 30000 x 512, 5 queries
// 31.9 -> 29.7; 100000 x 1024, 16 74.9 -> 72.2; 8000 x 1024, 8 25.8 -> 24.9; 262144 x 1024, 37 156.1 -> 153.0 (154.1 with the
// pooled values stored at once, not behind the first histogram).
__device__ __forceinline__ void load_pooled(const PoolSrc &pool, const SelParams &p, int N, int lo, int nit, v4u *keys, f32x4 *quads,
                                            f32x4 (&pooled)[2])
{
    const int tid = threadIdx.x;
    const int h = (pool.window - 1) >> 1, a = h >> 2, b = h & 3, halo = a + 1;
    const int total = nit * 1024 + 2 * halo;             // quad i holds the tokens lo + 4 (i - halo) ..
    float *m = (float *)(quads + nit * 1024 + 2 * kPoolHaloQuads), *m2 = m + nit * 1024 + 2 * kPoolHaloQuads;
    __syncthreads();                                     // the last users of this LDS are through
    for (int i = tid; i < total; i += 1024) {
        const int t = lo + 4 * (i - halo);
        f32x4 x = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};          // outside the context: takes no part
        if (t >= 0 && t + 4 <= N) {
            x = *(const f32x4 *)(pool.best + t);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (t + j >= 0 && t + j < N) x[j] = pool.best[t + j];
        }
        quads[i] = x;
        m[i] = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
    }
    __syncthreads();
    int len = 1;
    for (; 2 * len <= 2 * a - 1; len *= 2) {             // m[i]: largest of the quads i .. i + len - 1
        for (int i = tid; i < total; i += 1024) m2[i] = i + len < total ? fmaxf(m[i], m[i + len]) : m[i];
        __syncthreads();
        float *other = m;
        m = m2;
        m2 = other;
    }
    const int tail = N - p.n_recent;
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        if (n >= nit) break;
        const int q = tid + n * 1024, i = q + halo, t = lo + 4 * q;
        f32x4 &y = pooled[n];
        if (a == 0) {
            const float *x = (const float *)(quads + i);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                y[j] = x[j];
                for (int d = 1; d <= h; ++d) y[j] = fmaxf(y[j], fmaxf(x[j - d], x[j + d]));
            }
        } else {
            const float core = fmaxf(m[i - a + 1], m[i + a - len]);
            const f32x4 l0 = quads[i - a - 1], l1 = quads[i - a], r0 = quads[i + a], r1 = quads[i + a + 1];
            // from the end: largest of the last 1 .. 7 tokens of l0 l1; from the start: of the first ones of r0 r1
            float left[8], right[8];
            left[0] = right[0] = core;
#pragma unroll
            for (int j = 1; j < 8; ++j) {
                left[j] = fmaxf(left[j - 1], j <= 4 ? l1[4 - j] : l0[8 - j]);
                right[j] = fmaxf(right[j - 1], j <= 4 ? r0[j - 1] : r1[j - 5]);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {                // 4 - j + b tokens of l0 l1, j + b + 1 of r0 r1
                float x = 0.f;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (b == c) x = fmaxf(left[4 - j + c], right[j + c + 1]);
                y[j] = x;
            }
        }
        v4u u;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            u[j] = t + j >= N ? 0u : t + j < p.n_sink || t + j >= tail ? 0xffffffffu : ordered_key(y[j]);
        keys[q] = u;
    }
    __syncthreads();
}

// The pooled values of load_pooled, out.
__device__ __forceinline__ void store_pooled(const PoolSrc &pool, int N, int lo, int nit, const f32x4 (&pooled)[2])
{
    const bool aligned = ((uintptr_t)pool.pooled & 15) == 0;
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const int t = lo + 4 * (int)(threadIdx.x + n * 1024);
        if (n >= nit) break;
        if (aligned && t + 4 <= N) {
            *(f32x4 *)(pool.pooled + t) = pooled[n];
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (t + j < N) pool.pooled[t + j] = pooled[n][j];
        }
    }
}

// select_alone for a row that is pooled on the way: by the workgroup's own number of tokens at a time, its own last.
__device__ __forceinline__ void select_alone_pooled(const PoolSrc &pool, const SelParams &p, int N, int lo, int nit, v4u *keys,
                                                    f32x4 *quads, int *h, int *wtot, int *sel, int *before, uint32_t &T, int &need_eq)
{
    const int tid = threadIdx.x, wave = tid >> 6, step = nit * 4096;
    const v4u *mine = keys + wave * (nit * 64);
    f32x4 unused[2];
    uint32_t prefix = 0u;
    int krem = p.k, in_bin;
#pragma unroll 1
    for (int pass = 0; pass < 3; ++pass) {
        const int bits = pass == 2 ? 10 : 11, shift = pass == 0 ? 21 : pass == 1 ? 10 : 0;
        __syncthreads();
        h[tid] = 0;
        h[tid + 1024] = 0;
#pragma unroll 1
        for (int at = 0; at < N; at += step) {
            load_pooled(pool, p, N, at, nit, keys, quads, unused);
            radix_hist(mine, N, at + wave * (nit * 256), nit, shift, bits, prefix, h);
        }
        __syncthreads();
        bin_pick(bits, prefix, krem, in_bin, h, wtot, sel);
    }
    T = prefix;
    need_eq = krem;
    if (tid < 2) before[tid] = 0;
#pragma unroll 1
    for (int at = 0; at <= lo; at += step) {             // up to its own, whose keys stay
        load_pooled(pool, p, N, at, nit, keys, quads, unused);
        if (at == lo) break;
        int gt, eq;
        range_count(mine, N, at + wave * (nit * 256), nit, T, gt, eq);
        if ((tid & 63) == 0) {
            atomicAdd(&before[0], gt);
            atomicAdd(&before[1], eq);
        }
    }
    __syncthreads();
}

// All 1024 threads, without the other workgroups: the threshold key of row s, how many candidates equal
// to it are selected, and how many above / equal to it lie before index `lo`.
__device__ __forceinline__ void select_alone(const SelParams &p, const float *s, int N, int lo, int *h, int *wtot,
                                             int *sel, int *before, uint32_t &T, int &need_eq)
{
    const int tid = threadIdx.x;
    uint32_t prefix = 0u;
    int krem = p.k, in_bin;
#pragma unroll 1
    for (int pass = 0; pass < 3; ++pass) {
        const int bits = pass == 2 ? 10 : 11, shift = pass == 0 ? 21 : pass == 1 ? 10 : 0;
        __syncthreads();
        h[tid] = 0;
        h[tid + 1024] = 0;
        __syncthreads();
#pragma unroll 1
        for (long t = tid; t < N; t += 1024) {
            const uint32_t u = sel_key(p, s, t);
            if ((u >> shift) >> bits == prefix) atomicAdd(&h[(u >> shift) & ((1u << bits) - 1u)], 1);
        }
        __syncthreads();
        bin_pick(bits, prefix, krem, in_bin, h, wtot, sel);
    }
    T = prefix;
    need_eq = krem;
    if (tid < 2) before[tid] = 0;
    __syncthreads();
    int gt = 0, eq = 0;
#pragma unroll 1
    for (int t = tid; t < lo; t += 1024) {
        const uint32_t u = sel_key(p, s, t);
        gt += u > T;
        eq += u == T;
    }
    if (gt) atomicAdd(&before[0], gt);
    if (eq) atomicAdd(&before[1], eq);
    __syncthreads();
}

// BINS: a pass of bins before the digits (see kBins).  POOL: the row is max-pooled on the way in.  These launches are so short that
// code counts which is fetched and skipped: with the bins in every form 12000 of 15000 scores 50.4 -> 51.3 us.  What is
// pooled are similarities, so a row with POOL always has bins, and its first exchange is theirs.
template <bool MULTI, bool BINS, bool POOL>
__global__ __launch_bounds__(1024) void select_row(SelParams p, int parts, int nit, PoolSrc pool)
{
    static_assert(BINS || !POOL, "pooled values are stored in the exchange of the bins");
    extern __shared__ v4u keys[];                                 // [nit * 1024], with POOL its LDS behind them
    f32x4 *quads = (f32x4 *)(keys + nit * 1024);
    __shared__ __attribute__((aligned(16))) int h[2048];
    constexpr int LIST = kSelList<BINS>;
    __shared__ v4u list[LIST / 4];
    __shared__ int wtot[2][16];
    __shared__ int sel[3], before[2], list_n, stop;
    const int q = blockIdx.x / parts, part = blockIdx.x % parts;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int N = (int)p.N;
    const int wg_lo = part * (nit * 4096), w_lo = wg_lo + wave * (nit * 256);
    v4u *mine = keys + wave * (nit * 64);
    h[tid] = 0;
    h[tid + 1024] = 0;
    if (tid < 3) sel[tid] = 0;
    if (tid < 2) before[tid] = 0;
    if (tid == 2) list_n = 0;
    if (tid == 3) stop = 0;
    if (tid < LIST / 4) list[tid] = (v4u){0u, 0u, 0u, 0u};
    __syncthreads();
    f32x4 pooled[2];
    if constexpr (POOL) load_pooled(pool, p, N, wg_lo, nit, keys, quads, pooled);
    else load_keys(p, p.vals + (size_t)q * p.ld, N, w_lo, nit, mine);
    if (!MULTI && !p.pre_zeroed)
        for (long i = (long)q * 1024 + tid; i < p.zero_extra_n; i += (long)gridDim.x * 1024) p.zero_extra[i] = 0;

    uint32_t prefix = 0u;
    int krem = p.k, in_bin = N, shift = kBinShift;
    bool alone = false;                                           // MULTI: this workgroup waits no more
    // Bins, then 11 and 6 bits; or, without bins or behind them, 11, 11 and 10.  Cleared words of the row (MULTI): 2048 for each of
    // three passes; the bins and the last digits behind them share the first.
    int *rh = p.hist + (size_t)q * 3 * 2048;
    // The workgroups' histograms together, in place of this one's.
    auto exchange = [&](int *gh, int digits, bool bins) {
        __syncthreads();
        if constexpr (MULTI) {
            for (int i = tid; i < digits; i += 1024)
                if (h[i]) atomicAdd(&gh[i], h[i]);
            if (POOL && bins) store_pooled(pool, N, wg_lo, nit, pooled);    // while the others' counts are on their way
            __syncthreads();
            alone = !multi_wait_hist(p, gh, digits, in_bin, h, wtot[0], &stop);
        } else if (POOL && bins) {
            store_pooled(pool, N, wg_lo, nit, pooled);
        }
    };
    bool binned = false;                                          // bins have settled the threshold's first bits
    if constexpr (BINS) {
        const int base = bin_base((uint32_t)p.bin_top);
        bin_hist(mine, N, w_lo, nit, base, h);
        exchange(rh, kBins, true);
        if (!alone) {
            uint32_t bin = 0u;
            int rest = krem, inside = N;
            bin_pick(10, bin, rest, inside, h, wtot[0], sel);
            if (bin > 0u && bin < (uint32_t)kBins - 1u) {
                binned = true;
                prefix = (uint32_t)base + bin;
                krem = rest;
                in_bin = inside;
            }
        }
    }
#pragma unroll 1
    for (int pass = 1; !alone && shift > 0 && (in_bin > LIST || (pass == 1 && !binned)); ++pass) {
        const int bits = binned ? (pass == 1 ? 11 : 6) : pass == 3 ? 10 : 11;
        shift = binned ? (pass == 1 ? 6 : 0) : pass == 1 ? 21 : pass == 2 ? 10 : 0;
        if (BINS || pass > 1) {
            h[tid] = 0;
            h[tid + 1024] = 0;
            __syncthreads();
        }
        radix_hist(mine, N, w_lo, nit, shift, bits, prefix, h);
        exchange(!BINS ? rh + (pass - 1) * 2048 : pass == 3 ? rh + 1024 : rh + pass * 2048, 1 << bits, false);
        if (!alone) bin_pick(bits, prefix, krem, in_bin, h, wtot[0], sel);
    }
    // here prefix holds the threshold's bits from `shift` up, shared by in_bin candidates
    uint32_t T = prefix;
    int need_eq = max(krem, 0);
    const bool listed = shift > 0 && !alone;
    int *c = p.blk_cnt + (size_t)q * parts * 2;                   // MULTI: cleared words, 0 = not published yet
    if (listed) {
        int *spare = !BINS || binned ? rh + 2 * 2048 : rh + 1024; // the last pass's histogram is still clear
        unsigned long long *glist = (unsigned long long *)spare;  // up to kSelList, and their number behind them
        int *gcount = spare + 1023;
        unsigned long long *own = (unsigned long long *)h;        // of many entries this workgroup's, see kSelDirect
        int gt = 0;
#pragma unroll 1
        for (int it = 0; it < nit; ++it) {
            const v4u u = mine[it * 64 + lane];
            const int t = w_lo + it * 256 + 4 * lane;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (MULTI) gt += __popcll(__ballot(t + j < N && u[j] >> shift > prefix));
                if (t + j < N && u[j] >> shift == prefix) {
                    const unsigned at = MULTI && (!BINS || in_bin <= kSelDirect) ? atomicAdd(gcount, 1) : atomicAdd(&list_n, 1);
                    if (at >= LIST) continue;
                    if (!MULTI) {
                        ((uint32_t *)list)[at] = u[j];
                        continue;
                    }
                    const unsigned long long e = (unsigned long long)u[j] << 32 | (unsigned)(t + j + 1);
                    if (!BINS || in_bin <= kSelDirect) __hip_atomic_store(&glist[at], e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    else own[at] = e;
                }
            }
        }
        int at = N;
        uint32_t key = 0u;
        if constexpr (MULTI) {
            if (lane == 0) wtot[0][wave] = gt;
            __syncthreads();
            if (tid == 0) {
                int tot = 0;
#pragma unroll
                for (int w = 0; w < 16; ++w) tot += wtot[0][w];
                __hip_atomic_store(&c[2 * part], tot + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (BINS && list_n) sel[2] = atomicAdd(gcount, list_n);
            }
            if (BINS && in_bin > kSelDirect) __syncthreads();
            if (BINS && tid < list_n && sel[2] + tid < LIST)              // always, whatever the keys were
                __hip_atomic_store(&glist[sel[2] + tid], own[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (tid < in_bin) {
                const unsigned long long e = multi_wait_word(p, &glist[tid], &stop);
                key = (uint32_t)(e >> 32);
                at = (int)(uint32_t)e - 1;
                ((uint32_t *)list)[tid] = key;
            } else if (tid >= 512 && tid - 512 < part) {          // part < 128
                atomicAdd(&before[0], max(multi_wait_word(p, &c[2 * (tid - 512)], &stop) - 1, 0));
            }
        }
        __syncthreads();
        alone = MULTI && stop;
        if (!alone) list_pick<BINS>(list, in_bin, krem, shift, T, need_eq, sel);
        if (MULTI && !alone && at < wg_lo) {
            if (key > T) atomicAdd(&before[0], 1);
            if (key == T) atomicAdd(&before[1], 1);
        }
    }
    int gt_w, eq_w;
    if (!alone) {
        range_count(mine, N, w_lo, nit, T, gt_w, eq_w);
        if (lane == 0) { wtot[0][wave] = gt_w; wtot[1][wave] = eq_w; }
        __syncthreads();
        if (MULTI && !listed) {
            if (tid < 2) {
                int tot = 0;
#pragma unroll
                for (int w = 0; w < 16; ++w) tot += wtot[tid][w];
                __hip_atomic_store(&c[2 * part + tid], tot + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            // candidates above / equal to T in the workgroups before this one (2 * parts <= 256 < 1024 threads)
            if (tid < 2 * part) atomicAdd(&before[tid & 1], max(multi_wait_word(p, &c[tid], &stop) - 1, 0));
            __syncthreads();
            alone = stop;
        }
    }
    if (MULTI && alone) {
        if constexpr (POOL) select_alone_pooled(pool, p, N, wg_lo, nit, keys, quads, h, wtot[0], sel, before, T, need_eq);
        else select_alone(p, p.vals + (size_t)q * p.ld, N, wg_lo, h, wtot[0], sel, before, T, need_eq);
        range_count(mine, N, w_lo, nit, T, gt_w, eq_w);
        if (lane == 0) { wtot[0][wave] = gt_w; wtot[1][wave] = eq_w; }
        __syncthreads();
    }
    int base_gt, base_eq;                                         // above / equal to T before this wave's range
    waves_total(wtot[0], base_gt);
    waves_total(wtot[1], base_eq);
    base_gt += before[0];
    base_eq += before[1];
    range_emit(p, q, mine, N, w_lo, nit, T, need_eq, base_gt + min(base_eq, need_eq), base_eq);
}

#define RF_CHECK_LAUNCH()                     \
    do {                                      \
        hipError_t e_ = hipGetLastError();    \
        if (e_ != hipSuccess) return e_;      \
    } while (0)

template <bool MULTI, bool BINS, bool POOL = false>
static hipError_t launch_select_row(const SelParams &p, long parts, int nit, hipStream_t st, const PoolSrc &pool = {})
{
    auto kern = select_row<MULTI, BINS, POOL>;
    const size_t lds = (size_t)nit * 4096 * 4 + (POOL ? pool_lds_bytes(nit) : 0);
    // the keys of nit = 8, and those of 2 with their pooling, need more than the default 64 KB of LDS: raised once per device, not
    // per launch
    static std::atomic<bool> lds_raised[64];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64 || !lds_raised[dev].load(std::memory_order_acquire)) {
        e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 8 * 4096 * 4);
        if (e != hipSuccess) return e;
        if (dev >= 0 && dev < 64) lds_raised[dev].store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(p.nq * parts)), dim3(1024), lds, st, p, (int)parts, nit, pool);
    return hipGetLastError();
}

// A compute unit takes about 1 us per 4096 candidates and step of the selection, three exchanges
// between workgroups about 6 us in all, and an eviction pays a launch that clears the histograms.
// One workgroup per row / several, whole calls: gather of one row of 6000 27.6 / 30.4 us, of 12000 32.4 /
// 29.2 us, of 30000 74.5 / 58.5 us, 16 rows of 30000 55.4 / 43.7 us; eviction, 8 rows of 4113 37.2 / 40.9
// us, of 32000 82.0 / 64.8 us.
constexpr int kFusedMaxN = 8192;
// Longer rows of up to kRowMaxN candidates (what the LDS holds) that are too many for that still take one
// workgroup each rather than five launches (five / one): gather of 65 rows of 8300 64 / 48 us, of 100 rows of
// 30000 100 / 94 us, of 1000 rows of 32768 440 / 386 us; eviction, 130 rows of 9192 233 / 214 us, 600 rows
// of 16384 938 / 909 us.
constexpr int kRowMaxN = 8 * 4096;

template <int PER>
static hipError_t select_rest(const SelParams &p, hipStream_t st)
{
    const dim3 grid((p.nblk + PER - 1) / PER, p.nq), few(min((int)grid.x, max(1, kRestWorkgroups / p.nq)), p.nq);
    hipLaunchKernelGGL(select_hist_rest<PER>, few, dim3(256), 0, st, p);
    RF_CHECK_LAUNCH();
    hipLaunchKernelGGL(select_count_rest<PER>, few, dim3(256), 0, st, p);
    RF_CHECK_LAUNCH();
    hipLaunchKernelGGL(select_write_rest<PER>, grid, dim3(256), 0, st, p);
    RF_CHECK_LAUNCH();
    return hipSuccess;
}

// Several workgroups per row when they can all be resident together: at most half of the
// compute units (a partitioned device has fewer than 256).  False: not for these rows.
static bool select_shared(const SelParams &p, int &nit, int &parts)
{
    if (p.N <= kFusedMaxN || !p.multi_groups || !p.gave_up) return false;
    const long max_groups = min((long)p.multi_groups, (long)device_compute_units() / 2);
    for (nit = 1; nit <= 8; nit *= 2) {
        const long w = (p.N + (long)nit * 4096 - 1) / ((long)nit * 4096);
        parts = (int)w;
        if ((long)p.nq * w <= max_groups) return true;
    }
    return false;
}

// Pools and selects in one launch where a workgroup of it takes at most 8192 tokens; true if it does.  More of them would be
// pooled one batch after the other, while pool_window has a workgroup for every 512.
bool select_pooled(const PoolParams &p, hipStream_t st, hipError_t &e)
{
    int nit = 1, parts = 1;
    const bool multi = select_shared(p.sel, nit, parts);
    if (!multi) nit = p.N <= 4096 ? 1 : 2;
    if (!p.sel.pre_zeroed || nit > 2 || (long)parts * nit * 4096 < p.N) return false;
    const PoolSrc pool = {p.best, p.pooled, p.window};
    e = multi ? launch_select_row<true, true, true>(p.sel, parts, nit, st, pool) : launch_select_row<false, true, true>(p.sel, 1, nit, st, pool);
    return true;
}

hipError_t select_topk(const SelParams &p, hipStream_t st)
{
    int nit = 0, parts = 1;
    const bool multi = select_shared(p, nit, parts);
    if (!multi && p.N <= kRowMaxN) {
        // this launch would clear the bitmap of a call that has not, while its other workgroups mark in it
        if (p.mark && !p.pre_zeroed) return hipErrorInvalidValue;
        for (nit = 1; nit * 4096 < p.N;) nit *= 2;
        return p.bin_top ? launch_select_row<false, true>(p, 1, nit, st) : launch_select_row<false, false>(p, 1, nit, st);
    }
    if (!p.pre_zeroed) {
        const long nz = max((long)p.nq * 3 * 2048, (long)p.zero_extra_n);
        hipLaunchKernelGGL(sel_zero, dim3((unsigned)((nz + 255) / 256)), dim3(256), 0, st, p);
        RF_CHECK_LAUNCH();
    }
    if (multi) return p.bin_top ? launch_select_row<true, true>(p, parts, nit, st) : launch_select_row<true, false>(p, parts, nit, st);
    const dim3 sgrid(p.nblk, p.nq);
    const int hblk = max(1, kHistWorkgroups / p.nq);       // workgroups per row of the histogram passes
    const dim3 hgrid(min(p.nblk, hblk), p.nq);
    if (p.own_vals && p.k <= p.N / kCompactShare && !p.n_sink && !p.n_recent && !p.out_rank && !p.side_src && !p.union_idx &&
        (p.ld & 3) == 0 && ((uintptr_t)p.vals & 15) == 0) {
        hipLaunchKernelGGL(select_hist, hgrid, dim3(256), 0, st, p, 0);
        RF_CHECK_LAUNCH();
        hipLaunchKernelGGL(select_compact, hgrid, dim3(256), 0, st, p);
        RF_CHECK_LAUNCH();
        return (long)p.nblk * p.nq <= kRestFewBlocks ? select_rest<1>(p, st) : select_rest<4>(p, st);
    }
    for (int pass = 0; pass < 3; ++pass) {
        hipLaunchKernelGGL(select_hist, hgrid, dim3(256), 0, st, p, pass);
        RF_CHECK_LAUNCH();
    }
    hipLaunchKernelGGL(select_count, sgrid, dim3(256), 0, st, p);
    RF_CHECK_LAUNCH();
    hipLaunchKernelGGL(select_write, sgrid, dim3(256), 0, st, p);
    RF_CHECK_LAUNCH();
    return hipSuccess;
}

}  // namespace reform
