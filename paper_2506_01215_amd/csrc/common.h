// Shared device helpers and launch-parameter structs of the gfx950 kernels.
// Nothing here is shared with the CPU oracle.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace reform {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16;
// 16-byte register quad as a native vector (HIP's uint4 is a struct whose copies lower to
// memcpy and can strand small arrays in scratch memory).
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));

constexpr int kWave = 64;

struct AttnParams {
    const void *q, *k, *v;
    void *out;
    float *lse;      // never null inside the kernels (caller's buffer or workspace)
    float *score;    // may be null for the forward kernel
    int Hq, Hkv, G, D;
    int M, Ct, cap, n;
    long q_hs, q_rs, o_hs, o_rs;
    float scale;
    int W;           // resolved observation window, 1..Ct
    int accumulate;
    int n_row_blocks;
    int by_head;     // how a row block's rows are dealt to the waves (see fwd_segment)
    // forward pass with the key range split over workgroups (see attn_fwd_bf16); shares == 0: whole
    int shares;      // workgroups per KV head, each an equal share of the list of the head's key tiles
    int start;       // places of that list left empty before each row block's tiles
    int tiles;       // length of the list: key tiles of one KV head and empty places (tiles * shares < 2^31)
    int part_rows;   // query rows (over the heads of a group and the chunk rows) of one partial result
    float *part_o;   // [workgroup][2][part_rows][D] unnormalised outputs
    float2 *part_ml; // [workgroup][2][part_rows] reference maximum (log2 units) and running sum
    // score pass with the observing rows cut into slices (see attn_score_bf16)
    int slices;                // number of slices (1: uncut), = slices of the tiles x head_slices
    int slice_tiles, head_slices, slice_heads;   // query tiles of 64 rows and heads of the group in each
    float *part_score;         // [slice][KV head][n] column sums of one slice, when there are several
    int in_short;              // host only: waves of attn_fwd_short where that forms the forward pass (see fwd_short)
    int narrow;                // host only: row blocks of 128 rows and workgroups of four waves, not 256 and eight (see fwd_choose)
};

constexpr int kMoveTileBytes = 32768;  // bytes of destination rows per workgroup of the in-place move
constexpr int kMoveRowBytes = 16384;    // rows whose size divides this move in place
constexpr int kMultiMaxGroups = 128;        // see select_row
constexpr int kUnionWordsPerBlock = 256;   // bitmap words per workgroup of the union kernels

// Top-k selection problem: nq rows of N candidates (row stride ld), k winners per row.
struct SelParams {
    const float *vals;
    long ld, N;
    int nq, k;
    int n_sink, n_recent;    // first / last slots that are always selected (count inside k)
    int bin_top;             // sign and exponent bits of the largest values as ordered keys, 0: not known (see kBins)
    int *hist;               // [nq][3][2048]
    uint32_t *sel_prefix;    // [3][nq]  selection state after each radix pass
    int *sel_krem;           // [3][nq]
    int *blk_cnt;            // [nq][nblk][2]   (above, equal) per workgroup
    int nblk;                // ceil(N / 4096)
    int32_t *out_idx;        // [nq][out_ld], ascending
    float *out_val;          // nullable, values of the selected candidates
    long out_ld;
    int32_t *out_rank;       // nullable [nq][ld]: rank[t] = number of selected candidates below t
    const int32_t *side_src; // nullable [nq][ld]: a 4-byte companion of every candidate ...
    int32_t *side_dst;       // ... copied to [nq][out_ld] for the selected ones (same order as out_idx)
    uint32_t *mark;          // nullable: bitmap over the candidates (shared by the rows; cleared by an earlier kernel of
    long mark_radius;        // ... the call, see pre_zeroed) in which every selected one and its neighbours up to this
                             // distance are marked
    int32_t *union_idx;      // nullable (one row): the winners a second time, and how many they are: the union of one
    int32_t *union_count;    // ... query's winners without neighbours
    int *zero_extra;         // nullable: zero_extra_n more ints cleared by the histogram-clearing launch
    int zero_extra_n;
    int own_vals;            // vals is scratch of the call: the rows may be compacted in place
    int pre_zeroed;          // hist and zero_extra were cleared by an earlier kernel of the same call
    int multi_groups;        // rows too long for one workgroup may be selected in one launch by several
                             // workgroups that wait for each other, at most this many in all (0: never;
                             // needs hist, blk_cnt and gave_up)
    int *gave_up;            // nullable: cleared with them, set to 1 if a wait between workgroups expired (the
                             // selection is exact all the same)
    int spin_limit;          // polls of such a wait (0: it expires at once)
};

struct EvictParams {
    void *k, *v;
    float *score;
    int32_t *pos;
    int32_t *kept;      // [Hkv][B]
    void *stage_k, *stage_v;   // [Hkv][B][row_bytes]
    float *stage_score;        // [Hkv][B]
    int32_t *stage_pos;        // [Hkv][B]
    SelParams sel;             // top-B over score
    int *sync;                 // in-place move: error word, per-stream tickets, per-tile flags; null = staged move
    int ntile;                 // tiles per stream of the in-place move
    int spin_limit;            // polls a tile spends on another tile's flag before giving up (0: see the kernel)
    int poll_delay;            // units of 1024 clocks before the first of them
    int Hkv, n, B, cap, n_sink, n_recent;
    int row_bytes;      // head_dim * sizeof(element), multiple of 16
};

struct RowsParams {
    const void *table;       // [n_table][row_bytes]
    void *out;               // [n_idx][row_bytes]
    const int32_t *idx;      // [n_idx]
    const int32_t *count;    // nullable device scalar: only the first min(*count, n_idx) indices are used
    int *err;                // nullable device word, bit 0 set if an index was outside the table
    long n_table, n_idx, row_bytes, pieces;
};

struct RopeParams {
    void *k;                 // [Hkv][cap][d], rows [0, n_rows) already compacted
    const int32_t *kept;     // [Hkv][kept_ld]: slot each row came from
    long n_rows, cap, kept_ld;
    int Hkv, rot;            // rot: rotated leading elements of a row (even)
    int row_bytes;
    double neg2_log2_theta_over_rot;   // -2 log2(theta) / rot
};

struct EmbedParams {
    const void *src;     // first token's head vector
    void *emb;           // embedding row of the first token
    long n_rows;
    long src_stride_bytes, emb_stride_bytes, col_bytes;
    long src_head_bytes, head_bytes;   // per head (blockIdx.y): source offset, column offset
    int n_heads;
    int pieces, group;   // 16-byte pieces per head vector; lanes per row (power of two >= pieces, <= 64)
    float eps;
};

constexpr int kCosineTop = 0x17f;           // SelParams::bin_top of values from 1 up to 2

constexpr int kPoolMaxWindow = 1025;        // odd; halo of 512 on each side

struct PoolParams {
    const float *best;   // [N] largest similarity over the query tokens
    float *pooled;       // [N]
    SelParams sel;       // budget selection over pooled (one row)
    long N;
    int window;          // odd, <= the kernel's maximum
};

struct GatherParams {
    const void *emb, *qry;
    float *sim;          // [nq][sim_ld]
    long sim_ld;         // row pitch of sim in floats (>= N)
    int32_t *topk_idx;   // [nq][k]
    float *topk_score;   // nullable
    int32_t *union_idx;  // nullable
    int32_t *union_count;
    SelParams sel;       // per-query top-k over sim
    uint32_t *bitmap;    // [nwords]
    int *word_cnt;       // [n_union_blocks]
    long N;
    int D, nq, k, radius, n_head, n_tail;
    int nwords;          // bitmap words
    float eps;
    int q0, nq_grp;      // first query and number of queries of this similarity launch
};

// Compute units of the current device (reform_api.hip; cached per device, 0 if it cannot be told).
int device_compute_units();

__device__ __forceinline__ float bf16_bits_to_f32(u16 b) { return __uint_as_float(((uint32_t)b) << 16); }

// fp32 -> bf16 bits, round to nearest even (finite inputs; NaN stays NaN).
__device__ __forceinline__ u16 f32_to_bf16_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u16)((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (u16)(u >> 16);
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    f32x2 v = {lo, hi};
    bf16x2 r = __builtin_convertvector(v, bf16x2);   // v_cvt_pk_bf16_f32 on gfx950 (RNE)
    return __builtin_bit_cast(uint32_t, r);
}

__device__ __forceinline__ bf16x8 as_bf16x8(v4u v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ float wave_sum(float x)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
    return x;
}
__device__ __forceinline__ float wave_max(float x)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
    return x;
}

// Inclusive sums over the 16 lanes of a row and over the wave, by data-parallel primitives: a shuffle goes through the
// LDS unit and takes about 100 clocks, one of these moves some eight.
__device__ __forceinline__ int row_incl_scan(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);      // from 1, 2, 4, 8 lanes below
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    return x;
}
__device__ __forceinline__ int wave_incl_scan(int x)
{
    x = row_incl_scan(x);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);      // lane 15 to row 1, lane 47 to row 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);      // lane 31 to rows 2 and 3
    return x;
}

// Monotone map float -> uint32: a > b  <=>  key(a) > key(b) (finite values; -0 and +0 map alike).
__device__ __forceinline__ uint32_t ordered_key(float f)
{
    uint32_t u = __float_as_uint(f);
    if (u == 0x80000000u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Clears the selection's histograms and extra ints; thread i0 of `stride` threads.  Called at the
// start of a kernel that runs before the selection in the same library call, which saves the
// selection its own clearing launch.
__device__ __forceinline__ void sel_clear(const SelParams &p, long i0, long stride)
{
    const long nh = (long)p.nq * 3 * 2048;
    for (long i = i0; i < nh; i += stride) p.hist[i] = 0;
    for (long i = i0; i < p.zero_extra_n; i += stride) p.zero_extra[i] = 0;
    if (p.multi_groups)
        for (long i = i0; i < (long)p.nq * p.nblk * 2; i += stride) p.blk_cnt[i] = 0;
    if (p.gave_up && i0 == 0) *p.gave_up = 0;
}

// Exclusive scan of one int per thread over a 256-thread workgroup (tmp: 4 ints of LDS);
// returns the exclusive prefix, `total` receives the workgroup sum.
__device__ __forceinline__ int block256_excl_scan(int x, int *tmp, int &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int incl = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
    }
    __syncthreads();
    if (lane == 63) tmp[wave] = incl;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const int t = tmp[w];
        if (w < wave) base += t;
        tot += t;
    }
    total = tot;
    return base + incl - x;
}

}  // namespace reform
