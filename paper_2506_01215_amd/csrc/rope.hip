// Position reassignment after compression (arXiv 2506.01215, Sec. 3.1: after compression the
// tokens of the compressed cache get consecutive position ids).  The cache stores rotary-embedded
// keys; the key now at slot r came from slot kept[r] and is rotated by delta = r - kept[r]
// positions (half-split pairing: element c with element c + rot/2, frequency theta^(-2c/rot);
// elements beyond `rot` are left alone).  Rows that did not move (a prefix) are skipped.
//
// A thread owns one 16-byte piece of the low half of a row and the matching piece of the high
// half.  The angle delta * theta^(-2c/rot) reaches tens of thousands of radians, so it is formed
// and reduced to a quarter turn in fp64; sine and cosine of the reduced angle are fp32.
//
// Bound: HBM, as long as the arithmetic per pair stays short.  A frequency per pair in fp64 (exp2)
// and the library's sincosf took more time than the stream, so a workgroup forms the rot/2
// frequencies once into LDS and the sine and cosine come from sin_cos_quarter: 8 heads x 32768
// rows x 128 bf16 37 -> 22 us (134 MB), 8 x 4096 rows 9.2 -> 6.2 us.
#include "common.h"

namespace reform {

constexpr int kRopeTable = 1024;     // frequencies of rotary dimensions up to 2048 are tabulated

// Quarter turns per position of the pair c.
__device__ __forceinline__ double rope_quarters(const RopeParams &p, int c)
{
    return exp2(p.neg2_log2_theta_over_rot * (double)c) * 0.63661977236758134;
}

// sin and cos of `turns4` quarter turns.  The fraction of a quarter turn, |x| <= 1/2, is exact in
// fp64 and rounded once; sin(pi/2 x) = x (pi/2 + x^2 ...) and cos(pi/2 x) = 1 + x^2 ... are
// polynomials interpolated at Chebyshev points of x^2 on [0, 1/4] (error 3e-9 and 4e-9), pi/2
// in two parts.  Over whole turns the error against 64 bits is 1.7e-8 in the root mean square (a
// fraction of a turn rounded to fp32, times 2 pi, into an exact sine: 6.0e-8), at most 7.4e-8.
//
// Rounding to whole quarter turns is an addition of 1.5 * 2^52, which leaves the whole number in the sum's low bits: at most
// 2^31 positions of at most one radian each (theta > 1) are far below the 2^51 up to which it is exact.
// (rint and a conversion to 64 bits for the quadrant are a fifth of a pair's instructions: 8 heads x 4096 rows x 128 bf16 6.2 -> 5.6 us, x
// 32768 rows 25.0 -> 24.0, 8 x 12000 rows of 64 7.6 -> 6.8.)
__device__ __forceinline__ void sin_cos_quarter(double turns4, float &sn, float &cs)
{
    constexpr double kRound = 6755399441055744.0;
    const double t = turns4 + kRound;
    const uint32_t quadrant = (uint32_t)__double2loint(t);
    const float x = (float)(turns4 - (t - kRound)), u = x * x;
    float a = fmaf(0.00015820629902386097f, u, -0.004681266254496438f);
    a = fmaf(a, u, 0.07969258272529528f);
    a = fmaf(a, u, -0.6459640961467789f);
    a = fmaf(a, u, -4.371139006309477e-08f);
    const float s = fmaf(x, 1.5707963705062866f, x * a);
    float b = fmaf(-2.490919492953205e-05f, u, 0.0009191963136408901f);
    b = fmaf(b, u, -0.020863475054467458f);
    b = fmaf(b, u, 0.25366950772246427f);
    b = fmaf(b, u, -1.2337005501352676f);
    const float c = fmaf(b, u, 1.0f);
    const bool odd = quadrant & 1;
    sn = __uint_as_float(__float_as_uint(odd ? c : s) ^ ((quadrant << 30) & 0x80000000u));
    cs = __uint_as_float(__float_as_uint(odd ? s : c) ^ (((quadrant + 1) << 30) & 0x80000000u));
}

template <bool BF16>
__global__ __launch_bounds__(256) void rope_rerotate(RopeParams p)
{
    __shared__ double table[kRopeTable];
    constexpr int E = BF16 ? 8 : 4;                      // elements per 16-byte piece
    const int tpr = p.rot / (2 * E);                     // threads per row
    const long gid = (long)blockIdx.x * 256 + threadIdx.x;
    // 32-bit division where it suffices: the 64-bit one is some hundred instructions
    const long row = gid < (1l << 31) ? (long)((unsigned)gid / (unsigned)tpr) : gid / tpr;
    const int piece = (int)(gid - row * tpr);
    const int g = blockIdx.y;
    // the loads are under way while the frequencies are formed
    const int delta = row < p.n_rows ? (int)row - p.kept[(size_t)g * p.kept_ld + row] : 0;
    char *base = (char *)p.k + ((size_t)g * p.cap + row) * p.row_bytes;
    v4u *plo = (v4u *)(base + piece * 16);
    v4u *phi = (v4u *)(base + (p.rot / 2) * (BF16 ? 2 : 4) + piece * 16);
    v4u lo = {0u, 0u, 0u, 0u}, hi = lo;
    if (delta != 0) {
        lo = *plo;
        hi = *phi;
    }
    const bool tabulated = p.rot <= 2 * kRopeTable;
    if (tabulated) {
        for (int c = threadIdx.x; c < p.rot / 2; c += 256) table[c] = rope_quarters(p, c);
        __syncthreads();
    }
    if (delta == 0) return;
    float x0[E], x1[E];
    if (BF16) {
        const uint32_t a[4] = {lo.x, lo.y, lo.z, lo.w}, b[4] = {hi.x, hi.y, hi.z, hi.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x0[2 * i] = __uint_as_float(a[i] << 16);
            x0[2 * i + 1] = __uint_as_float(a[i] & 0xffff0000u);
            x1[2 * i] = __uint_as_float(b[i] << 16);
            x1[2 * i + 1] = __uint_as_float(b[i] & 0xffff0000u);
        }
    } else {
        x0[0] = __uint_as_float(lo.x); x0[1] = __uint_as_float(lo.y);
        x0[2] = __uint_as_float(lo.z); x0[3] = __uint_as_float(lo.w);
        x1[0] = __uint_as_float(hi.x); x1[1] = __uint_as_float(hi.y);
        x1[2] = __uint_as_float(hi.z); x1[3] = __uint_as_float(hi.w);
    }
    float y0[E], y1[E];
#pragma unroll
    for (int i = 0; i < E; ++i) {
        const int c = piece * E + i;
        float sn, cs;
        sin_cos_quarter((double)delta * (tabulated ? table[c] : rope_quarters(p, c)), sn, cs);
        y0[i] = x0[i] * cs - x1[i] * sn;
        y1[i] = x1[i] * cs + x0[i] * sn;
    }
    v4u olo, ohi;
    if (BF16) {
        olo.x = pack_bf16x2(y0[0], y0[1]); olo.y = pack_bf16x2(y0[2], y0[3]);
        olo.z = pack_bf16x2(y0[4], y0[5]); olo.w = pack_bf16x2(y0[6], y0[7]);
        ohi.x = pack_bf16x2(y1[0], y1[1]); ohi.y = pack_bf16x2(y1[2], y1[3]);
        ohi.z = pack_bf16x2(y1[4], y1[5]); ohi.w = pack_bf16x2(y1[6], y1[7]);
    } else {
        olo.x = __float_as_uint(y0[0]); olo.y = __float_as_uint(y0[1]);
        olo.z = __float_as_uint(y0[2]); olo.w = __float_as_uint(y0[3]);
        ohi.x = __float_as_uint(y1[0]); ohi.y = __float_as_uint(y1[1]);
        ohi.z = __float_as_uint(y1[2]); ohi.w = __float_as_uint(y1[3]);
    }
    *plo = olo;
    *phi = ohi;
}

hipError_t rope_rerotate_launch(const RopeParams &p, bool bf16, hipStream_t st)
{
    if (p.n_rows == 0 || p.rot == 0) return hipSuccess;
    const int tpr = p.rot / (2 * (bf16 ? 8 : 4));
    const long threads = p.n_rows * tpr;
    const dim3 grid((unsigned)((threads + 255) / 256), (unsigned)p.Hkv);
    if (bf16) hipLaunchKernelGGL(rope_rerotate<true>, grid, dim3(256), 0, st, p);
    else hipLaunchKernelGGL(rope_rerotate<false>, grid, dim3(256), 0, st, p);
    return hipGetLastError();
}

}  // namespace reform
