// dct_decode.h -- single-texel decoding of DCT-compressed textures (section
// "Results", texture compression: 8x8 blocks, six lowest-frequency DCT
// coefficients per channel in one 32-bit word, 7-bit DC and 5-bit AC).
//
// Word layout: bits 0..6 DC code d; then five 5-bit AC codes (bits 7..11,
// 12..16, 17..21, 22..26, 27..31) for the zigzag coefficients (v, u) =
// (0,1), (1,0), (2,0), (1,1), (0,2), each stored as q + 16 with q in
// -15..15.  Dequantised values: d * 8/127 and q * 2/15.  The texel at (x, y)
// of its block is the orthonormal inverse DCT of these six coefficients:
//   f = a0^2 d 8/127 + sum_k q_k (2/15) a(u_k) a(v_k) cos((2x+1) u_k pi/16) cos((2y+1) v_k pi/16)
// with a(0) = sqrt(1/8), a(k > 0) = 1/2.  So f = d/127 + K (q1 c1(x) +
// q2 c1(y) + q3 c2(y) + q5 c2(x)) + K11 q4 c1(x) c1(y), where c1(i) =
// cos((2i+1) pi/16), c2(i) = cos((2i+1) pi/8), K = (2/15)/(4 sqrt 2) and
// K11 = (2/15)/4.
//
// Device layout: blocks row-major, CAP words per block (channels padded with
// zero words to a multiple of 4, so a block's channels load as 16-byte
// vectors).
#pragma once

#include "device_common.h"

namespace stf {

constexpr float DCT_DC = 0x1.020408p-7f;           // fl32(1/127)
constexpr float DCT_K = 0x1.822cb2p-6f;            // fl32((2/15) / (4 sqrt 2)) = 0.0235702...
constexpr float DCT_K11 = 0x1.111112p-5f;          // fl32((2/15) / 4) = 0.0333333...
// |cos(k pi/16)| for k = 1, 3, 5, 7 and |cos(k pi/8)| for k = 1, 3
constexpr float DCT_C1 = 0x1.f6297cp-1f, DCT_C3 = 0x1.a9b662p-1f, DCT_C5 = 0x1.1c73b4p-1f, DCT_C7 = 0x1.8f8b84p-3f;
constexpr float DCT_D1 = 0x1.d906bcp-1f, DCT_D3 = 0x1.87de2ap-2f;

// c1(i) = cos((2i+1) pi/16): +C1 +C3 +C5 +C7 -C7 -C5 -C3 -C1 for i = 0..7.
__device__ __forceinline__ float dct_c1(int i)
{
    int j = i < 4 ? i : 7 - i;
    float m = j == 0 ? DCT_C1 : (j == 1 ? DCT_C3 : (j == 2 ? DCT_C5 : DCT_C7));
    return i < 4 ? m : -m;
}

// c2(i) = cos((2i+1) pi/8): +D1 +D3 -D3 -D1 -D1 -D3 +D3 +D1 for i = 0..7.
__device__ __forceinline__ float dct_c2(int i)
{
    float m = (i == 0 || i == 3 || i == 4 || i == 7) ? DCT_D1 : DCT_D3;
    return (i >= 2 && i <= 5) ? -m : m;
}

// The five AC basis values of texel (xi, yi) of a block, scaled by the
// dequantisation step: B[k-1] for zigzag coefficient k = 1..5.
struct DctBasis {
    float b[5];
};

__device__ __forceinline__ DctBasis dct_basis(int xi, int yi)
{
    const float c1x = dct_c1(xi), c1y = dct_c1(yi), c2x = dct_c2(xi), c2y = dct_c2(yi);
    DctBasis B;
    B.b[0] = DCT_K * c1x;           // (v, u) = (0, 1)
    B.b[1] = DCT_K * c1y;           // (1, 0)
    B.b[2] = DCT_K * c2y;           // (2, 0)
    B.b[3] = (DCT_K11 * c1x) * c1y; // (1, 1)
    B.b[4] = DCT_K * c2x;           // (0, 2)
    return B;
}

// Decode one channel word at a texel with basis B.  The AC codes become
// 5-bit two's complement q by flipping bit 4 of every field (q + 16 xor 16 =
// q mod 32), and are sign-extended by a signed bit-field extract.
__device__ __forceinline__ float dct_decode_word(uint32_t word, const DctBasis& B)
{
    const uint32_t w = word ^ 0x84210800u;   // bit 4 of each AC field (bits 11, 16, 21, 26, 31)
    float f = (float)(word & 127u) * DCT_DC;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const int q = __builtin_amdgcn_sbfe((int)w, 7 + 5 * k, 5);
        f = __builtin_fmaf((float)q, B.b[k], f);
    }
    return f;
}

// ---------------------------------------------------------------------------
// Weighted sums of decoded texels by block.
//
// A texel is a sum of six products of a code and a function of x and of y, so
// a tensor-product weighted sum of the texels of one block needs no texel.  In
// units of 1/127, with S0 = sum wx, S1 = sum wx e1(x), S2 = sum wx e2(x) over
// the window's columns in the block, e_k = 127 K c_k, and T0..T2 the same over
// its rows,
//   127 sum wx wy f(x, y) = d T0 S0 + q1 T0 S1 + q2 T1 S0 + q3 T2 S0 +
//                           (60/127) q4 T1 S1 + q5 T0 S2
// (127 K11 c1 c1 = (60/127) e1 e1): six multiply-adds per channel and block
// instead of a decode per tap.  The taps of a 4x4 window meet 1.9 blocks on
// average (1, 2 or 4).
//
// Rounding.  The DC term carries nearly all of a sum, and one error in its
// factor is an error of the whole result, where a decode per tap averages the
// errors of 16 taps.  So that term is kept nearly free of them: d is taken as
// the integer it is, the larger weight sum of an axis's two blocks is what the
// smaller one leaves of the axis's total (a constant of the kind, so a window
// within one block has an exact factor, and an error moves weight between two
// neighbouring blocks instead of adding some; the smaller one keeps its
// relative error, for the blocks next to black ones), and the AC terms are
// added up by themselves before the DC term.  Against binary64 the results of
// all kinds are nearer than the sums of texels decoded one by one: B-spline
// 4.9e-8 to 7.2e-8, Keys 5.0e-8 to 8.3e-8 (relative root mean square, noise
// textures; 9.1e-8 and 11.4e-8 with the DC term first, the 1/127 and 1/36 in
// its factor and every sum added up).
// ---------------------------------------------------------------------------
constexpr double DCT_E = 127.0 * (2.0 / 15.0) / (4.0 * 1.4142135623730951);   // 127 K
constexpr float DCT_R11 = (float)(60.0 / 127.0);

// The weight sums of the columns (or rows) of a window in one block.
struct DctAxis {
    float s0, s1, s2;
};

// The row sums as a y block's factors take them, shared by its x blocks.
struct DctRow {
    float t0, t1, t2, r1;
};

__device__ __forceinline__ DctRow dct_row(const DctAxis& t)
{
    return {t.s0, t.s1, t.s2, DCT_R11 * t.s1};
}

// Factors of the DC code and the five AC codes of every channel of a block
// (named values: an indexed array here would leave the registers).
struct DctFactors {
    float b0, b1, b2, b3, b4, b5;
};

__device__ __forceinline__ DctFactors dct_factors(const DctRow& r, const DctAxis& s)
{
    return {r.t0 * s.s0, r.t0 * s.s1, r.t1 * s.s0, r.t2 * s.s0, r.r1 * s.s1, r.t0 * s.s2};
}

// The six codes of a channel word as binary32 (exact): DC 0..127, AC -15..15.
struct DctCodes {
    float c0, c1, c2, c3, c4, c5;
};

__device__ __forceinline__ DctCodes dct_codes(uint32_t word)
{
    const int w = (int)(word ^ 0x84210800u);   // as in dct_decode_word
    return {(float)(word & 127u),
            (float)(int)__builtin_amdgcn_sbfe(w, 7, 5),
            (float)(int)__builtin_amdgcn_sbfe(w, 12, 5),
            (float)(int)__builtin_amdgcn_sbfe(w, 17, 5),
            (float)(int)__builtin_amdgcn_sbfe(w, 22, 5),
            (float)(int)__builtin_amdgcn_sbfe(w, 27, 5)};
}

// acc + sum_k c_k b_k, in this order wherever the codes come from.
__device__ __forceinline__ float dct_accumulate(const DctCodes& c, const DctFactors& F, float acc)
{
    float t = c.c5 * F.b5;
    t = __builtin_fmaf(c.c4, F.b4, t);
    t = __builtin_fmaf(c.c3, F.b3, t);
    t = __builtin_fmaf(c.c2, F.b2, t);
    t = __builtin_fmaf(c.c1, F.b1, t);
    return acc + __builtin_fmaf(c.c0, F.b0, t);
}

// acc / (127 S), the reciprocal in two parts where its rounding (1.8e-8 for
// the B-spline's 36, 3.7e-9 for 1 and 4) would show.
template <int S>
__device__ __forceinline__ float dct_unscale(float acc)
{
    constexpr double inv = 1.0 / (127.0 * S);
    constexpr float hi = (float)inv, lo = (float)(inv - (double)hi);
    if constexpr (S == 1 || S == 4) return acc * hi;
    return __builtin_fmaf(acc, hi, acc * lo);
}

// e1(i), e2(i) for i = 0..7 in LDS, filled by the block's first eight
// threads; the caller synchronises before the first read.
__device__ __forceinline__ void dct_fill_cosines(float2* tab)
{
    constexpr double C[4] = {0.98078528040323044913, 0.83146961230254523708, 0.55557023301960222474,
                             0.19509032201612826785};   // cos(k pi/16), k = 1, 3, 5, 7
    constexpr double D[2] = {0.92387953251128675613, 0.38268343236508977173};   // cos(k pi/8), k = 1, 3
    const int i = (int)threadIdx.x;
    if (i >= 8) return;
    const int j = i < 4 ? i : 7 - i;
    const float e1 = j == 0 ? (float)(DCT_E * C[0]) : j == 1 ? (float)(DCT_E * C[1]) : j == 2 ? (float)(DCT_E * C[2]) : (float)(DCT_E * C[3]);
    const float e2 = j == 0 || j == 3 ? (float)(DCT_E * D[0]) : (float)(DCT_E * D[1]);
    tab[i] = make_float2(i < 4 ? e1 : -e1, j < 2 ? e2 : -e2);
}

// Adds the tap at (clamped) texel coordinate x with weight w to S1 and S2.
__device__ __forceinline__ void dct_axis_add(DctAxis& a, const float2* tab, int x, float w)
{
    const float2 c = tab[x & 7];
    a.s1 = __builtin_fmaf(w, c.x, a.s1);
    a.s2 = __builtin_fmaf(w, c.y, a.s2);
}

// The weight sums of NT <= 8 consecutive taps from x0, clamped to [0, hi], in
// the (at most two) blocks they meet; total: the sum of the weights.
struct DctAxisPair {
    int blk0, blk1;
    DctAxis a0, a1;
};

template <int NT>
__device__ __forceinline__ DctAxisPair dct_axis_pair(const float2* tab, int x0, int hi, const float (&w)[4], float total)
{
    auto clamped = [&](int x) { return x < 0 ? 0 : (x > hi ? hi : x); };
    DctAxisPair r = {clamped(x0) >> 3, clamped(x0 + NT - 1) >> 3, {0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f}};
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        const int x = clamped(x0 + k);
        const bool second = (x >> 3) != r.blk0;
        const float w0 = second ? 0.0f : w[k], w1 = second ? w[k] : 0.0f;
        r.a0.s0 += w0;
        r.a1.s0 += w1;
        dct_axis_add(r.a0, tab, x, w0);
        dct_axis_add(r.a1, tab, x, w1);
    }
    const float s0 = r.a0.s0, s1 = r.a1.s0;
    const bool first = __builtin_fabsf(s0) > __builtin_fabsf(s1);
    r.a0.s0 = first ? total - s1 : s0;
    r.a1.s0 = first ? s1 : total - s0;
    return r;
}

}  // namespace stf
