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
// A texel is a sum of six products of a coefficient and a function of x and
// of y, so a tensor-product weighted sum of the texels of one block needs no
// texel: with S0 = sum wx, S1 = sum wx c1(x), S2 = sum wx c2(x) over the
// window's columns in the block, and T0..T2 the same over its rows,
//   sum wx wy f(x, y) = d (T0 S0)/127 + K (q1 T0 S1 + q2 T1 S0 + q3 T2 S0 +
//                       q5 T0 S2) + K11 q4 T1 S1,
// six multiply-adds per channel and block instead of a decode per tap.  The
// taps of a 4x4 window meet 1.9 blocks on average (1, 2 or 4).
// ---------------------------------------------------------------------------

// The weight sums of the columns (or rows) of a window in one block.
struct DctAxis {
    float s0, s1, s2;
};

// The row sums scaled by the dequantisation steps: one per y block, shared by
// its x blocks.
struct DctRow {
    float dc, k0, k1, k2, k11;
};

__device__ __forceinline__ DctRow dct_row(const DctAxis& t)
{
    return {DCT_DC * t.s0, DCT_K * t.s0, DCT_K * t.s1, DCT_K * t.s2, DCT_K11 * t.s1};
}

// Factors of the DC code and the five AC codes of every channel of a block
// (named values: an indexed array here would leave the registers).
struct DctFactors {
    float b0, b1, b2, b3, b4, b5;
};

__device__ __forceinline__ DctFactors dct_factors(const DctRow& r, const DctAxis& s)
{
    return {r.dc * s.s0, r.k0 * s.s1, r.k1 * s.s0, r.k2 * s.s0, r.k11 * s.s1, r.k0 * s.s2};
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
    acc = __builtin_fmaf(c.c0, F.b0, acc);
    acc = __builtin_fmaf(c.c1, F.b1, acc);
    acc = __builtin_fmaf(c.c2, F.b2, acc);
    acc = __builtin_fmaf(c.c3, F.b3, acc);
    acc = __builtin_fmaf(c.c4, F.b4, acc);
    return __builtin_fmaf(c.c5, F.b5, acc);
}

// c1(i), c2(i) for i = 0..7 in LDS, filled by the block's first eight
// threads; the caller synchronises before the first read.
__device__ __forceinline__ void dct_fill_cosines(float2* tab)
{
    if (threadIdx.x < 8) tab[threadIdx.x] = make_float2(dct_c1((int)threadIdx.x), dct_c2((int)threadIdx.x));
}

// Adds the tap at (clamped) texel coordinate x with weight w.
__device__ __forceinline__ void dct_axis_add(DctAxis& a, const float2* tab, int x, float w)
{
    const float2 c = tab[x & 7];
    a.s0 += w;
    a.s1 = __builtin_fmaf(w, c.x, a.s1);
    a.s2 = __builtin_fmaf(w, c.y, a.s2);
}

// The weight sums of NT <= 8 consecutive taps from x0, clamped to [0, hi], in
// the (at most two) blocks they meet.
struct DctAxisPair {
    int blk0, blk1;
    DctAxis a0, a1;
};

template <int NT>
__device__ __forceinline__ DctAxisPair dct_axis_pair(const float2* tab, int x0, int hi, const float (&w)[4])
{
    auto clamped = [&](int x) { return x < 0 ? 0 : (x > hi ? hi : x); };
    DctAxisPair r = {clamped(x0) >> 3, clamped(x0 + NT - 1) >> 3, {0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f}};
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        const int x = clamped(x0 + k);
        const bool second = (x >> 3) != r.blk0;
        dct_axis_add(r.a0, tab, x, second ? 0.0f : w[k]);
        dct_axis_add(r.a1, tab, x, second ? w[k] : 0.0f);
    }
    return r;
}

}  // namespace stf
