// filter2d.hip -- filtering of 2D textures: bilinear / bicubic B-spline,
// deterministic (all 4 / 16 taps, Eq. filtered-texture with tensor-product
// weights) and stochastic (one tap per query, Eq. stochastic-sum with the
// per-axis draw of Eq. stochastic-bilerp / the bicubic sampling of section
// "B-Spline and Anisotropic Filters").  The interpolating cubics (Keys,
// Mitchell) filter deterministically with their 16 weights and
// stochastically by positivization: one tap from the positive and one from
// the negative weights (interp.h).
//
// Every kernel is generic over its texel source: stored texels of a format
// (DenseSrc), or DCT-compressed blocks (DctSrc), of which the stochastic
// filters decode one texel per lookup, the case the paper makes for
// compressed formats.  The deterministic filters of DCT blocks have kernels
// of their own, which weigh the blocks' coefficients and decode no texel.
//
// Raster position: x = uv.x * W - 0.5 (texel centres at half-integers of
// uv * W); taps are clamped to the texture.
#include <limits.h>
#include <math.h>

#include "dct_decode.h"
#include "device_common.h"
#include "interp.h"
#include "stf_internal.h"

using namespace stf;

namespace {

constexpr int BLOCK = 256;

__device__ __forceinline__ int clampi(int v, int hi)
{
    return v < 0 ? 0 : (v > hi ? hi : v);
}

// Stored texels: C channels of format FMT, row-major.  A texel, or a row of
// neighbouring texels, is read with as few loads as its size allows.
template <int FMT, int C>
struct DenseSrc {
    static constexpr int CAP = C;
    static constexpr bool DECODES = false;   // a texel is a plain load
    static constexpr bool WINDOWS = true;    // rows of taps are contiguous
    static constexpr int FORMAT = FMT;
    // Deterministic sums take U8 codes as they are and divide the sum by 255:
    // one instruction a value to decode, and the sum's own rounding only.
    static constexpr float RAW_SCALE = FMT == U8 ? 255.0f : 1.0f;
    TexLevel L;
    __device__ int w() const { return L.w; }
    __device__ int h() const { return L.h; }
    __device__ int channels() const { return C; }
    __device__ __forceinline__ const void* at(int x, int y) const
    {
        return static_cast<const char*>(L.texels) + ((int64_t)y * L.w + x) * (C * fmt_bytes(FMT));
    }
    __device__ void load(int x, int y, float (&v)[CAP]) const
    {
        TexelRun<FMT, C> t;
        t.load(at(x, y));
#pragma unroll
        for (int c = 0; c < C; ++c) v[c] = t.value(c);
    }
    __device__ void load_raw(int x, int y, float (&v)[CAP]) const
    {
        TexelRun<FMT, C> t;
        t.load(at(x, y));
#pragma unroll
        for (int c = 0; c < C; ++c) v[c] = t.template value<true>(c);
    }
};

// Material texels (8 bytes: albedo RGB UNORM8, roughness UNORM8, tangent
// normal x and y binary16; stored in 4x4-texel tiles, material_index) of
// level 0, decoded exactly to six channels.
struct MaterialSrc {
    static constexpr int CAP = 6;
    static constexpr bool DECODES = false;
    static constexpr bool WINDOWS = false;
    static constexpr float RAW_SCALE = 1.0f;
    TexLevel L;
    __device__ int w() const { return L.w; }
    __device__ int h() const { return L.h; }
    __device__ int channels() const { return 6; }
    __device__ void load(int x, int y, float (&v)[CAP]) const
    {
        const uint2 t = reinterpret_cast<const uint2*>(L.texels)[material_index(x, y, L.w)];
        v[0] = dec_u8(t.x & 0xffu);
        v[1] = dec_u8((t.x >> 8) & 0xffu);
        v[2] = dec_u8((t.x >> 16) & 0xffu);
        v[3] = dec_u8(t.x >> 24);
        v[4] = dec_f16((uint16_t)(t.y & 0xffffu));
        v[5] = dec_f16((uint16_t)(t.y >> 16));
    }
    __device__ void load_raw(int x, int y, float (&v)[CAP]) const { load(x, y, v); }
};

// DCT blocks: CAP words per block (a multiple of 4), C <= CAP channels used.
template <int CAP_>
struct DctSrc {
    static constexpr int CAP = CAP_;
    static constexpr bool DECODES = true;   // a texel costs an inverse DCT per channel
    const uint32_t* blocks;
    int32_t W, H, BW, C;
    __device__ int w() const { return W; }
    __device__ int h() const { return H; }
    __device__ int channels() const { return C; }
    __device__ void load(int x, int y, float (&v)[CAP]) const
    {
        const uint4* b = reinterpret_cast<const uint4*>(blocks + ((int64_t)(y >> 3) * BW + (x >> 3)) * CAP);
        const DctBasis B = dct_basis(x & 7, y & 7);
#pragma unroll
        for (int g = 0; g < CAP / 4; ++g) {
            const uint4 q = b[g];
            v[4 * g] = dct_decode_word(q.x, B);
            v[4 * g + 1] = dct_decode_word(q.y, B);
            v[4 * g + 2] = dct_decode_word(q.z, B);
            v[4 * g + 3] = dct_decode_word(q.w, B);
        }
    }
};

template <class Src>
__device__ __forceinline__ void store_channels(const Src& S, float* __restrict__ out, int64_t oi, const float* v)
{
    const int C = S.channels();
#pragma unroll
    for (int c = 0; c < Src::CAP; ++c)
        if (c < C) out[oi * C + c] = v[c];
}

// Stores the C results of every live query of the block.  In batch order the
// block's results are one contiguous span of cnt * C floats: each thread
// stages its values in LDS and the block writes the span with consecutive
// 16-byte stores (4-byte ones if the span is not 16-byte aligned), instead of
// C strided 4-byte stores per lane.  Scattered results (an ordered stream
// with STF_ORDER_SCATTER) are stored directly.  Every thread of the block
// must call this (it synchronises the block).
template <class Src>
__device__ __forceinline__ void block_store_via(const Src& S, float* __restrict__ out, int32_t n, bool live, int64_t oi,
                                                const float (&v)[Src::CAP], bool scattered, float* stage)
{
    const int C = S.channels();
    if (scattered) {
        if (live) store_channels(S, out, oi, v);
        return;
    }
#pragma unroll
    for (int c = 0; c < Src::CAP; ++c)
        if (c < C) stage[threadIdx.x * C + c] = v[c];
    __syncthreads();
    const int64_t first = (int64_t)blockIdx.x * BLOCK;
    const int cnt = (int)((int64_t)n - first < BLOCK ? (int64_t)n - first : BLOCK);
    const int total = cnt * C;
    float* dst = out + first * C;
    int k0 = 0;
    // the results are streamed out: nontemporal stores (1.37x on the DCT
    // set's stochastic bilinear, whose 36 bytes of results per lookup are
    // most of its traffic)
    typedef float f32x4_nt __attribute__((ext_vector_type(4)));
    if ((reinterpret_cast<uintptr_t>(dst) & 15u) == 0) {
        const int n4 = total >> 2;
        for (int k = threadIdx.x; k < n4; k += BLOCK)
            __builtin_nontemporal_store(reinterpret_cast<const f32x4_nt*>(stage)[k],
                                        reinterpret_cast<f32x4_nt*>(dst) + k);
        k0 = n4 << 2;
    }
    for (int k = k0 + threadIdx.x; k < total; k += BLOCK) __builtin_nontemporal_store(stage[k], dst + k);
}

// block_store_via with LDS of its own (BLOCK * CAP floats, 16-byte aligned).
template <class Src>
__device__ __forceinline__ void block_store(const Src& S, float* __restrict__ out, int32_t n, bool live, int64_t oi,
                                            const float (&v)[Src::CAP], bool scattered)
{
    __shared__ __align__(16) float stage[BLOCK * Src::CAP];
    block_store_via(S, out, n, live, oi, v, scattered, stage);
}

// Query i of a batch (i valid), drawn with id qid0 + i (or order[i]): its
// values, its tap (INT32_MIN for a non-finite query) and where its results go.
template <class Src, bool CUBIC, bool FIS = false>
__device__ __forceinline__ void tex2d_stochastic_eval(const Src& S, const float* __restrict__ q, int32_t i, uint32_t key,
                                                      uint32_t qid0, const int32_t* __restrict__ order, int scatter,
                                                      float (&v)[Src::CAP], int& sx, int& sy, int64_t& oi)
{
    const int32_t id = order ? order[i] : (int32_t)(qid0 + (uint32_t)i);
    oi = (order && scatter) ? (int64_t)id : (int64_t)i;
    float2 uv = reinterpret_cast<const float2*>(q)[i];
    float x = uv.x * (float)S.w() - 0.5f;
    float y = uv.y * (float)S.h() - 0.5f;
    int cx, cy;
    float tx, ty;
    bool ok = cell_of(x, cx, tx) & cell_of(y, cy, ty);
    sx = BAD_INDEX;
    sy = BAD_INDEX;
    if (ok) {
        uint32_t b = pcg(key ^ (uint32_t)id);
        if constexpr (FIS) {
            sx = fis_tap<CUBIC>(x, b, 0);
            sy = fis_tap<CUBIC>(y, b, 1);
        } else {
            float ux = axis_uniform(b, 0), uy = axis_uniform(b, 1);
            if constexpr (CUBIC) {
                sx = cx + choose_cubic(tx, ux);
                sy = cy + choose_cubic(ty, uy);
            } else {
                sx = cx + choose_linear(tx, ux);
                sy = cy + choose_linear(ty, uy);
            }
        }
        sx = clampi(sx, S.w() - 1);
        sy = clampi(sy, S.h() - 1);
        S.load(sx, sy, v);
    } else {
#pragma unroll
        for (int c = 0; c < Src::CAP; ++c) v[c] = __builtin_nanf("");
    }
}

template <class Src, bool CUBIC, bool FIS>
__global__ __launch_bounds__(BLOCK) void k_tex2d_stochastic(Src S, const float* __restrict__ q, int32_t n,
                                                            uint32_t key, float* __restrict__ out,
                                                            int32_t* __restrict__ idx, const int32_t* __restrict__ order,
                                                            int scatter)
{
    const int32_t i = blockIdx.x * BLOCK + threadIdx.x;
    const bool live = i < n;
    float v[Src::CAP];
    int sx, sy;
    int64_t oi;
    tex2d_stochastic_eval<Src, CUBIC, FIS>(S, q, live ? i : 0, key, 0u, order, scatter, v, sx, sy, oi);
    block_store(S, out, n, live, oi, v, order && scatter);
    if (live && idx) {
        idx[2 * oi] = sx;
        idx[2 * oi + 1] = sy;
    }
}

// Positivized estimate of an interpolating cubic for query i: two clamped
// taps, value (S+ t(j+) - S- t(j-)) / scale^2; index (x+, y+, x-, y-), the
// negative tap INT32_MIN when S- = 0.
template <class Src, int KIND>
__global__ __launch_bounds__(BLOCK) void k_tex2d_positivized(Src S, const float* __restrict__ q, int32_t n,
                                                             uint32_t key, float* __restrict__ out,
                                                             int32_t* __restrict__ idx,
                                                             const int32_t* __restrict__ order, int scatter)
{
    constexpr int CAP = Src::CAP;
    const int32_t i0 = blockIdx.x * BLOCK + threadIdx.x;
    const bool live = i0 < n;
    const int32_t i = live ? i0 : 0;
    const int32_t id = order ? order[i] : i;
    const int64_t oi = (order && scatter) ? (int64_t)id : (int64_t)i;
    float2 uv = reinterpret_cast<const float2*>(q)[i];
    float x = uv.x * (float)S.w() - 0.5f;
    float y = uv.y * (float)S.h() - 0.5f;
    int cx, cy;
    float tx, ty;
    bool ok = cell_of(x, cx, tx) & cell_of(y, cy, ty);
    float v[CAP];
    int ix[4] = {BAD_INDEX, BAD_INDEX, BAD_INDEX, BAD_INDEX};
    if (ok) {
        const float t[2] = {tx, ty};
        const PosDraw<2> d = positivized_draw<2, KIND>(t, pcg(key ^ (uint32_t)id));
        ix[0] = clampi(cx + d.op[0], S.w() - 1);
        ix[1] = clampi(cy + d.op[1], S.h() - 1);
        float vp[CAP], vn[CAP];
        S.load(ix[0], ix[1], vp);
        if (d.neg) {
            ix[2] = clampi(cx + d.on[0], S.w() - 1);
            ix[3] = clampi(cy + d.on[1], S.h() - 1);
            S.load(ix[2], ix[3], vn);
        }
        constexpr float inv = inv_scale<2, KIND>();
#pragma unroll
        for (int c = 0; c < CAP; ++c) v[c] = (d.neg ? d.sp * vp[c] - d.sn * vn[c] : d.sp * vp[c]) * inv;
    } else {
#pragma unroll
        for (int c = 0; c < CAP; ++c) v[c] = __builtin_nanf("");
    }
    block_store(S, out, n, live, oi, v, order && scatter);
    if (live && idx) {
#pragma unroll
        for (int k = 0; k < 4; ++k) idx[4 * oi + k] = ix[k];
    }
}

// Serving: block b serves chunk c with start[c] <= b < start[c + 1].
template <class Src, bool CUBIC>
__global__ __launch_bounds__(BLOCK) void k_tex2d_serve(Src S, const ServeChunk* __restrict__ chunks, int32_t nchunks)
{
    int lo = 0, hi = nchunks - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) / 2;
        if (chunks[mid].block0 <= (int32_t)blockIdx.x) lo = mid;
        else hi = mid - 1;
    }
    const ServeChunk c = chunks[lo];
    const int32_t i = ((int32_t)blockIdx.x - c.block0) * BLOCK + threadIdx.x;
    if (i >= c.count) return;
    float v[Src::CAP];
    int sx, sy;
    int64_t oi;
    tex2d_stochastic_eval<Src, CUBIC>(S, c.q, i, c.key, c.qid0, nullptr, 0, v, sx, sy, oi);
    store_channels(S, c.out, oi, v);
    if (c.idx) {
        c.idx[2 * oi] = sx;
        c.idx[2 * oi + 1] = sy;
    }
}

template <class Src, int KIND>
__global__ __launch_bounds__(BLOCK) void k_tex2d_deterministic(Src S, const float* __restrict__ q, int32_t n,
                                                               float* __restrict__ out, const int32_t* __restrict__ order,
                                                               int scatter)
{
    constexpr int NT = KIND == KIND_LINEAR ? 2 : 4;
    constexpr int CAP = Src::CAP;
    const int32_t i0 = blockIdx.x * BLOCK + threadIdx.x;
    const bool live = i0 < n;
    const int32_t i = live ? i0 : 0;
    const int64_t oi = (order && scatter) ? (int64_t)order[i] : (int64_t)i;
    float2 uv = reinterpret_cast<const float2*>(q)[i];
    float x = uv.x * (float)S.w() - 0.5f;
    float y = uv.y * (float)S.h() - 0.5f;
    int cx = 0, cy = 0;
    float tx = 0.0f, ty = 0.0f;
    const bool ok = cell_of(x, cx, tx) & cell_of(y, cy, ty);
    float acc[CAP];
    float wx[4], wy[4];
    cx += axis_weights_scaled<KIND>(tx, wx);
    cy += axis_weights_scaled<KIND>(ty, wy);
#pragma unroll
    for (int c = 0; c < CAP; ++c) acc[c] = 0.0f;
    // A row of NT taps is read whole, as the run of NT texels that holds every
    // tap the clamping leaves (from column xs): 4 loads of 16 bytes for 8-bit
    // RGBA and 16 taps instead of 64 of a byte each with their addresses.
    // Only where a lane of the wave has a tap to clamp, the texels of a row
    // are moved to their taps (taps left of the run take its first texel,
    // taps right of it its last).  Otherwise (tiled materials, textures
    // narrower than a row) every tap is loaded by itself; the values and the
    // order of the sum are the same.  2M pixels of a frame, 4096^2 8-bit RGBA,
    // bicubic: 59 us (loads and decoding) -> 20 us (half of it the streams);
    // scattered over 4096^2 binary32 RGBA: 332 -> 205 us (its lines); over 50
    // columns of one bfloat16 channel, every wave at a border: 31 -> 17 us.
    bool whole = false;
    if constexpr (Src::WINDOWS) whole = S.w() >= NT;
    if (whole) {
        if constexpr (Src::WINDOWS) {
            const int xs = clampi(cx, S.w() - NT), d = cx - xs;
            const bool clamps = __any(d != 0);
            TexelRun<Src::FORMAT, NT * CAP> run[NT];
#pragma unroll
            for (int b = 0; b < NT; ++b) run[b].load(S.at(xs, clampi(cy + b, S.h() - 1)));
#pragma unroll
            for (int b = 0; b < NT; ++b) {
                float t[NT][CAP];
#pragma unroll
                for (int a = 0; a < NT; ++a)
#pragma unroll
                    for (int c = 0; c < CAP; ++c) t[a][c] = run[b].template value<true>(a * CAP + c);
                if (clamps) {
#pragma unroll
                    for (int c = 0; c < CAP; ++c) {
                        if constexpr (NT == 4) {
                            const bool l1 = d == 1 || d >= 3, l2 = d >= 2, r1 = d == -1 || d <= -3, r2 = d <= -2;
                            t[0][c] = l1 ? t[1][c] : t[0][c];
                            t[1][c] = l1 ? t[2][c] : t[1][c];
                            t[2][c] = l1 ? t[3][c] : t[2][c];
                            t[0][c] = l2 ? t[2][c] : t[0][c];
                            t[1][c] = l2 ? t[3][c] : t[1][c];
                            t[2][c] = l2 ? t[3][c] : t[2][c];
                            t[3][c] = r1 ? t[2][c] : t[3][c];
                            t[2][c] = r1 ? t[1][c] : t[2][c];
                            t[1][c] = r1 ? t[0][c] : t[1][c];
                            t[3][c] = r2 ? t[1][c] : t[3][c];
                            t[2][c] = r2 ? t[0][c] : t[2][c];
                            t[1][c] = r2 ? t[0][c] : t[1][c];
                        } else {
                            const float t0 = t[0][c];
                            t[0][c] = d >= 1 ? t[1][c] : t0;
                            t[1][c] = d <= -1 ? t0 : t[1][c];
                        }
                    }
                }
                float row[CAP];
#pragma unroll
                for (int c = 0; c < CAP; ++c) row[c] = 0.0f;
#pragma unroll
                for (int a = 0; a < NT; ++a)
#pragma unroll
                    for (int c = 0; c < CAP; ++c) row[c] = __builtin_fmaf(wx[a], t[a][c], row[c]);
#pragma unroll
                for (int c = 0; c < CAP; ++c) acc[c] = __builtin_fmaf(wy[b], row[c], acc[c]);
            }
        }
    } else {
        // Wide sources (materials, six channels) keep one row of taps in
        // flight: unrolling all rows would hold every tap's texel at once.
        constexpr int ROWS_UNROLLED = CAP > 4 ? 1 : NT;
#pragma unroll ROWS_UNROLLED
        for (int b = 0; b < NT; ++b) {
            int yy = clampi(cy + b, S.h() - 1);
            float row[CAP];
#pragma unroll
            for (int c = 0; c < CAP; ++c) row[c] = 0.0f;
#pragma unroll
            for (int a = 0; a < NT; ++a) {
                float v[CAP];
                S.load_raw(clampi(cx + a, S.w() - 1), yy, v);
#pragma unroll
                for (int c = 0; c < CAP; ++c) row[c] = __builtin_fmaf(wx[a], v[c], row[c]);
            }
#pragma unroll
            for (int c = 0; c < CAP; ++c) acc[c] = __builtin_fmaf(wy[b], row[c], acc[c]);
        }
    }
    // 36 (B-spline), 4 (Keys), 324 (Mitchell), by the 255 of U8 codes
    constexpr float S2 = axis_scale<KIND>() * axis_scale<KIND>() * Src::RAW_SCALE;
#pragma unroll
    for (int c = 0; c < CAP; ++c) acc[c] = !ok ? __builtin_nanf("") : (S2 == 1.0f ? acc[c] : acc[c] / S2);
    block_store(S, out, n, live, oi, acc, order && scatter);
}

// Discrete Gaussian weights of the 4x4 window i-1..i+2 (binary64, unnormalised).
__device__ __forceinline__ void gauss_discrete_weights(double t, double inv2s2, double (&w)[4])
{
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double d = (double)(k - 1) - t;
        w[k] = exp(-(d * d) * inv2s2);
    }
}

// The discrete Gaussian mean (normalised 4x4 window) as a deterministic kind.
constexpr int KIND_GAUSS_MEAN = 100;

template <int CAP>
__device__ __forceinline__ void dct_load_words(const DctSrc<CAP>& S, int bx, int by, uint4 (&w4)[CAP / 4])
{
    const uint4* b = reinterpret_cast<const uint4*>(S.blocks + ((int64_t)by * S.BW + bx) * CAP);
#pragma unroll
    for (int g = 0; g < CAP / 4; ++g) w4[g] = b[g];
}

// Adds a block's channels (`left` of the four words) to their sums, a whole
// group without a test between them.  By value: the two ways' common code,
// merged over references, would index the sums at run time.
__device__ __forceinline__ float4 dct_add_group(uint4 w, DctFactors F, int left, float4 a)
{
    if (left >= 4) {
        a.x = dct_accumulate(dct_codes(w.x), F, a.x);
        a.y = dct_accumulate(dct_codes(w.y), F, a.y);
        a.z = dct_accumulate(dct_codes(w.z), F, a.z);
        a.w = dct_accumulate(dct_codes(w.w), F, a.w);
    } else {
        if (left > 0) a.x = dct_accumulate(dct_codes(w.x), F, a.x);
        if (left > 1) a.y = dct_accumulate(dct_codes(w.y), F, a.y);
        if (left > 2) a.z = dct_accumulate(dct_codes(w.z), F, a.z);
    }
    return a;
}

template <int CAP>
__device__ __forceinline__ void dct_add_words(const uint4 (&w4)[CAP / 4], const DctFactors& F, int C,
                                              float (&acc)[CAP])
{
#pragma unroll
    for (int g = 0; g < CAP / 4; ++g) {
        const float4 a = dct_add_group(w4[g], F, C - 4 * g,
                                       make_float4(acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]));
        acc[4 * g] = a.x;
        acc[4 * g + 1] = a.y;
        acc[4 * g + 2] = a.z;
        acc[4 * g + 3] = a.w;
    }
}

// Deterministic filtering of a DCT texture by blocks (dct_decode.h): the
// window's weight sums per axis and block, then six multiply-adds per channel
// and block the window meets, instead of decoding each of its 4 or 16 texels.
//
// With STAGE (the 16-tap kinds) the threads first decide together whether
// their windows lie close enough to share blocks, as those of a frame in
// pixel order or of a sorted stream do: at least STAGE_REUSE queries per block
// of the bounding box of their taps, and the codes of its blocks fit the
// tile.  Then the codes of the box's blocks are unpacked once into LDS (8
// floats per channel: 6 codes, 16-byte reads); otherwise each query unpacks
// the words of its own blocks.  Both ways see the same codes and accumulate
// them in the same order, so the results are the same, bit for bit.
//
// Bound by VALU issue (weight sums and the multiply-adds; the streams alone
// would take 75 us of the frame below).  4K frame of a 4096^2 set of 9
// channels, 16 taps: 507 us with each texel of the taps' box decoded into
// LDS once, 124 us so (128 as the sums are rounded now); 2M uniform uv: 228 us
// decoding every tap, 106 us so; 4 taps, 4 channels, 2M pixels of a frame: 20.9 and 15.2 us.  An unguarded
// group of four channels lets its LDS reads overlap (a test per channel: 141
// us); tiles of 16, 20 and 32 KiB: 127, 124 and 147 us (the last one leaves 4
// blocks per CU).
constexpr int STAGE_FLOATS = 5120;   // 20 KiB per block: 8 blocks per CU
// A staged block costs about as much as two queries unpacking it.
constexpr int STAGE_REUSE = 2;

template <int CAP, int KIND, bool STAGE>
__global__ __launch_bounds__(BLOCK) void k_dct_det(DctSrc<CAP> S, const float* __restrict__ q, int32_t n,
                                                   float* __restrict__ out, const int32_t* __restrict__ order,
                                                   int scatter, unsigned long long* __restrict__ counters, float sigma)
{
    constexpr int NT = KIND == KIND_LINEAR ? 2 : 4;
    constexpr int TILE = STAGE ? STAGE_FLOATS : BLOCK * CAP;
    static_assert(BLOCK * CAP <= TILE, "the tile also stages the block's results");
    __shared__ __align__(16) float tile[TILE];
    __shared__ float2 cosines[8];
    __shared__ int box[5][BLOCK / 64];
    dct_fill_cosines(cosines);
    const int32_t i0 = blockIdx.x * BLOCK + threadIdx.x;
    const bool live = i0 < n;
    const int32_t i = live ? i0 : 0;
    const int64_t oi = (order && scatter) ? (int64_t)order[i] : (int64_t)i;
    const float2 uv = reinterpret_cast<const float2*>(q)[i];
    const float x = uv.x * (float)S.w() - 0.5f;
    const float y = uv.y * (float)S.h() - 0.5f;
    int cx = 0, cy = 0;
    float tx = 0.0f, ty = 0.0f;
    const bool ok = cell_of(x, cx, tx) & cell_of(y, cy, ty);
    float wx[4], wy[4];
    if constexpr (KIND == KIND_GAUSS_MEAN) {
        // as k_tex2d_gauss's discrete mean: binary64 weights, normalised, in binary32
        const double sg = (double)sigma, inv2s2 = 1.0 / (2.0 * sg * sg);
        const double xe = (double)x, ye = (double)y;
        double dx[4], dy[4];
        gauss_discrete_weights(xe - floor(xe), inv2s2, dx);
        gauss_discrete_weights(ye - floor(ye), inv2s2, dy);
        const double nx = ((dx[0] + dx[1]) + dx[2]) + dx[3], ny = ((dy[0] + dy[1]) + dy[2]) + dy[3];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            wx[k] = (float)(dx[k] / nx);
            wy[k] = (float)(dy[k] / ny);
        }
        cx -= 1;
        cy -= 1;
    } else {
        cx += axis_weights_scaled<KIND>(tx, wx);
        cy += axis_weights_scaled<KIND>(ty, wy);
    }
    const int W1 = S.w() - 1, H1 = S.h() - 1;
    const int C = S.channels();
    // each channel's 6 codes take 8 floats; an odd multiple of 8 per block
    // spreads the blocks a wave reads over the banks
    const int bstride = (C | 1) * 8;
    bool stage = false;
    int bx0 = 0, by0 = 0, nbx = 0, nby = 0;   // the box's blocks
    if constexpr (STAGE) {
        // box of the clamped taps of the block's queries (clamping is monotone)
        const bool in = live && ok;
        const int m[4] = {wave_min(in ? clampi(cx, W1) : INT_MAX), wave_min(in ? -clampi(cx + NT - 1, W1) : INT_MAX),
                          wave_min(in ? clampi(cy, H1) : INT_MAX), wave_min(in ? -clampi(cy + NT - 1, H1) : INT_MAX)};
        const int cnt = __popcll(__ballot(in));
        if (threadIdx.x % 64 == 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) box[k][threadIdx.x / 64] = m[k];
            box[4][threadIdx.x / 64] = cnt;
        }
    }
    __syncthreads();
    if constexpr (STAGE) {
        // wave-uniform from here on
        int r[4], nin = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            int v = box[k][0];
#pragma unroll
            for (int w = 1; w < BLOCK / 64; ++w) v = min(v, box[k][w]);
            r[k] = __builtin_amdgcn_readfirstlane(v);
        }
#pragma unroll
        for (int w = 0; w < BLOCK / 64; ++w) nin += __builtin_amdgcn_readfirstlane(box[4][w]);
        if (nin) {
            bx0 = r[0] >> 3;
            by0 = r[2] >> 3;
            nbx = (-r[1] >> 3) - bx0 + 1;   // 1..8192 blocks per axis
            nby = (-r[3] >> 3) - by0 + 1;
        }
        const int nb = nbx * nby;   // at most 2^26
        // the same decision in every thread of the block
        stage = nb && nb <= TILE / bstride && nb * STAGE_REUSE <= nin;
        if (counters && threadIdx.x == 0) {   // {blocks that staged, blocks}, when counting is on
            if (stage) atomicAdd(&counters[0], 1ull);
            atomicAdd(&counters[1], 1ull);
        }
        if (stage) {
            // a thread unpacks four channel words of a block
            constexpr int G = CAP / 4;
            const float inv_nbx = 1.0f / (float)nbx;
            for (int t = threadIdx.x; t < nb * G; t += BLOCK) {
                const int b = t / G, g = t - b * G;
                const int yb = (int)(((float)b + 0.5f) * inv_nbx), xb = b - yb * nbx;   // b < 512: exact
                const uint4 w4 = reinterpret_cast<const uint4*>(
                    S.blocks + ((int64_t)(by0 + yb) * S.BW + bx0 + xb) * CAP)[g];
                float* e = tile + b * bstride + g * 32;
                const uint32_t w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (4 * g + j < C) {
                        const DctCodes k = dct_codes(w[j]);
                        *reinterpret_cast<float4*>(e + 8 * j) = make_float4(k.c0, k.c1, k.c2, k.c3);
                        *reinterpret_cast<float2*>(e + 8 * j + 4) = make_float2(k.c4, k.c5);
                    }
                }
            }
            __syncthreads();
        }
    }
    // the weights of an axis add up to the kind's scale (the mean's are normalised)
    constexpr float total = KIND == KIND_GAUSS_MEAN ? 1.0f : axis_scale<KIND>();
    const DctAxisPair px = dct_axis_pair<NT>(cosines, cx, W1, wx, total);
    const DctAxisPair py = dct_axis_pair<NT>(cosines, cy, H1, wy, total);
    float acc[CAP];
#pragma unroll
    for (int c = 0; c < CAP; ++c) acc[c] = 0.0f;
    const bool use = live && ok;
    if constexpr (!STAGE) {
        // The first block, then the lane's second one along x or y (along
        // neither: weight 0), their words in flight together, then for lanes
        // with taps in four blocks the other two.  On scattered queries a wave
        // meets all four, but a lane in 64 has four: block after block for the
        // whole wave 6M random uv of 9 channels take 297 us, so 146 (4
        // channels, 2M: 69 and 26).
        const bool sx = px.blk1 != px.blk0, sy = py.blk1 != py.blk0;
        const bool more = __any(use && (sx || sy));
        uint4 w0[CAP / 4], w1[CAP / 4];
        dct_load_words(S, px.blk0, py.blk0, w0);
        if (more) dct_load_words(S, px.blk1, sx ? py.blk0 : py.blk1, w1);
        const DctRow r0 = dct_row(py.a0), r1 = dct_row(py.a1);
        dct_add_words<CAP>(w0, dct_factors(r0, px.a0), C, acc);
        if (more) {
            const DctRow r = {sx ? r0.t0 : r1.t0, sx ? r0.t1 : r1.t1, sx ? r0.t2 : r1.t2, sx ? r0.r1 : r1.r1};
            const DctAxis a = {sx ? px.a1.s0 : px.a0.s0, sx ? px.a1.s1 : px.a0.s1, sx ? px.a1.s2 : px.a0.s2};
            dct_add_words<CAP>(w1, dct_factors(r, a), C, acc);
            if (use && sx && sy) {
                dct_load_words(S, px.blk0, py.blk1, w0);
                dct_load_words(S, px.blk1, py.blk1, w1);
                dct_add_words<CAP>(w0, dct_factors(r1, px.a0), C, acc);
                dct_add_words<CAP>(w1, dct_factors(r1, px.a1), C, acc);
            }
        }
    } else {
        // the (at most) four blocks; a second block without taps has weight 0
        const int nv = __any(use && py.blk1 != py.blk0) ? 2 : 1, nu = __any(use && px.blk1 != px.blk0) ? 2 : 1;
#pragma unroll 1
        for (int v = 0; v < nv; ++v) {
            const DctRow row = dct_row({v ? py.a1.s0 : py.a0.s0, v ? py.a1.s1 : py.a0.s1, v ? py.a1.s2 : py.a0.s2});
            const int by = v ? py.blk1 : py.blk0;
#pragma unroll 1
            for (int u = 0; u < nu; ++u) {
                const DctFactors F = dct_factors(row, {u ? px.a1.s0 : px.a0.s0, u ? px.a1.s1 : px.a0.s1,
                                                       u ? px.a1.s2 : px.a0.s2});
                const int bx = u ? px.blk1 : px.blk0;
                // whole groups of four channels without a test between them
                if (stage) {   // (a query without a cell reads the first block)
                    const float* e = tile + (use ? ((by - by0) * nbx + (bx - bx0)) * bstride : 0);
                    auto one = [&](int c) {
                        const float4 k0 = *reinterpret_cast<const float4*>(e + 8 * c);
                        const float2 k1 = *reinterpret_cast<const float2*>(e + 8 * c + 4);
                        acc[c] = dct_accumulate({k0.x, k0.y, k0.z, k0.w, k1.x, k1.y}, F, acc[c]);
                    };
#pragma unroll
                    for (int g = 0; g < CAP; g += 4) {
                        if (g + 4 <= C) {
                            one(g);
                            one(g + 1);
                            one(g + 2);
                            one(g + 3);
                        } else {
                            if (g < C) one(g);
                            if (g + 1 < C) one(g + 1);
                            if (g + 2 < C) one(g + 2);
                        }
                    }
                } else {
                    uint4 w4[CAP / 4];
                    dct_load_words(S, bx, by, w4);
                    dct_add_words<CAP>(w4, F, C, acc);
                }
            }
        }
    }
#pragma unroll
    for (int c = 0; c < CAP; ++c) acc[c] = ok ? dct_unscale<(int)(total * total)>(acc[c]) : __builtin_nanf("");
    if constexpr (STAGE) __syncthreads();   // every thread is done with the tile: it now stages the results
    block_store_via(S, out, n, live, oi, acc, order && scatter, tile);
}

// Bilinear filtering of a DCT texture in small calls, a thread per query and
// group of four channels: with all channels in one thread the chain of its up to
// four blocks is the time of a call that leaves most of the chip idle.  The
// sums are those of k_dct_det, in its order: the same bits.  1,000 scattered
// queries of 16 channels: 5.7 us decoding each tap, 7.9 with a thread per query,
// 3.0 so; 60,000 of 9: 5.3, 5.0, 4.2; 200,000 in a frame: 8.7, 5.9, 7.9, hence
// the line.
constexpr int64_t DCT_GROUPS_TO = 65536;   // a block of queries per CU

template <int CAP>
__global__ __launch_bounds__(BLOCK) void k_dct_linear_groups(DctSrc<CAP> S, const float* __restrict__ q, int32_t n,
                                                             float* __restrict__ out, const int32_t* __restrict__ order,
                                                             int scatter)
{
    constexpr int G = CAP / 4;
    __shared__ float2 cosines[8];
    dct_fill_cosines(cosines);
    __syncthreads();
    const int32_t t = blockIdx.x * BLOCK + threadIdx.x, i = t / G, g = t % G;   // t < 4 DCT_GROUPS_TO + BLOCK
    const int left = S.channels() - 4 * g;
    if (i >= n || left <= 0) return;
    const float2 uv = reinterpret_cast<const float2*>(q)[i];
    int cx = 0, cy = 0;
    float tx = 0.0f, ty = 0.0f;
    const bool ok = cell_of(uv.x * (float)S.w() - 0.5f, cx, tx) & cell_of(uv.y * (float)S.h() - 0.5f, cy, ty);
    float wx[4], wy[4];
    cx += axis_weights_scaled<KIND_LINEAR>(tx, wx);
    cy += axis_weights_scaled<KIND_LINEAR>(ty, wy);
    const DctAxisPair px = dct_axis_pair<2>(cosines, cx, S.w() - 1, wx, 1.0f);
    const DctAxisPair py = dct_axis_pair<2>(cosines, cy, S.h() - 1, wy, 1.0f);
    const bool sx = px.blk1 != px.blk0, sy = py.blk1 != py.blk0;
    auto words = [&](int bx, int by) {
        return reinterpret_cast<const uint4*>(S.blocks + ((int64_t)by * S.BW + bx) * CAP)[g];
    };
    // a lane without a second, third or fourth block asks for its first again
    const uint4 w0 = words(px.blk0, py.blk0), w1 = words(px.blk1, sx ? py.blk0 : py.blk1),
                w2 = words(px.blk0, py.blk1), w3 = words(px.blk1, py.blk1);
    const DctRow r0 = dct_row(py.a0), r1 = dct_row(py.a1);
    float4 acc = dct_add_group(w0, dct_factors(r0, px.a0), left, make_float4(0.0f, 0.0f, 0.0f, 0.0f));
    const DctRow r = {sx ? r0.t0 : r1.t0, sx ? r0.t1 : r1.t1, sx ? r0.t2 : r1.t2, sx ? r0.r1 : r1.r1};
    const DctAxis a = {sx ? px.a1.s0 : px.a0.s0, sx ? px.a1.s1 : px.a0.s1, sx ? px.a1.s2 : px.a0.s2};
    acc = dct_add_group(w1, dct_factors(r, a), left, acc);
    if (sx && sy) {
        acc = dct_add_group(w2, dct_factors(r1, px.a0), left, acc);
        acc = dct_add_group(w3, dct_factors(r1, px.a1), left, acc);
    }
    const float v[4] = {acc.x, acc.y, acc.z, acc.w};
    float* o = out + ((order && scatter) ? (int64_t)order[i] : (int64_t)i) * S.channels() + 4 * g;
#pragma unroll
    for (int c = 0; c < 4; ++c)
        if (c < left) o[c] = ok ? dct_unscale<1>(v[c]) : __builtin_nanf("");
}

// channel-0 moments of the stochastic estimator over many seeds
template <class Src, int KIND>
__global__ __launch_bounds__(BLOCK) void k_tex2d_moments(Src S, const float* __restrict__ q, int32_t n,
                                                         uint64_t seed_base, int32_t n_seeds,
                                                         double* __restrict__ sum, double* __restrict__ sumsq)
{
    constexpr int CAP = Src::CAP;
    __shared__ double s1[BLOCK], s2[BLOCK];
    int32_t i = blockIdx.x;
    float2 uv = reinterpret_cast<const float2*>(q)[i];
    float x = uv.x * (float)S.w() - 0.5f;
    float y = uv.y * (float)S.h() - 0.5f;
    int cx, cy;
    float tx, ty;
    bool ok = cell_of(x, cx, tx) & cell_of(y, cy, ty);
    double a1 = 0.0, a2 = 0.0;
    if (ok) {
        for (int32_t k = threadIdx.x; k < n_seeds; k += BLOCK) {
            uint32_t b = pcg(seed_key(seed_base + (uint64_t)k) ^ (uint32_t)i);
            float e;
            if constexpr (KIND == KIND_KEYS || KIND == KIND_MITCHELL) {
                const float t[2] = {tx, ty};
                const PosDraw<2> d = positivized_draw<2, KIND>(t, b);
                float vp[CAP], vn[CAP];
                S.load(clampi(cx + d.op[0], S.w() - 1), clampi(cy + d.op[1], S.h() - 1), vp);
                e = d.sp * vp[0];
                if (d.neg) {
                    S.load(clampi(cx + d.on[0], S.w() - 1), clampi(cy + d.on[1], S.h() - 1), vn);
                    e = e - d.sn * vn[0];
                }
                e = e * inv_scale<2, KIND>();
            } else {
                float ux = axis_uniform(b, 0), uy = axis_uniform(b, 1);
                int sx, sy;
                if constexpr (KIND == KIND_BSPLINE) {
                    sx = cx + choose_cubic(tx, ux); sy = cy + choose_cubic(ty, uy);
                } else {
                    sx = cx + choose_linear(tx, ux); sy = cy + choose_linear(ty, uy);
                }
                float v[CAP];
                S.load(clampi(sx, S.w() - 1), clampi(sy, S.h() - 1), v);
                e = v[0];
            }
            double d = (double)e;
            a1 += d;
            a2 += d * d;
        }
    } else {
        a1 = a2 = __builtin_nan("");
    }
    s1[threadIdx.x] = a1;
    s2[threadIdx.x] = a2;
    __syncthreads();
    for (int stride = BLOCK / 2; stride > 0; stride >>= 1) {
        if (threadIdx.x < stride) {
            s1[threadIdx.x] += s1[threadIdx.x + stride];
            s2[threadIdx.x] += s2[threadIdx.x + stride];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        sum[i] = s1[0];
        sumsq[i] = s2[0];
    }
}

// ---------------------------------------------------------------------------
// Gaussian filters (sections "Filter Importance Sampling" and "Results",
// magnification).  Decisions and weights in binary64; sigma in texels.
//   GAUSS_FIS: offset sigma (r cos 2 pi u1, r sin 2 pi u1), r = sqrt(-2 ln(1 -
//     u0)) (Box-Muller of hash indices 0, 1), nearest texel floor(x' + 1/2).
//   GAUSS_FIS_MEAN: the Gaussian convolved with the nearest-texel box (what
//     GAUSS_FIS estimates): per-axis weights Phi((k + 1/2 - x)/sigma) -
//     Phi((k - 1/2 - x)/sigma) over |k - floor(x)| <= R = ceil(6 sigma) + 1.
//   GAUSS_DISCRETE: window i-1..i+2, per-axis weights exp(-(d - t)^2 /
//     (2 sigma^2)), one tap per axis by the cumulative rule (hash index a).
//   GAUSS_DISCRETE_MEAN: the normalised sum over that window.
// ---------------------------------------------------------------------------
enum GaussMode { GAUSS_FIS = 0, GAUSS_FIS_MEAN = 1, GAUSS_DISCRETE = 2, GAUSS_DISCRETE_MEAN = 3 };
constexpr int GAUSS_MAX_TAPS = 52;   // 2 R + 2 for sigma <= 4 (GAUSS_FIS_MEAN)

__device__ __forceinline__ double gauss_phi(double z)
{
    return 0.5 * erfc(-z * 0.70710678118654752440);
}

__device__ __forceinline__ int gauss_pick(const double (&m)[4], double u)
{
    const double total = ((m[0] + m[1]) + m[2]) + m[3];
    const int last = m[3] > 0.0 ? 3 : (m[2] > 0.0 ? 2 : (m[1] > 0.0 ? 1 : 0));
    const double T = u * total;
    int j = (T >= m[0]) + (T >= m[0] + m[1]) + (T >= (m[0] + m[1]) + m[2]);
    return j > last ? last : j;
}

// The discrete pick with binary32 weights, for sigma >= 1/4 (every weight is
// then at least e^-32: none underflows and none is clamped).  A weight is
// 2^(a log2 e) with a = -d^2 / (2 sigma^2), |a| <= 32, by the hardware's 2^x.
// The exponent carries a few ulps from d^2, 1/(2 sigma^2) and the scaling by
// log2 e (at most 1.4e-5 + 4.2e-6 absolute), and 2^x is within 8.5e-8
// relative over [-64, 0] (measured on every binary32 value there against
// binary64), so each weight is within 2e-5 relative of its binary64 value,
// and u * total and the cumulative sums lie within 4e-5 total of theirs;
// where u * total is at least total 2^-12 from every cumulative sum, the pick
// is the binary64 pick.  Returns -1 otherwise.
__device__ __forceinline__ int gauss_pick_fast(float t, float inv2s2, float u)
{
    float m[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float d = (float)(k - 1) - t;
        m[k] = __builtin_amdgcn_exp2f((-(d * d) * inv2s2) * 1.44269504088896341f);
    }
    const float c1 = m[0], c2 = m[0] + m[1], c3 = (m[0] + m[1]) + m[2];
    const float total = c3 + m[3];
    const float T = u * total;
    if (fminf(fminf(fabsf(T - c1), fabsf(T - c2)), fabsf(T - c3)) < total * 0x1p-12f) return -1;
    return (T >= c1) + (T >= c2) + (T >= c3);
}

template <class Src, int GMODE>
__global__ __launch_bounds__(BLOCK) void k_tex2d_gauss(Src S, const float* __restrict__ q, int32_t n, float sigma,
                                                       int32_t radius, uint32_t key, float* __restrict__ out,
                                                       int32_t* __restrict__ idx)
{
    constexpr int CAP = Src::CAP;
    const int32_t i0 = blockIdx.x * BLOCK + threadIdx.x;
    const bool live = i0 < n;
    const int32_t i = live ? i0 : 0;
    float2 uv = reinterpret_cast<const float2*>(q)[i];
    const float x = uv.x * (float)S.w() - 0.5f;
    const float y = uv.y * (float)S.h() - 0.5f;
    int cx = 0, cy = 0;
    float tx = 0.0f, ty = 0.0f;
    const bool ok = cell_of(x, cx, tx) & cell_of(y, cy, ty);
    const double xe = (double)x, ye = (double)y, sg = (double)sigma;
    float v[CAP];
    int sx = BAD_INDEX, sy = BAD_INDEX;
    if constexpr (GMODE == GAUSS_FIS || GMODE == GAUSS_DISCRETE) {
        if (ok) {
            const uint32_t b = pcg(key ^ (uint32_t)i);
            const float u0f = axis_uniform(b, 0), u1f = axis_uniform(b, 1);
            const double u0 = (double)u0f, u1 = (double)u1f;
            if constexpr (GMODE == GAUSS_FIS) {
                // The offset is first formed in binary32 with the hardware's
                // log2, square root, sine and cosine (the last two take the
                // angle in turns, so u1 needs no scaling by 2 pi).  1 - u0 is
                // exact, and over all 2^24 values a uniform can take, r is
                // within 4.9e-7 of sqrt(-2 ln(1 - u0)) and the sine and cosine
                // within 1.3e-7 of sin and cos(2 pi u1) (measured exhaustively
                // against binary64), so with the products' rounding the offset
                // lies within 2e-6 sigma texels of the binary64 offset
                // (r <= 5.8).  A sample at least sigma 2^-14 from a texel edge
                // therefore takes the same texel as the binary64 sample;
                // nearer ones (about one query in 4,000 per unit sigma) redo
                // the offset in binary64.
                const float rf = __builtin_amdgcn_sqrtf(-1.38629436112f * __builtin_amdgcn_logf(1.0f - u0f));
                const float sf = __builtin_amdgcn_sinf(u1f), cf = __builtin_amdgcn_cosf(u1f);
                const double zx = (xe + (double)(sigma * (rf * cf))) + 0.5;
                const double zy = (ye + (double)(sigma * (rf * sf))) + 0.5;
                double fx = floor(zx), fy = floor(zy);
                const double margin = sg * 0x1p-14;
                if (fmin(fmin(zx - fx, (fx + 1.0) - zx), fmin(zy - fy, (fy + 1.0) - zy)) < margin) {
                    const double r = sqrt(-2.0 * log(1.0 - u0));
                    const double a = 6.28318530717958647692 * u1;
                    double sa, ca;
                    sincos(a, &sa, &ca);   // one argument reduction for both
                    const double xs = xe + sg * (r * ca), ys = ye + sg * (r * sa);
                    fx = floor(xs + 0.5);
                    fy = floor(ys + 0.5);
                }
                sx = (int)fmin(fmax(fx, -1.0), (double)S.w());
                sy = (int)fmin(fmax(fy, -1.0), (double)S.h());
            } else {
                const double inv2s2 = 1.0 / (2.0 * sg * sg);
                int jx = -1, jy = -1;
                if (sigma >= 0.25f) {
                    jx = gauss_pick_fast(x - floorf(x), (float)inv2s2, u0f);
                    jy = gauss_pick_fast(y - floorf(y), (float)inv2s2, u1f);
                }
                if (jx < 0) {
                    double wx[4];
                    gauss_discrete_weights(xe - floor(xe), inv2s2, wx);
                    jx = gauss_pick(wx, u0);
                }
                if (jy < 0) {
                    double wy[4];
                    gauss_discrete_weights(ye - floor(ye), inv2s2, wy);
                    jy = gauss_pick(wy, u1);
                }
                sx = cx - 1 + jx;
                sy = cy - 1 + jy;
            }
            sx = clampi(sx, S.w() - 1);
            sy = clampi(sy, S.h() - 1);
            S.load(sx, sy, v);
        } else {
#pragma unroll
            for (int c = 0; c < CAP; ++c) v[c] = __builtin_nanf("");
        }
    } else if constexpr (GMODE == GAUSS_DISCRETE_MEAN) {
        const double inv2s2 = 1.0 / (2.0 * sg * sg);
        double dx[4], dy[4];
        gauss_discrete_weights(xe - floor(xe), inv2s2, dx);
        gauss_discrete_weights(ye - floor(ye), inv2s2, dy);
        const double nx = ((dx[0] + dx[1]) + dx[2]) + dx[3], ny = ((dy[0] + dy[1]) + dy[2]) + dy[3];
        float wx[4], wy[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            wx[k] = (float)(dx[k] / nx);
            wy[k] = (float)(dy[k] / ny);
        }
        float acc[CAP];
#pragma unroll
        for (int c = 0; c < CAP; ++c) acc[c] = 0.0f;
        for (int b = 0; b < 4; ++b) {
            const int yy = clampi(cy - 1 + b, S.h() - 1);
            float row[CAP];
#pragma unroll
            for (int c = 0; c < CAP; ++c) row[c] = 0.0f;
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                float t[CAP];
                S.load(clampi(cx - 1 + a, S.w() - 1), yy, t);
#pragma unroll
                for (int c = 0; c < CAP; ++c) row[c] = __builtin_fmaf(wx[a], t[c], row[c]);
            }
#pragma unroll
            for (int c = 0; c < CAP; ++c) acc[c] = __builtin_fmaf(wy[b], row[c], acc[c]);
        }
#pragma unroll
        for (int c = 0; c < CAP; ++c) v[c] = ok ? acc[c] : __builtin_nanf("");
    } else {   // GAUSS_FIS_MEAN
        // The x weights of the window are kept in LDS, one column per thread
        // (a run-time sized array in registers would live in scratch), in
        // 2R + 2 rows of BLOCK floats sized at launch, so that the block
        // takes no more LDS than its radius needs; the y weights follow as
        // running differences in the row loop.
        extern __shared__ float wxs[];
        const int nt = 2 * radius + 2;
        double px = gauss_phi(((double)(cx - radius) - xe - 0.5) / sg);
        double py = gauss_phi(((double)(cy - radius) - ye - 0.5) / sg);
        for (int k = 0; k < nt; ++k) {
            const double qx = gauss_phi(((double)(cx - radius + k) - xe + 0.5) / sg);
            wxs[k * BLOCK + threadIdx.x] = (float)(qx - px);
            px = qx;
        }
        float acc[CAP];
#pragma unroll
        for (int c = 0; c < CAP; ++c) acc[c] = 0.0f;
        for (int b = 0; b < nt; ++b) {
            const double qy = gauss_phi(((double)(cy - radius + b) - ye + 0.5) / sg);
            const float wyb = (float)(qy - py);
            py = qy;
            const int yy = clampi(cy - radius + b, S.h() - 1);
            float row[CAP];
#pragma unroll
            for (int c = 0; c < CAP; ++c) row[c] = 0.0f;
            for (int a = 0; a < nt; ++a) {
                float t[CAP];
                S.load(clampi(cx - radius + a, S.w() - 1), yy, t);
                const float wxa = wxs[a * BLOCK + threadIdx.x];
#pragma unroll
                for (int c = 0; c < CAP; ++c) row[c] = __builtin_fmaf(wxa, t[c], row[c]);
            }
#pragma unroll
            for (int c = 0; c < CAP; ++c) acc[c] = __builtin_fmaf(wyb, row[c], acc[c]);
        }
#pragma unroll
        for (int c = 0; c < CAP; ++c) v[c] = ok ? acc[c] : __builtin_nanf("");
    }
    block_store(S, out, n, live, (int64_t)i, v, false);
    if (live && idx && (GMODE == GAUSS_FIS || GMODE == GAUSS_DISCRETE)) {
        idx[2 * (int64_t)i] = sx;
        idx[2 * (int64_t)i + 1] = sy;
    }
}

// GAUSS_FIS_MEAN of a DCT texture by blocks (dct_decode.h): the (2R + 2)^2
// taps meet at most ((2R + 8) / 8 + 1)^2 blocks, six multiply-adds per channel
// each, instead of a decode per tap.  Each thread keeps the weight sums of its
// columns per block in LDS (three values a block, one column per thread, rows
// sized at launch) and takes its rows block by block, so that the lanes of a
// wave read words together whatever their phase in a block.  Bound by the
// binary64 erfc of each window edge; 2M pixels of a frame, 9 channels, sigma
// 0.5 (100 taps): 1238 us with a decode per tap, 320 us so.
template <int CAP>
__global__ __launch_bounds__(BLOCK) void k_dct_gauss_mean(DctSrc<CAP> S, const float* __restrict__ q, int32_t n,
                                                          float sigma, int32_t radius, float* __restrict__ out)
{
    extern __shared__ __align__(16) float sums[];
    __shared__ float2 cosines[8];
    dct_fill_cosines(cosines);
    __syncthreads();
    const int32_t i0 = blockIdx.x * BLOCK + threadIdx.x;
    const bool live = i0 < n;
    const float2 uv = reinterpret_cast<const float2*>(q)[live ? i0 : 0];
    const float x = uv.x * (float)S.w() - 0.5f;
    const float y = uv.y * (float)S.h() - 0.5f;
    int cx = 0, cy = 0;
    float tx = 0.0f, ty = 0.0f;
    const bool ok = cell_of(x, cx, tx) & cell_of(y, cy, ty);
    const int nt = live && ok ? 2 * radius + 2 : 0;   // no taps without a cell
    const double sg = (double)sigma;
    // weights of one axis in tap order: running differences of Phi
    const int W1 = S.w() - 1, H1 = S.h() - 1, x0 = cx - radius, y0 = cy - radius;
    const double xe = (double)x, ye = (double)y;
    const int bx0 = clampi(x0, W1) >> 3;
    int nbx = 0;
    {
        double p = gauss_phi(((double)x0 - xe - 0.5) / sg);
        for (int k = 0; __any(k < nt);) {
            DctAxis a = {0.0f, 0.0f, 0.0f};
            const double first = p;
            for (int b = clampi(x0 + k, W1) >> 3; k < nt && clampi(x0 + k, W1) >> 3 == b; ++k) {
                const double e = gauss_phi(((double)(x0 + k) - xe + 0.5) / sg);
                dct_axis_add(a, cosines, clampi(x0 + k, W1), (float)(e - p));
                p = e;
            }
            a.s0 = (float)(p - first);   // the differences' sum, rounded once
            sums[(3 * nbx) * BLOCK + threadIdx.x] = a.s0;   // (a lane that is done writes zeros, at most
            sums[(3 * nbx + 1) * BLOCK + threadIdx.x] = a.s1;   // as many rows as the widest lane)
            sums[(3 * nbx + 2) * BLOCK + threadIdx.x] = a.s2;
            ++nbx;
        }
    }
    float acc[CAP];
#pragma unroll
    for (int c = 0; c < CAP; ++c) acc[c] = 0.0f;
    const int C = S.channels(), BX1 = W1 >> 3;
    double p = gauss_phi(((double)y0 - ye - 0.5) / sg);
    for (int k = 0; __any(k < nt);) {
        DctAxis a = {0.0f, 0.0f, 0.0f};
        const int by = clampi(y0 + k, H1) >> 3;
        const double first = p;
        for (; k < nt && clampi(y0 + k, H1) >> 3 == by; ++k) {
            const double e = gauss_phi(((double)(y0 + k) - ye + 0.5) / sg);
            dct_axis_add(a, cosines, clampi(y0 + k, H1), (float)(e - p));
            p = e;
        }
        a.s0 = (float)(p - first);
        const DctRow row = dct_row(a);
        for (int u = 0; u < nbx; ++u) {   // the same count in every lane of the wave
            const float* e = sums + 3 * u * BLOCK + threadIdx.x;
            const DctFactors F = dct_factors(row, {e[0], e[BLOCK], e[2 * BLOCK]});
            const int bx = bx0 + u < BX1 ? bx0 + u : BX1;
            const uint4* b = reinterpret_cast<const uint4*>(S.blocks + ((int64_t)by * S.BW + bx) * CAP);
#pragma unroll
            for (int g = 0; g < CAP / 4; ++g) {
                if (4 * g < C) {   // (padding words of the last group add to unused channels)
                    const uint4 w = b[g];
                    acc[4 * g] = dct_accumulate(dct_codes(w.x), F, acc[4 * g]);
                    acc[4 * g + 1] = dct_accumulate(dct_codes(w.y), F, acc[4 * g + 1]);
                    acc[4 * g + 2] = dct_accumulate(dct_codes(w.z), F, acc[4 * g + 2]);
                    acc[4 * g + 3] = dct_accumulate(dct_codes(w.w), F, acc[4 * g + 3]);
                }
            }
        }
    }
#pragma unroll
    for (int c = 0; c < CAP; ++c) acc[c] = ok ? dct_unscale<1>(acc[c]) : __builtin_nanf("");
    __syncthreads();   // the LDS rows now stage the results
    block_store_via(S, out, n, live, (int64_t)i0, acc, false, sums);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <class Src, int KIND>
void launch2d_kind(const Src& S, const float* q, int32_t n, int mode, uint32_t key, float* out, int32_t* idx,
                   const int32_t* order, int scatter, hipStream_t stream)
{
    dim3 grid((n + BLOCK - 1) / BLOCK), block(BLOCK);
    if (mode == STF_STOCHASTIC) {
        if constexpr (KIND == KIND_KEYS || KIND == KIND_MITCHELL)
            hipLaunchKernelGGL((k_tex2d_positivized<Src, KIND>), grid, block, 0, stream, S, q, n, key, out, idx, order,
                               scatter);
        else
            hipLaunchKernelGGL((k_tex2d_stochastic<Src, KIND == KIND_BSPLINE, false>), grid, block, 0, stream, S, q, n,
                               key, out, idx, order, scatter);
    } else if (mode == STF_STOCHASTIC_FIS) {
        if constexpr (KIND == KIND_LINEAR || KIND == KIND_BSPLINE)
            hipLaunchKernelGGL((k_tex2d_stochastic<Src, KIND == KIND_BSPLINE, true>), grid, block, 0, stream, S, q, n,
                               key, out, idx, order, scatter);
    } else {
        if constexpr (Src::DECODES && KIND == KIND_LINEAR && Src::CAP > 4)
            if (n <= DCT_GROUPS_TO) {
                hipLaunchKernelGGL((k_dct_linear_groups<Src::CAP>), dim3((unsigned)((n * (Src::CAP / 4) + BLOCK - 1) / BLOCK)),
                                   block, 0, stream, S, q, n, out, order, scatter);
                return;
            }
        if constexpr (Src::DECODES)   // by blocks; bilinear windows (2x2) share too little to stage
            hipLaunchKernelGGL((k_dct_det<Src::CAP, KIND, KIND != KIND_LINEAR>), grid, block, 0, stream, S, q, n, out,
                               order, scatter, KIND != KIND_LINEAR ? stage_counters() : nullptr, 0.0f);
        else
            hipLaunchKernelGGL((k_tex2d_deterministic<Src, KIND>), grid, block, 0, stream, S, q, n, out, order,
                               scatter);
    }
}

template <class Src>
hipError_t launch2d_src(const Src& S, const float* q, int32_t n, int filter, int mode, uint32_t key, float* out,
                        int32_t* idx, const int32_t* order, int scatter, hipStream_t stream)
{
    switch (filter) {
    case KIND_LINEAR: launch2d_kind<Src, KIND_LINEAR>(S, q, n, mode, key, out, idx, order, scatter, stream); break;
    case KIND_BSPLINE: launch2d_kind<Src, KIND_BSPLINE>(S, q, n, mode, key, out, idx, order, scatter, stream); break;
    case KIND_KEYS: launch2d_kind<Src, KIND_KEYS>(S, q, n, mode, key, out, idx, order, scatter, stream); break;
    case KIND_MITCHELL: launch2d_kind<Src, KIND_MITCHELL>(S, q, n, mode, key, out, idx, order, scatter, stream); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <class Src>
hipError_t moments2d_src(const Src& S, const float* q, int32_t n, int filter, uint64_t seed_base, int32_t n_seeds,
                         double* sum, double* sumsq, hipStream_t stream)
{
    dim3 grid(n), block(BLOCK);
    switch (filter) {
    case KIND_LINEAR:
        hipLaunchKernelGGL((k_tex2d_moments<Src, KIND_LINEAR>), grid, block, 0, stream, S, q, n, seed_base, n_seeds, sum,
                           sumsq);
        break;
    case KIND_BSPLINE:
        hipLaunchKernelGGL((k_tex2d_moments<Src, KIND_BSPLINE>), grid, block, 0, stream, S, q, n, seed_base, n_seeds,
                           sum, sumsq);
        break;
    case KIND_KEYS:
        hipLaunchKernelGGL((k_tex2d_moments<Src, KIND_KEYS>), grid, block, 0, stream, S, q, n, seed_base, n_seeds, sum,
                           sumsq);
        break;
    case KIND_MITCHELL:
        hipLaunchKernelGGL((k_tex2d_moments<Src, KIND_MITCHELL>), grid, block, 0, stream, S, q, n, seed_base, n_seeds,
                           sum, sumsq);
        break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int FMT, class F>
hipError_t with_dense(const stf_texture* t, F&& f)
{
    const TexLevel& L = t->level[0];
    switch (t->channels) {
    case 1: return f(DenseSrc<FMT, 1>{L});
    case 2: return f(DenseSrc<FMT, 2>{L});
    case 3: return f(DenseSrc<FMT, 3>{L});
    case 4: return f(DenseSrc<FMT, 4>{L});
    }
    return hipErrorInvalidValue;
}

// Calls f with the texel source of a 2D texture: a dense format and channel
// count, or DCT blocks and their padded word count.
template <class F>
hipError_t with_src(const stf_texture* t, F&& f)
{
    if (t->kind == STF_KIND_MATERIAL) return f(MaterialSrc{t->level[0]});
    if (t->kind == STF_KIND_DCT2D) {
        const TexLevel& L = t->level[0];
        const uint32_t* b = static_cast<const uint32_t*>(L.texels);
        switch (t->dct_wpb) {
        case 4: return f(DctSrc<4>{b, L.w, L.h, L.w / 8, t->channels});
        case 8: return f(DctSrc<8>{b, L.w, L.h, L.w / 8, t->channels});
        case 12: return f(DctSrc<12>{b, L.w, L.h, L.w / 8, t->channels});
        case 16: return f(DctSrc<16>{b, L.w, L.h, L.w / 8, t->channels});
        }
        return hipErrorInvalidValue;
    }
    switch (t->fmt) {
    case F32: return with_dense<F32>(t, f);
    case F16: return with_dense<F16>(t, f);
    case BF16: return with_dense<BF16>(t, f);
    case FP8_E4M3: return with_dense<FP8_E4M3>(t, f);
    case U8: return with_dense<U8>(t, f);
    }
    return hipErrorInvalidValue;
}

template <class Src>
hipError_t gauss2d_src(const Src& S, const float* q, int32_t n, float sigma, int gmode, uint32_t key, float* out,
                       int32_t* idx, hipStream_t stream)
{
    dim3 grid((n + BLOCK - 1) / BLOCK), block(BLOCK);
    const int32_t radius = (int32_t)ceilf(6.0f * sigma) + 1;
    switch (gmode) {
    case GAUSS_FIS:
        hipLaunchKernelGGL((k_tex2d_gauss<Src, GAUSS_FIS>), grid, block, 0, stream, S, q, n, sigma, radius, key, out,
                           idx);
        break;
    case GAUSS_FIS_MEAN:
        if (2 * radius + 2 > GAUSS_MAX_TAPS) return hipErrorInvalidValue;
        if constexpr (Src::DECODES) {
            const size_t rows = 3 * (size_t)((2 * radius + 2 + 6) / 8 + 1);   // blocks the columns can meet
            const size_t floats = rows > (size_t)Src::CAP ? rows : (size_t)Src::CAP;
            hipLaunchKernelGGL((k_dct_gauss_mean<Src::CAP>), grid, block, floats * BLOCK * sizeof(float), stream, S, q,
                               n, sigma, radius, out);
        } else {
            hipLaunchKernelGGL((k_tex2d_gauss<Src, GAUSS_FIS_MEAN>), grid, block,
                               (size_t)(2 * radius + 2) * BLOCK * sizeof(float), stream, S, q, n, sigma, radius, key,
                               out, idx);
        }
        break;
    case GAUSS_DISCRETE:
        hipLaunchKernelGGL((k_tex2d_gauss<Src, GAUSS_DISCRETE>), grid, block, 0, stream, S, q, n, sigma, radius, key,
                           out, idx);
        break;
    case GAUSS_DISCRETE_MEAN:
        if constexpr (Src::DECODES)
            hipLaunchKernelGGL((k_dct_det<Src::CAP, KIND_GAUSS_MEAN, true>), grid, block, 0, stream, S, q, n, out,
                               nullptr, 0, stage_counters(), sigma);
        else
            hipLaunchKernelGGL((k_tex2d_gauss<Src, GAUSS_DISCRETE_MEAN>), grid, block, 0, stream, S, q, n, sigma,
                               radius, key, out, idx);
        break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gauss2d(const stf_texture* t, const float* q, int32_t n, float sigma, int gmode, uint32_t key,
                          float* out, int32_t* idx, hipStream_t s)
{
    return with_src(t, [&](auto S) { return gauss2d_src(S, q, n, sigma, gmode, key, out, idx, s); });
}

hipError_t launch_filter2d(const stf_texture* t, const float* q, int32_t n, int filter, int mode, uint32_t key,
                           float* out, int32_t* idx, const int32_t* order, int scatter, hipStream_t s)
{
    return with_src(t, [&](auto S) { return launch2d_src(S, q, n, filter, mode, key, out, idx, order, scatter, s); });
}

hipError_t launch_moments2d(const stf_texture* t, const float* q, int32_t n, int filter, uint64_t seed_base,
                            int32_t n_seeds, double* sum, double* sumsq, hipStream_t s)
{
    return with_src(t, [&](auto S) { return moments2d_src(S, q, n, filter, seed_base, n_seeds, sum, sumsq, s); });
}

int32_t serve2d_queries_per_block()
{
    return BLOCK;
}

hipError_t launch_serve2d(const stf_texture* t, int filter, const ServeChunk* chunks, int32_t nchunks, int32_t nblocks,
                          hipStream_t s)
{
    if (t->kind != STF_KIND_TEX2D && t->kind != STF_KIND_MATERIAL) return hipErrorInvalidValue;
    return with_src(t, [&](auto S) {
        using Src = decltype(S);
        if (filter == STF_CUBIC_BSPLINE)
            hipLaunchKernelGGL((k_tex2d_serve<Src, true>), dim3(nblocks), dim3(BLOCK), 0, s, S, chunks, nchunks);
        else
            hipLaunchKernelGGL((k_tex2d_serve<Src, false>), dim3(nblocks), dim3(BLOCK), 0, s, S, chunks, nchunks);
        return hipGetLastError();
    });
}
