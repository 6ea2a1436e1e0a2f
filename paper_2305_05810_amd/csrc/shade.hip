// shade.hip -- filtering with shading, section "Effect of Texture Filtering
// on Rendering" (Eqs. traditional-lighting-integral and
// our-lighting-integral): the texture filter applied to the material before
// the BSDF (shade after filter), to the shaded results of every tap (filter
// after shade), or sampled so that only one tap is shaded (stochastic; the
// filter factor f/p is 1).
//
// Shading is f^ = BSDF * cos(theta_i) for one incident direction: a GGX
// microfacet lobe (Trowbridge-Reitz D, height-correlated Smith G2, Schlick F
// with F0 = 0.04) plus a Lambertian albedo term, evaluated in binary32.
#include <math.h>

#include <type_traits>

#include "device_common.h"
#include "shade_grid.h"
#include "stf_internal.h"

using namespace stf;

namespace {

constexpr int BLOCK = 256;
constexpr float INV_PI = 0.318309886183790672f;

struct V3 {
    float x, y, z;
};

// Each operation rounded by itself: what decides the horizon and the specular
// peak, whose width is down to alpha = 1e-3, keeps its rounding.
__device__ __forceinline__ float dot(V3 a, V3 b)
{
    return a.x * b.x + a.y * b.y + a.z * b.z;
}

__device__ __forceinline__ float cross_norm2(V3 a, V3 b)
{
    const float cx = a.y * b.z - a.z * b.y;
    const float cy = a.z * b.x - a.x * b.z;
    const float cz = a.x * b.y - a.y * b.x;
    return cx * cx + cy * cy + cz * cz;
}

// Fused, for the shadowing terms, which are smooth.
__device__ __forceinline__ float cross_norm2_fma(V3 a, V3 b)
{
    const float cx = __builtin_fmaf(a.y, b.z, -(a.z * b.y));
    const float cy = __builtin_fmaf(a.z, b.x, -(a.x * b.z));
    const float cz = __builtin_fmaf(a.x, b.y, -(a.y * b.x));
    return __builtin_fmaf(cz, cz, __builtin_fmaf(cy, cy, cx * cx));
}

// The shading arithmetic uses the hardware's reciprocal, square root and
// reciprocal square root (about one ulp each) instead of correctly rounded
// division and square root sequences: the shaded value is already sensitive
// to the binary32 rounding of the half vector at the 1e-5 level, and no
// decision of the filter depends on it.
__device__ __forceinline__ float frcp(float x)
{
    return __builtin_amdgcn_rcpf(x);
}

__device__ __forceinline__ float fsqrt(float x)
{
    return __builtin_amdgcn_sqrtf(x);
}

// What the shading of every tap of a query shares: the directions, their half
// vector and the specular lobe's factor F / (2 pi).
struct Frame {
    V3 wo, wi, h;
    float ks;
};

__device__ __forceinline__ Frame frame_of(V3 wo, V3 wi)
{
    Frame f;
    f.wo = wo;
    f.wi = wi;
    V3 h = {wo.x + wi.x, wo.y + wi.y, wo.z + wi.z};
    const float il = __builtin_amdgcn_rsqf(h.x * h.x + h.y * h.y + h.z * h.z);
    f.h = {h.x * il, h.y * il, h.z * il};
    const float x = 1.0f - dot(wi, f.h), x2 = x * x;
    f.ks = (0.04f + 0.96f * (x2 * x2 * x)) * (0.5f * INV_PI);
    return f;
}

// f^ of a material is diffuse albedo / pi + ks specular, with
//   diffuse = n.wi,
//   specular = a^2 n.wi / (den^2 (n.wi Ro + n.wo Ri)),
//   den = a^2 (n.h)^2 + |n x h|^2,  Rw = sqrt((n.w)^2 + a^2 |n x w|^2):
// the product D G2 F n.wi / (4 n.wo n.wi) with Smith's
// G2 = 1 / (1 + Lambda(wo) + Lambda(wi)) = 2 n.wo n.wi / (n.wi Ro + n.wo Ri),
// so one reciprocal serves all of it.  Both are zero below the horizon.
__device__ __forceinline__ void lobes(const Frame& fr, float nx, float ny, float rough, float& diffuse, float& specular)
{
    const V3 n = {nx, ny, fsqrt(fmaxf(0.0f, 1.0f - nx * nx - ny * ny))};
    const float alpha = fmaxf(rough * rough, 1e-3f), a2 = alpha * alpha;
    const float no = dot(n, fr.wo), ni = dot(n, fr.wi), nh = dot(n, fr.h);
    const float den = nh * nh * a2 + cross_norm2(n, fr.h);
    const float Ro = fsqrt(__builtin_fmaf(a2, cross_norm2_fma(n, fr.wo), no * no));
    const float Ri = fsqrt(__builtin_fmaf(a2, cross_norm2_fma(n, fr.wi), ni * ni));
    const bool lit = (no > 0.0f) & (ni > 0.0f);
    const float s = a2 * ni * frcp(den * den * __builtin_fmaf(ni, Ro, no * Ri));
    diffuse = lit ? ni : 0.0f;
    specular = lit ? s : 0.0f;
}

// The texel's eight bytes: albedo and roughness codes, the normal's x and y.
struct Texel {
    float albedo[3];   // codes: 255 times the albedo
    float rough, nx, ny;
};

__device__ __forceinline__ Texel decode_texel(uint2 t)
{
    Texel m;
    m.albedo[0] = (float)(t.x & 0xffu);
    m.albedo[1] = (float)((t.x >> 8) & 0xffu);
    m.albedo[2] = (float)((t.x >> 16) & 0xffu);
    m.rough = dec_u8(t.x >> 24);
    m.nx = dec_f16((uint16_t)(t.y & 0xffffu));
    m.ny = dec_f16((uint16_t)(t.y >> 16));
    return m;
}

// The taps' weights of an axis add up to this: cubic6's are six times the
// B-spline's, and the scale goes with the constants at the end (a sixth rounded
// in every weight is off by 3e-8 each time).
template <bool CUBIC>
constexpr double window_scale()
{
    return CUBIC ? 36.0 : 1.0;
}

// A channel of f^ from sums over the taps: of the diffuse lobe times the albedo
// codes and of the specular one, or (ONE_SPECULAR) the specular lobe of the
// filtered material.  1 / (255 pi) scales the codes in two parts: one part alone
// is off by 5.2e-8, more than the rest of a matt value's rounding.
template <bool CUBIC, bool ONE_SPECULAR>
__device__ __forceinline__ float finish(const Frame& fr, float codes, float specular)
{
    constexpr double inv = 1.0 / (255.0 * 3.14159265358979323846 * window_scale<CUBIC>());
    constexpr float hi = (float)inv, lo = (float)(inv - (double)hi);
    const float d = __builtin_fmaf(codes, hi, codes * lo);
    const float ks = ONE_SPECULAR || !CUBIC ? fr.ks : fr.ks * (float)(1.0 / window_scale<CUBIC>());
    return specular == 0.0f ? d : __builtin_fmaf(ks, specular, d);   // ks has no value for opposite directions
}

__device__ __forceinline__ int clampi(int v, int hi)
{
    return v < 0 ? 0 : (v > hi ? hi : v);
}

struct Levels {
    TexLevel lv[3];
    int32_t n;
};

__device__ __forceinline__ int dpp_xor1(int v) { return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true); }   // quad_perm [1,0,3,2]
__device__ __forceinline__ int dpp_xor2(int v) { return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true); }   // quad_perm [2,3,0,1]
__device__ __forceinline__ float dpp_xor1(float v) { return __builtin_bit_cast(float, dpp_xor1(__builtin_bit_cast(int, v))); }
__device__ __forceinline__ float dpp_xor2(float v) { return __builtin_bit_cast(float, dpp_xor2(__builtin_bit_cast(int, v))); }

// The value of lane K of each group of N neighbouring lanes (2 or 4), in all of them.
template <int N, int K>
__device__ __forceinline__ int lane_of(int v)
{
    constexpr int CTRL = N == 4 ? K * 0x55 : (K ? 0xF5 : 0xA0);   // quad_perm [K,K,K,K], [K,K,2+K,2+K]
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, true);
}
template <int N, int K>
__device__ __forceinline__ float lane_of(float v)
{
    return __builtin_bit_cast(float, lane_of<N, K>(__builtin_bit_cast(int, v)));
}

// Sum over N neighbouring lanes (2 or 4), left in each of them.
template <int N>
__device__ __forceinline__ float lane_sum(float v)
{
    v += dpp_xor1(v);
    if constexpr (N == 4) v += dpp_xor2(v);
    return v;
}

// Sums of v[k] over the N lanes of a group, lane k ending with that of v[k]:
// each step keeps half of the values and adds the partner's share of them.
// The same sums, in the same order, as lane_sum's.
template <int N>
__device__ __forceinline__ float lane_sum_own(const float (&v)[N], int a)
{
    const bool odd = a & 1;
    const float r0 = (odd ? v[1] : v[0]) + dpp_xor1(odd ? v[0] : v[1]);
    if constexpr (N == 2) return r0;
    else {
        const float r1 = (odd ? v[3] : v[2]) + dpp_xor1(odd ? v[2] : v[3]);
        return (a & 2 ? r1 : r0) + dpp_xor2(a & 2 ? r0 : r1);
    }
}

// Calls f with the constants 0 .. N - 1.
template <int N, int K = 0, class F>
__device__ __forceinline__ void for_each(F&& f)
{
    if constexpr (K < N) {
        f(std::integral_constant<int, K>{});
        for_each<N, K + 1>(f);
    }
}

// Filtering before or after shading, a lane per column of the window (two or
// four lanes a query), so that a query's load is one row of the window: 16 or
// 32 bytes, one or two lines.
//
// On scattered queries the time goes into whole 128-byte lines, 3.1 a query for
// the 4 x 4 window: 1.8 GB for 4M queries, at 7.7 TB/s from the L2s' far side.
// With a lane per query the lines in flight exceeded the L2s, a line's halves
// were asked for by different instructions (31.8M requests for 14.1M lines, now
// 17.0M) and 16 loads a lane kept the address units busy. 4M
// scattered queries, 4 x 4: after shading 284 -> 238 us, before 282 -> 238.
template <bool CUBIC, int MODE>
__global__ __launch_bounds__(BLOCK) void k_shade_taps(Levels L, const float* __restrict__ q, int32_t n,
                                                      float* __restrict__ out)
{
    constexpr int NT = CUBIC ? 4 : 2;
    const int32_t i = blockIdx.x * (BLOCK / NT) + threadIdx.x / NT;
    const int a = threadIdx.x % NT;
    if (i >= n) return;
    const float* e = q + 9 * (int64_t)i;
    float r[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) r[k] = __builtin_nontemporal_load(e + k);   // streamed in
#pragma unroll
    for (int k = 0; k < 9; ++k) asm volatile("" : "+v"(r[k]));   // all of the record at once (see k_shade_one)
    const float u = r[0], v = r[1], s = r[2];
    int l = (int)(s >= 1.41421354f) + (int)(s >= 2.82842708f);
    l = l < L.n - 1 ? l : L.n - 1;
    const TexLevel T = l == 0 ? L.lv[0] : (l == 1 ? L.lv[1] : L.lv[2]);
    const uint2* tex = reinterpret_cast<const uint2*>(T.texels);
    int cx = 0, cy = 0;
    float tx = 0.0f, ty = 0.0f;
    const bool ok = cell_of(u * (float)T.w - 0.5f, cx, tx) & cell_of(v * (float)T.h - 0.5f, cy, ty);
    float wx, wy[NT];
    int x0 = cx, y0 = cy;
    if constexpr (CUBIC) {
        const Cubic6 ca = cubic6(tx), cb = cubic6(ty);
        wx = a == 0 ? ca.a0 : a == 1 ? ca.a1 : a == 2 ? ca.a2 : ca.a3;
        wy[0] = cb.a0; wy[1] = cb.a1; wy[2] = cb.a2; wy[3] = cb.a3;
        x0 -= 1;
        y0 -= 1;
    } else {
        wx = a ? tx : 1.0f - tx;
        wy[0] = 1.0f - ty; wy[1] = ty;
    }
    uint2 texel[NT];
    const int xx = clampi(x0 + a, T.w - 1);
#pragma unroll
    for (int b = 0; b < NT; ++b) texel[b] = tex[material_index(xx, clampi(y0 + b, T.h - 1), T.w)];
    const Frame fr = frame_of({r[3], r[4], r[5]}, {r[6], r[7], r[8]});
    float codes[3] = {0.0f, 0.0f, 0.0f}, spec = 0.0f, rough = 0.0f, nx = 0.0f, ny = 0.0f;
#pragma unroll
    for (int b = 0; b < NT; ++b) {
        const Texel m = decode_texel(texel[b]);
        const float w = wx * wy[b];
        float wd = w;   // the albedo's weight
        if constexpr (MODE == STF_SHADE_AFTER_FILTER) {
            rough = __builtin_fmaf(w, m.rough, rough);
            nx = __builtin_fmaf(w, m.nx, nx);
            ny = __builtin_fmaf(w, m.ny, ny);
        } else {
            float d, sp;
            lobes(fr, m.nx, m.ny, m.rough, d, sp);
            wd *= d;
            spec = __builtin_fmaf(w, sp, spec);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) codes[c] = __builtin_fmaf(wd, m.albedo[c], codes[c]);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) codes[c] = lane_sum<NT>(codes[c]);
    if constexpr (MODE == STF_SHADE_AFTER_FILTER) {
        float d;
        constexpr float inv = (float)(1.0 / window_scale<CUBIC>());
        lobes(fr, lane_sum<NT>(nx) * inv, lane_sum<NT>(ny) * inv, lane_sum<NT>(rough) * inv, d, spec);
#pragma unroll
        for (int c = 0; c < 3; ++c) codes[c] *= d;
    } else {
        spec = lane_sum<NT>(spec);
    }
    float* o = out + 3 * (int64_t)i;   // results are streamed out (nontemporal stores)
    auto put = [&](int c, float code) {
        __builtin_nontemporal_store(ok ? finish<CUBIC, MODE == STF_SHADE_AFTER_FILTER>(fr, code, spec) : __builtin_nanf(""), o + c);
    };
    if constexpr (CUBIC) {
        if (a < 3) put(a, a == 0 ? codes[0] : a == 1 ? codes[1] : codes[2]);
    } else {
        put(a, a ? codes[1] : codes[0]);
        if (a) put(2, codes[2]);
    }
}

// The same with a query a lane, for calls that fill the chip: the record, the
// location and the shading of a filtered texel are formed once, where above
// every lane of a group forms them for itself.  That work, not the lines, is
// the time where the texels come from the caches.  The lanes of a bicubic
// window's group take their columns of one query of the group after another
// (sixteen loads, all in flight), by moves within the group, and each ends with
// the sums of its own query; a bilinear window's four loads are a lane's own.
// The sums keep their order: the results are the same, bit for bit.  4M queries,
// before with a lane's sixteen loads, with a group a query, so:
//   4 x 4, scattered: 4096^2 253, 230, 228 us; 256^2 147, 141, 97;
//   frame: 4096^2 105, 120, 107; 256^2 73, 107, 74;
//   2 x 2 before shading, 256^2: scattered 80, 84, 78; frame 45, 51, 44;
//   after shading: 86, 93, 80; 60, 57, 56.
template <bool CUBIC, int MODE>
__global__ __launch_bounds__(BLOCK) void k_shade_lane(Levels L, const float* __restrict__ q, int32_t n,
                                                      float* __restrict__ out)
{
    constexpr int NT = CUBIC ? 4 : 2;
    constexpr bool AFTER = MODE == STF_SHADE_AFTER_FILTER;
    static_assert(AFTER || !CUBIC, "bicubic windows after shading go by groups");
    const int64_t own = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
    const bool live = own < n;
    const int64_t i = live ? own : n - 1;
    const float* e = q + 9 * i;
    float r[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) r[k] = __builtin_nontemporal_load(e + k);   // streamed in
#pragma unroll
    for (int k = 0; k < 9; ++k) asm volatile("" : "+v"(r[k]));   // all of the record at once (see k_shade_one)
    const float u = r[0], v = r[1], s = r[2];
    int l = (int)(s >= 1.41421354f) + (int)(s >= 2.82842708f);
    l = l < L.n - 1 ? l : L.n - 1;
    const TexLevel T0 = L.lv[0], T1 = L.lv[1], T2 = L.lv[2];
    const uint2* tex = static_cast<const uint2*>(l == 0 ? T0.texels : l == 1 ? T1.texels : T2.texels);
    const int W = l == 0 ? T0.w : l == 1 ? T1.w : T2.w, H = l == 0 ? T0.h : l == 1 ? T1.h : T2.h;
    int cx = 0, cy = 0;
    float tx = 0.0f, ty = 0.0f;
    const bool ok = cell_of(u * (float)W - 0.5f, cx, tx) & cell_of(v * (float)H - 0.5f, cy, ty);
    float wx[NT], wy[NT];
    if constexpr (CUBIC) {
        const Cubic6 ca = cubic6(tx), cb = cubic6(ty);
        wx[0] = ca.a0; wx[1] = ca.a1; wx[2] = ca.a2; wx[3] = ca.a3;
        wy[0] = cb.a0; wy[1] = cb.a1; wy[2] = cb.a2; wy[3] = cb.a3;
        cx -= 1;
        cy -= 1;
    } else {
        wx[0] = 1.0f - tx; wx[1] = tx;
        wy[0] = 1.0f - ty; wy[1] = ty;
    }
    // a texel's index is its row's share plus its column's (material_index; below 2^32)
    uint32_t row[NT];
#pragma unroll
    for (int b = 0; b < NT; ++b) row[b] = (uint32_t)material_index(0, clampi(cy + b, H - 1), W);
    auto column = [](int x) { return (uint32_t)((x >> 2) << 4 | (x & 3)); };
    // sums of the albedo codes, and of roughness and normal or the specular lobe
    constexpr int NS = AFTER ? 6 : 4;
    float sum[NS];
    auto add = [&](float (&t)[NS], uint2 texel, float w, const Frame& fr) {
        const Texel m = decode_texel(texel);
        float wd = w;   // the albedo's weight
        if constexpr (AFTER) {
            t[3] = __builtin_fmaf(w, m.rough, t[3]);
            t[4] = __builtin_fmaf(w, m.nx, t[4]);
            t[5] = __builtin_fmaf(w, m.ny, t[5]);
        } else {
            float d, sp;
            lobes(fr, m.nx, m.ny, m.rough, d, sp);
            wd *= d;
            t[3] = __builtin_fmaf(w, sp, t[3]);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) t[c] = __builtin_fmaf(wd, m.albedo[c], t[c]);
    };
    const Frame fr = frame_of({r[3], r[4], r[5]}, {r[6], r[7], r[8]});
    if constexpr (!CUBIC) {
        uint2 texel[NT][NT];
#pragma unroll
        for (int a = 0; a < NT; ++a) {
            const uint32_t col = column(clampi(cx + a, W - 1));
#pragma unroll
            for (int b = 0; b < NT; ++b) texel[a][b] = tex[row[b] + col];
        }
        float t[NT][NS];
#pragma unroll
        for (int a = 0; a < NT; ++a) {
#pragma unroll
            for (int j = 0; j < NS; ++j) t[a][j] = 0.0f;
#pragma unroll
            for (int b = 0; b < NT; ++b) add(t[a], texel[a][b], wx[a] * wy[b], fr);
        }
#pragma unroll
        for (int j = 0; j < NS; ++j) sum[j] = t[0][j] + t[1][j];
    } else {
        const int a = threadIdx.x % NT;
        typedef const __attribute__((address_space(1))) uint64_t* GlobalTexels;
        uint64_t texel[NT][NT];
        for_each<NT>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            auto of = [](auto x) { return lane_of<NT, k>(x); };
            const uint64_t base = (uint64_t)(uintptr_t)tex;
            const GlobalTexels tk = (GlobalTexels)((uint64_t)(uint32_t)of((int)(base >> 32)) << 32 | (uint32_t)of((int)base));
            const uint32_t col = column(clampi(of(cx) + a, of(W) - 1));
#pragma unroll
            for (int b = 0; b < NT; ++b) texel[k][b] = tk[(uint32_t)of((int)row[b]) + col];
        });
        float t[NT][NS];
        for_each<NT>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            auto of = [](auto x) { return lane_of<NT, k>(x); };
            float w = of(wx[0]);
#pragma unroll
            for (int j = 1; j < NT; ++j) {
                const float z = of(wx[j]);   // moved by every lane, chosen or not
                w = a == j ? z : w;
            }
#pragma unroll
            for (int j = 0; j < NS; ++j) t[k][j] = 0.0f;
#pragma unroll
            for (int b = 0; b < NT; ++b)
                add(t[k], make_uint2((uint32_t)texel[k][b], (uint32_t)(texel[k][b] >> 32)), w * of(wy[b]), fr);
        });
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            const float v[NT] = {t[0][j], t[1][j], t[2][j], t[3][j]};
            sum[j] = lane_sum_own<NT>(v, a);
        }
    }
    float codes[3] = {sum[0], sum[1], sum[2]}, spec = sum[3];
    if constexpr (AFTER) {
        float d;
        constexpr float inv = (float)(1.0 / window_scale<CUBIC>());
        lobes(fr, sum[4] * inv, sum[5] * inv, sum[3] * inv, d, spec);
#pragma unroll
        for (int c = 0; c < 3; ++c) codes[c] *= d;
    }
    if (!live) return;
    float* o = out + 3 * i;
#pragma unroll
    for (int c = 0; c < 3; ++c)
        __builtin_nontemporal_store(ok ? finish<CUBIC, AFTER>(fr, codes[c], spec) : __builtin_nanf(""), o + c);
}

// One tap, chosen at random, is shaded.
template <bool CUBIC>
__global__ __launch_bounds__(BLOCK) void k_shade_one(Levels L, const float* __restrict__ q, int32_t n,
                                                     uint32_t key, float* __restrict__ out, int32_t* __restrict__ idx)
{
    int32_t i = blockIdx.x * BLOCK + threadIdx.x;
    if (i >= n) return;
    const float* e = q + 9 * (int64_t)i;
    float r[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) r[k] = __builtin_nontemporal_load(e + k);   // streamed in
    // all of the record is asked for here: loads moved behind the wait for the
    // position find its lines evicted (112 us for 4M scattered queries, 97 so)
    __builtin_amdgcn_sched_barrier(0);
    float u = r[0], v = r[1], s = r[2];
    V3 wo = {r[3], r[4], r[5]}, wi = {r[6], r[7], r[8]};
    int l = (int)(s >= 1.41421354f) + (int)(s >= 2.82842708f);
    l = l < L.n - 1 ? l : L.n - 1;
    TexLevel T = l == 0 ? L.lv[0] : (l == 1 ? L.lv[1] : L.lv[2]);
    const uint2* tex = reinterpret_cast<const uint2*>(T.texels);
    float x = u * (float)T.w - 0.5f, y = v * (float)T.h - 0.5f;
    int cx = 0, cy = 0;
    float tx = 0.0f, ty = 0.0f;
    bool ok = cell_of(x, cx, tx) & cell_of(y, cy, ty);
    const uint32_t b = pcg(key ^ (uint32_t)i);
    const uint32_t base = pcg_base(b);
    const float mx = hash_m(pcg_from_base(base, 0u)), my = hash_m(pcg_from_base(base, 1u));
    int sx, sy;
    if constexpr (CUBIC) {
        sx = cx + choose_cubic_m(tx, mx);
        sy = cy + choose_cubic_m(ty, my);
    } else {
        sx = cx + choose_linear_m(tx, mx);
        sy = cy + choose_linear_m(ty, my);
    }
    sx = clampi(sx, T.w - 1);
    sy = clampi(sy, T.h - 1);
    const uint2 texel = tex[material_index(sx, sy, T.w)];
    const Frame fr = frame_of(wo, wi);
    const Texel m = decode_texel(texel);
    float d, sp;
    lobes(fr, m.nx, m.ny, m.rough, d, sp);
    float f[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) f[c] = ok ? finish<false, true>(fr, d * m.albedo[c], sp) : __builtin_nanf("");
    if (idx) {
        idx[3 * (int64_t)i] = ok ? sx : BAD_INDEX;
        idx[3 * (int64_t)i + 1] = ok ? sy : BAD_INDEX;
        idx[3 * (int64_t)i + 2] = ok ? l : BAD_INDEX;
    }
    // results are streamed out (nontemporal stores)
    __builtin_nontemporal_store(f[0], out + 3 * (int64_t)i);
    __builtin_nontemporal_store(f[1], out + 3 * (int64_t)i + 1);
    __builtin_nontemporal_store(f[2], out + 3 * (int64_t)i + 2);
}

// From how many queries on a query a lane is the faster: fewer leave lanes idle
// that a group a query gives work to.  4 x 4 windows before filtering 200,000
// scattered queries: 15.0 us by groups, 15.3 by lanes; a million in a frame of a
// 256^2 material 28.3 and 21.1; 2 x 2 windows 60,000 and 200,000: 2.7 and 2.5,
// 5.8 and 5.0.  After shading, a million: 24.4 and 20.5, but 200,000 in a frame
// 7.6 and 8.0.  (4 x 4 windows after shading: always by groups, 47 and 50.)
template <bool CUBIC>
constexpr int64_t lane_from(bool after_filter)
{
    return !CUBIC && after_filter ? 1 << 16 : 1 << 18;
}

template <bool CUBIC>
hipError_t launch_shade_f(const Levels& L, const float* q, int32_t n, int mode, uint32_t key, float* out,
                          int32_t* idx, hipStream_t s)
{
    const dim3 block(BLOCK);
    if (mode != STF_SHADE_AFTER_FILTER && mode != STF_FILTER_AFTER_SHADE) {
        hipLaunchKernelGGL((k_shade_one<CUBIC>), dim3(shade_blocks(n, 1, BLOCK)), block, 0, s, L, q, n, key, out, idx);
        return hipGetLastError();
    }
    const bool after = mode == STF_SHADE_AFTER_FILTER;
    if (n >= lane_from<CUBIC>(after) && (after || !CUBIC)) {
        const dim3 grid(shade_blocks(n, 1, BLOCK));
        if (after) hipLaunchKernelGGL((k_shade_lane<CUBIC, STF_SHADE_AFTER_FILTER>), grid, block, 0, s, L, q, n, out);
        else if constexpr (!CUBIC)
            hipLaunchKernelGGL((k_shade_lane<false, STF_FILTER_AFTER_SHADE>), grid, block, 0, s, L, q, n, out);
        return hipGetLastError();
    }
    for (int64_t first = 0; first < n; first += SHADE_PART) {
        const int32_t m = (int32_t)shade_part(n, first);
        const dim3 grid(shade_blocks(m, CUBIC ? 4 : 2, BLOCK));
        const float* qp = q + 9 * first;
        float* op = out + 3 * first;
        if (after) hipLaunchKernelGGL((k_shade_taps<CUBIC, STF_SHADE_AFTER_FILTER>), grid, block, 0, s, L, qp, m, op);
        else hipLaunchKernelGGL((k_shade_taps<CUBIC, STF_FILTER_AFTER_SHADE>), grid, block, 0, s, L, qp, m, op);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

hipError_t launch_shade(const stf_texture* mat, const float* q, int32_t n, int filter, int mode, uint32_t key,
                        float* out, int32_t* idx, hipStream_t s)
{
    Levels L;
    L.n = mat->levels < 3 ? mat->levels : 3;
    for (int l = 0; l < 3; ++l) L.lv[l] = mat->level[l < L.n ? l : L.n - 1];
    return filter == STF_CUBIC_BSPLINE ? launch_shade_f<true>(L, q, n, mode, key, out, idx, s)
                                       : launch_shade_f<false>(L, q, n, mode, key, out, idx, s);
}
