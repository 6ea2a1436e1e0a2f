// neural.hip -- a neural texture (latent grid + MLP) trained on the GPU and
// filtered with BF16 MFMA inference.
//
// The paper argues that stochastic filtering makes expensive texel encodings
// viable because a lookup decodes one texel instead of one per filter tap
// (sections Introduction and Background, neural and compressed
// representations).  Here a W x H x 8 texture is represented by an
// LW x LH x 8 latent grid and an MLP 8 -> 64 -> 64 -> 8 (ReLU after the two
// hidden layers): texel (i, j) decodes to MLP(bilerp of the latent grid at
// X = (i + 1/2) LW/W - 1/2, clamped corners).  Filtering decodes every tap
// (deterministic) or the one sampled tap (stochastic), with the tap rules of
// the 2D filters.
//
// Training (binary32): per step a batch of texel positions, forward and
// backward through the MLP and the bilinear interpolation, mean squared
// error against the target texels, Adam.  One kernel processes tiles of 32
// samples on the binary32 matrix cores and sums weight gradients per block; a
// second one sums the blocks in a fixed order and makes the Adam steps; latent
// gradients are scattered with atomics.
//
// Inference: latents rounded to binary16, weights to bfloat16, biases kept in
// binary32.  Each wave decodes 32 texels per MFMA batch with
// v_mfma_f32_32x32x16_bf16 in the transposed form out^T = W in^T, so each
// layer's accumulator registers are already the next layer's B operand once
// the hidden units are stored in the order the accumulator layout produces.
// A wave runs two batches at a time: each of its 64 lanes does the tap
// choice, latent gather and interpolation of one of the 64 decodes, and a
// lane-half swap forms both batches' first B operands.  The 8 output channels
// use products of 16 columns.
#include <math.h>
#include <string.h>

#include <vector>

#include "device_common.h"
#include "stf_internal.h"

using namespace stf;

namespace {

constexpr int NL = 8, NH = 64, NO = 8;
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + NH * NL, OFF_W2 = OFF_B1 + NH, OFF_B2 = OFF_W2 + NH * NH,
              OFF_W3 = OFF_B2 + NH, OFF_B3 = OFF_W3 + NO * NH, NPARAM = OFF_B3 + NO;
constexpr int PSTRIDE = NPARAM + 1;   // per-block partial gradients + loss
constexpr int TS = 32;                 // samples per training tile
constexpr int TBLOCK = 512;
constexpr int TRAIN_BLOCKS = 512;      // one resident set: two blocks per CU
static_assert(NL == 8 && NO == 8 && NH == 64, "the training kernel's operand layouts");

struct TrainArgs {
    const float* lat;
    const float* mlp;
    const float* target;
    const int32_t* pos;   // nullable: positions drawn from the counter hash
    int32_t B, W, H, LW, LH;
    float rx, ry;         // LW / W, LH / H (powers of two)
    uint32_t kstep;
    float dscale;         // 2 / (8 B)
    float* g_lat;
    float* partial;
};

__device__ __forceinline__ int clampi(int v, int hi)
{
    return v < 0 ? 0 : (v > hi ? hi : v);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Row 4g + r of a 16-row operand block holds unit 4r + g of the block: the
// accumulator registers r of the lanes (g, n) are then the k-steps of the next
// product in unit order (step r, k-slot g: unit 4r + g).
__host__ __device__ constexpr int unit_of_row(int row)
{
    return 4 * (row % 4) + row / 4;
}

// Where the row of sample s begins in a [32][64] matrix in LDS: 16 (s % 4) +
// 4 (s / 4 % 4) banks on, so that the 16-byte accesses of 16 samples at one
// column and the 4-byte accesses of 16 columns of 4 successive samples both
// meet every bank once.
__host__ __device__ constexpr int train_row(int s)
{
    return s / 16 * 1280 + s / 4 % 4 * 324 + s % 4 * 80;
}
constexpr int TMAT = train_row(TS);

constexpr int ZSTRIDE = 16;
struct TrainShared {
    // [sample][row of the unit] (train_row); D1 takes the place of H2
    float h1[TMAT], h2d1[TMAT], d2[TMAT];
    float z[2][TS * ZSTRIDE];   // [sample][2g + t: channel 4t + g]; column 8 is 1, 9..15 are 0
    float y[TS * ZSTRIDE];      // the output's gradient, later the latents', columns as in z; 8..15 are 0
    float t[TS * NO];           // target, columns as in z; at the end the loss of either half
    float b1[NH], b2[NH], b3[16];   // biases by row
    f32x4 w2[16][64], w2t[16][64], w3[4][64], w1t[4][64];   // A operand images: [4 mb + kb or kb][lane], k-steps r
};
static_assert(sizeof(TrainShared) <= 80 * 1024, "two blocks per CU");

// What thread (sample s, channel k) of a tile reads from memory: the first 256
// threads the latent corners, the others the target.
struct TrainGather {
    float v0, v1, v2, v3;
    float w0, w1, w2, w3;
    uint32_t o0, o1, o2, o3;   // byte offsets of the corners' channel (a latent grid is below 4 GiB)
    bool live;
};

__device__ __forceinline__ TrainGather train_gather(const TrainArgs& a, int32_t tile, int s, int k, bool latents)
{
    TrainGather r = {};
    const int64_t gs = (int64_t)tile * TS + s;
    r.live = gs < a.B;
    int i = 0, j = 0;
    if (r.live) {
        // h mod size without a division where the size is a power of two
        auto mod = [](uint32_t h, uint32_t size) { return (int)((size & (size - 1)) ? h % size : h & (size - 1)); };
        if (a.pos) {   // caller-supplied positions are clamped into the texture
            i = clampi(a.pos[2 * gs], a.W - 1);
            j = clampi(a.pos[2 * gs + 1], a.H - 1);
        } else {
            const uint32_t h = pcg(a.kstep ^ (uint32_t)gs);
            i = mod(h, (uint32_t)a.W);
            j = mod(pcg(h + 1u), (uint32_t)a.H);
        }
    }
    if (!latents) {
        r.v0 = a.target[((int64_t)j * a.W + i) * NO + k];
        return r;
    }
    const float X = ((float)i + 0.5f) * a.rx - 0.5f, Y = ((float)j + 0.5f) * a.ry - 0.5f;
    const float fx0 = floorf(X), fy0 = floorf(Y);
    const float fx = X - fx0, fy = Y - fy0;
    const int x0 = (int)fx0, y0 = (int)fy0;
    const int xa = clampi(x0, a.LW - 1), xb = clampi(x0 + 1, a.LW - 1);
    const int ya = clampi(y0, a.LH - 1), yb = clampi(y0 + 1, a.LH - 1);
    auto corner = [&](int x, int y) { return (uint32_t)(y * a.LW + x) * (NL * 4u) + 4u * (uint32_t)k; };
    r.o0 = corner(xa, ya);
    r.o1 = corner(xb, ya);
    r.o2 = corner(xa, yb);
    r.o3 = corner(xb, yb);
    r.w0 = (1.0f - fx) * (1.0f - fy);
    r.w1 = fx * (1.0f - fy);
    r.w2 = (1.0f - fx) * fy;
    r.w3 = fx * fy;
    auto load = [&](uint32_t o) {
        return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(a.lat) + (size_t)o);
    };
    r.v0 = load(r.o0);
    r.v1 = load(r.o1);
    r.v2 = load(r.o2);
    r.v3 = load(r.o3);
    return r;
}

// Adds a tile's latent gradient (sample s, channel k) to the four corners.
__device__ __forceinline__ void train_scatter(const TrainArgs& a, const TrainGather& r, float dz)
{
    if (!r.live) return;
    auto add = [&](uint32_t o, float v) {
        atomicAdd(reinterpret_cast<float*>(reinterpret_cast<char*>(a.g_lat) + (size_t)o), v);
    };
    add(r.o0, r.w0 * dz);
    add(r.o1, r.w1 * dz);
    add(r.o2, r.w2 * dz);
    add(r.o3, r.w3 * dz);
}

// A chain of 16 matrix instructions: acc + A B over 64 k-slots, A from an
// operand image, B from the lane's sample's row in LDS (from its column 4g).
// Two blocks of operands in flight, held back by the scheduling barriers.
__device__ __forceinline__ f32x4 train_chain(const f32x4 (*A)[64], const float* B, int lane, f32x4 acc)
{
    f32x4 w[2], x[2];
    w[0] = A[0][lane];
    x[0] = *reinterpret_cast<const f32x4*>(B);
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
        if (kb < 3) {
            w[(kb + 1) % 2] = A[kb + 1][lane];
            x[(kb + 1) % 2] = *reinterpret_cast<const f32x4*>(B + 16 * (kb + 1));
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[kb % 2][r], x[kb % 2][r], acc, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
    return acc;
}

__device__ __forceinline__ f32x4 relu4(f32x4 v)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.0f);
    return v;
}

__device__ __forceinline__ f32x4 mask4(f32x4 v, const f32x4& h)   // v where h > 0
{
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = h[r] > 0.0f ? v[r] : 0.0f;
    return v;
}

// Forward and backward pass over tiles of 32 samples, eight waves per tile,
// every product on the binary32 matrix cores (v_mfma_f32_16x16x4_f32): wave
// (mb, nh) makes units 16 mb .. 16 mb + 15 of samples 16 nh .. 16 nh + 15 of
// each layer, and its share of the weight gradients.
//
// Activations are products [unit][sample]: lane (g, n) = (lane / 16, lane % 16)
// holds four units of sample 16 nh + n.  The waves exchange them through LDS,
// where a lane reads its sample's row as the next product's B operand; rows are
// numbered (unit_of_row) so that the k-slots of successive steps run through
// the units in order.  A matrix instruction adds its four products one after
// the other, each rounded once like an FMA, so every activation and every
// gradient has the bits of the plain FMA loops over units and samples.  The 8
// channels of the latents and of the output occupy rows 4g + {0, 1} (channels
// g and 4 + g).  A weight gradient sums over samples: its operands are read
// from the same LDS matrices with the sample in the k-slot, 4 bytes a lane,
// and each tile's sum, formed from zero, is added to the wave's registers.
//
// 576 matrix instructions of 32 cycles per tile would take 61 us for 262,144
// samples on 1,024 SIMDs; the chain of six barriers per tile, each with an
// LDS round trip and a dependent chain, holds the pass at 107 us.  Four waves
// per SIMD from two blocks per CU fill each other's gaps, and a tile's gathers
// are issued a tile ahead.  The products that not all waves share (the output,
// the latents' gradient, dW3) go to one wave per SIMD: with both halves of a
// product on one SIMD the pass took 124 us.  Left alone, the later block of a
// CU falls behind by a third per tile and ends alone; with the raised priority
// it falls behind by a fifth, as two blocks of evenly placed products do, so
// that the latents' atomics meet in nearly the same order from one arrangement
// to another (2.4% of the sums differ in their rounding, as between two runs;
// 3.6% without).  The same products as register-blocked FMAs from LDS took 220
// us.
__global__ __launch_bounds__(TBLOCK, 4) void k_ntex_train(TrainArgs a)
{
    __shared__ __align__(16) char smem[sizeof(TrainShared)];
    TrainShared& S = *reinterpret_cast<TrainShared*>(smem);
    const int t = threadIdx.x, lane = t % 64, wave = t / 64, n = lane % 16, g = lane / 16;
    const int mb = wave % 4, nh = wave / 4;
    // Two waves share a SIMD (waves 4 apart).  What only some waves do is given
    // to one wave per SIMD: the output of either sample half (SIMDs 0, 1), the
    // latents' gradient of either half (2, 3), a unit block of dW3 (all four).
    const bool makes_y = mb == nh, makes_dz = mb == 2 + nh, makes_w3 = !makes_y && !makes_dz;
    {   // Operand images: every weight is loaded once and put where its images
        // hold it -- lane l of an A operand holds row l % 16, k-slot l / 16.
        float* w2 = reinterpret_cast<float*>(S.w2);
        float* w2t = reinterpret_cast<float*>(S.w2t);
        float* w3 = reinterpret_cast<float*>(S.w3);
        float* w1t = reinterpret_cast<float*>(S.w1t);
        constexpr int PER = NH * NH / TBLOCK;   // 8 entries of a W2 row
        const f32x4 wa = *reinterpret_cast<const f32x4*>(a.mlp + OFF_W2 + PER * t),
                    wb = *reinterpret_cast<const f32x4*>(a.mlp + OFF_W2 + PER * t + 4);
        const float v1 = a.mlp[OFF_W1 + t], v3 = a.mlp[OFF_W3 + t];   // 512 of each
        auto place = [](int row, int k) { return (k / 16 * 64 + k % 4 * 16 + row) * 4 + k % 16 / 4; };
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const float v = e < 4 ? wa[e % 4] : wb[e % 4];
            const int m = PER * t / NH, k = PER * t % NH + e;
            w2[m / 16 * 1024 + place(unit_of_row(m % 16), k)] = v;
            w2t[k / 16 * 1024 + place(unit_of_row(k % 16), m)] = v;
        }
        w3[place(unit_of_row(t / NH), t % NH)] = v3;    // channel c in row unit_of_row(c), a row of two in four
        w1t[place(unit_of_row(t % NL), t / NL)] = v1;
        for (int e = t; e < 4 * 64 * 4; e += TBLOCK)
            if (e / 4 % 4 >= 2) w3[e] = w1t[e] = 0.0f;   // rows 4g + {2, 3} are padding
        for (int e = t; e < TS * (ZSTRIDE - 8); e += TBLOCK) {
            const int at = e / (ZSTRIDE - 8) * ZSTRIDE + 8 + e % (ZSTRIDE - 8);
            S.z[0][at] = S.z[1][at] = e % (ZSTRIDE - 8) == 0 ? 1.0f : 0.0f;
            S.y[at] = 0.0f;
        }
    }
    // this wave's smaller operands, in registers
    float w1[2], w3t[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int u = 16 * mb + unit_of_row(n), c = 4 * r + g;
        w1[r] = a.mlp[OFF_W1 + u * NL + c];
        w3t[r] = a.mlp[OFF_W3 + c * NH + u];
    }
    if (t < NH) {
        S.b1[t] = a.mlp[OFF_B1 + t / 16 * 16 + unit_of_row(t % 16)];
        S.b2[t] = a.mlp[OFF_B2 + t / 16 * 16 + unit_of_row(t % 16)];
    }
    if (t < 16) S.b3[t] = t % 4 < 2 ? a.mlp[OFF_B3 + unit_of_row(t)] : 0.0f;
    // LDS places: column 4g of the lane's sample (16-byte accesses), column n
    // of sample g, whose successors 4 j + g are constants further on (4-byte
    // accesses of the weight gradients)
    const int smp = 16 * nh + n, row0 = train_row(smp) + 4 * g, col0 = train_row(g) + n;
    // gradients over the block's tiles: dW2 rows of block mb, columns of
    // blocks 2 nh and 2 nh + 1; dW1 and db1 (nh = 0: column 8) or db2 (nh = 1:
    // column 8); dW3 of unit block mb (makes_w3); db3 (wave 0)
    f32x4 g20 = (f32x4)0.0f, g21 = g20, g1 = g20, g3 = g20;
    float gb3 = 0.0f, lacc = 0.0f;
    const int s8 = t % 256 / 8, k8 = t % 8, c8 = 2 * (k8 % 4) + k8 / 4;
    const bool latents = t < 256;
    const int32_t ntiles = (a.B - 1) / TS + 1;
    TrainGather cur = train_gather(a, blockIdx.x, s8, k8, latents), prev = {};
    int buf = 0;
    for (int32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        if (latents) {
            float z = 0.0f;
            z = __builtin_fmaf(cur.w0, cur.v0, z);
            z = __builtin_fmaf(cur.w1, cur.v1, z);
            z = __builtin_fmaf(cur.w2, cur.v2, z);
            z = __builtin_fmaf(cur.w3, cur.v3, z);
            S.z[buf][s8 * ZSTRIDE + c8] = cur.live ? z : 0.0f;
        } else {
            S.t[s8 * NO + c8] = cur.v0;
        }
        // the later one of a CU's two blocks, whose waves are served after the
        // earlier one's, goes first in every fourth tile (see above)
        __builtin_amdgcn_s_setprio(0);
        if (blockIdx.x >= TRAIN_BLOCKS / 2 && tile / TRAIN_BLOCKS % 4 == 0) __builtin_amdgcn_s_setprio(1);
        __syncthreads();   // z, t; the previous tile is done with the matrices
        if (latents) train_scatter(a, prev, S.y[s8 * ZSTRIDE + c8]);
        prev = cur;
        const int64_t next = (int64_t)tile + gridDim.x;
        cur = train_gather(a, next < ntiles ? (int32_t)next : tile, s8, k8, latents);
        const bool live = (int64_t)tile * TS + smp < a.B;
        // H1 = relu(W1 Z + b1)
        const float2 z = *reinterpret_cast<const float2*>(&S.z[buf][smp * ZSTRIDE + 2 * g]);
        const int own = row0 + 16 * mb;
        f32x4 h1 = *reinterpret_cast<const f32x4*>(&S.b1[16 * mb + 4 * g]);
        h1 = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[0], z.x, h1, 0, 0, 0);
        h1 = relu4(__builtin_amdgcn_mfma_f32_16x16x4f32(w1[1], z.y, h1, 0, 0, 0));
        *reinterpret_cast<f32x4*>(&S.h1[own]) = h1;
        __syncthreads();
        // H2 = relu(W2 H1 + b2)
        f32x4 h2 = *reinterpret_cast<const f32x4*>(&S.b2[16 * mb + 4 * g]);
        h2 = relu4(train_chain(&S.w2[4 * mb], S.h1 + row0, lane, h2));
        *reinterpret_cast<f32x4*>(&S.h2d1[own]) = h2;
        __syncthreads();
        if (makes_y) {   // Y = W3 H2 + b3, the loss and its gradient
            const f32x4 y = train_chain(S.w3, S.h2d1 + row0, lane, *reinterpret_cast<const f32x4*>(&S.b3[4 * g]));
            const float2 target = *reinterpret_cast<const float2*>(&S.t[smp * NO + 2 * g]);
            const float e0 = y[0] - target.x, e1 = y[1] - target.y;
            if (live) lacc = __builtin_fmaf(e1, e1, __builtin_fmaf(e0, e0, lacc));
            *reinterpret_cast<float2*>(&S.y[smp * ZSTRIDE + 2 * g]) =
                make_float2(live ? e0 * a.dscale : 0.0f, live ? e1 * a.dscale : 0.0f);
        }
        __syncthreads();
        {   // D2 = (W3^T dY) * [H2 > 0]
            const float2 dy = *reinterpret_cast<const float2*>(&S.y[smp * ZSTRIDE + 2 * g]);
            f32x4 d2 = __builtin_amdgcn_mfma_f32_16x16x4f32(w3t[0], dy.x, (f32x4)0.0f, 0, 0, 0);
            d2 = __builtin_amdgcn_mfma_f32_16x16x4f32(w3t[1], dy.y, d2, 0, 0, 0);
            *reinterpret_cast<f32x4*>(&S.d2[own]) = mask4(d2, h2);
        }
        if (makes_w3) {   // dW3^T += H2 dY^T
            const float* u = S.h2d1 + col0 + 16 * mb;
            f32x4 s0 = (f32x4)0.0f;
#pragma unroll
            for (int j = 0; j < TS / 4; ++j)
                s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(u[train_row(4 * j)], S.y[(4 * j + g) * ZSTRIDE + n], s0, 0, 0, 0);
            g3 += s0;
        } else if (wave == 0) {   // db3 += dY 1, a lane per column
            float s1 = 0.0f;
#pragma unroll
            for (int k = 0; k < TS; ++k) s1 += S.y[k * ZSTRIDE + n];
            gb3 += s1;
        }
        __syncthreads();
        // D1 = (W2^T D2) * [H1 > 0]
        *reinterpret_cast<f32x4*>(&S.h2d1[own]) =
            mask4(train_chain(&S.w2t[4 * mb], S.d2 + row0, lane, (f32x4)0.0f), h1);
        {   // dW2 += D2 H1^T over the samples
            const float *u = S.d2 + col0 + 16 * mb, *x = S.h1 + col0 + 32 * nh;
            f32x4 s0 = (f32x4)0.0f, s1 = (f32x4)0.0f;
#pragma unroll
            for (int j = 0; j < TS / 4; ++j) {
                const float d = u[train_row(4 * j)];
                s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(d, x[train_row(4 * j)], s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(d, x[train_row(4 * j) + 16], s1, 0, 0, 0);
            }
            g20 += s0;
            g21 += s1;
        }
        __syncthreads();
        if (makes_dz) {   // dZ = W1^T D1, scattered by the next tile's gather threads
            const f32x4 dz = train_chain(S.w1t, S.h2d1 + row0, lane, (f32x4)0.0f);
            *reinterpret_cast<float2*>(&S.y[smp * ZSTRIDE + 2 * g]) = make_float2(dz[0], dz[1]);
        }
        {   // dW1 += D1 Z^T and db1 += D1 1, or db2 += D2 1 (column 8)
            const float* u = (nh ? S.d2 : S.h2d1) + col0 + 16 * mb;
            f32x4 s0 = (f32x4)0.0f;
#pragma unroll
            for (int j = 0; j < TS / 4; ++j)
                s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(u[train_row(4 * j)], S.z[buf][(4 * j + g) * ZSTRIDE + n], s0, 0,
                                                          0, 0);
            g1 += s0;
        }
        buf ^= 1;
    }
    __syncthreads();
    if (latents) train_scatter(a, prev, S.y[s8 * ZSTRIDE + c8]);
    // row 4g + r of a product is unit 4r + g of its block, column n unit unit_of_row(n)
    float* out = a.partial + (int64_t)blockIdx.x * PSTRIDE;
    const int col = unit_of_row(n), ch = 4 * (n % 2) + n / 2;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int u = 16 * mb + 4 * r + g;
        out[OFF_W2 + u * NH + 32 * nh + col] = g20[r];
        out[OFF_W2 + u * NH + 32 * nh + 16 + col] = g21[r];
        if (nh == 0 && n < NL) out[OFF_W1 + u * NL + ch] = g1[r];
        if (n == 8) out[(nh ? OFF_B2 : OFF_B1) + u] = g1[r];
        if (makes_w3 && n < NL) out[OFF_W3 + ch * NH + u] = g3[r];
    }
    if (wave == 0 && lane < NO) out[OFF_B3 + ch] = gb3;
    if (makes_y) {
        for (int off = 32; off > 0; off >>= 1) lacc += __shfl_xor(lacc, off);
        if (lane == 0) S.t[nh] = lacc;
    }
    __syncthreads();
    if (t == 0) out[NPARAM] = S.t[0] + S.t[1];
}

// One Adam step of a value (beta1 = 0.9, beta2 = 0.999, eps = 1e-8, c1 and c2
// the bias corrections).
__device__ __forceinline__ void adam(float& p, float g, float& m, float& v, float lr, float c1, float c2)
{
    m = 0.9f * m + 0.1f * g;
    v = 0.999f * v + 0.001f * g * g;
    p -= lr * (m * c1) / (sqrtf(v * c2) + 1e-8f);
}

struct UpdateArgs {
    const float* partial;   // nblocks rows of PSTRIDE
    int32_t nblocks;
    float* g_mlp;           // written when the MLP is not stepped (mlp null)
    float *mlp, *m_mlp, *v_mlp;
    float *lat, *g_lat, *m_lat, *v_lat;   // nlat4 groups of four
    int32_t nlat4;
    float* loss;            // nullable
    float loss_scale, lr_mlp, lr_lat, c1, c2;
};

// After a pass, in one launch: the first UPDATE_MLP blocks sum the pass's
// per-block partials (64 values each; groups of RGROUP rows in row order, one
// group after another per wave, then the groups in order, so reproducible)
// and step the MLP with the result, the others step the latents, clearing the
// gradient they consumed.  Bound by memory (32 bytes moved per latent); two
// sums and two steps took four launches and 32 us a step, of which this takes
// 12 (512^2 latents).
//
// STREAMED: the moments go past the caches, for latents whose four arrays the
// 256 MB behind the L2s cannot hold from step to step (2048^2: 204 us a step of
// 16 samples in two launches, 210 in one, 140 so; 512^2, which they hold: 16.7
// and 18.4).
constexpr int64_t STREAM_FROM = (int64_t)1 << 24;   // latent values, 16 bytes each
constexpr int RGROUP = 32;
constexpr int UBLOCK = 512, UWAVES = UBLOCK / 64;
constexpr int UPDATE_MLP = (PSTRIDE + 63) / 64;

template <bool STREAMED>
__global__ __launch_bounds__(UBLOCK) void k_ntex_update(UpdateArgs a)
{
    if (blockIdx.x >= UPDATE_MLP) {
        const int32_t e = (int32_t)(blockIdx.x - UPDATE_MLP) * UBLOCK + (int32_t)threadIdx.x;
        if (e >= a.nlat4) return;
        f32x4 *pm = reinterpret_cast<f32x4*>(a.m_lat) + e, *pv = reinterpret_cast<f32x4*>(a.v_lat) + e;
        f32x4 p = reinterpret_cast<f32x4*>(a.lat)[e], m = STREAMED ? __builtin_nontemporal_load(pm) : *pm,
              v = STREAMED ? __builtin_nontemporal_load(pv) : *pv;
        const f32x4 g = reinterpret_cast<f32x4*>(a.g_lat)[e];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float pk = p[k], mk = m[k], vk = v[k];
            adam(pk, g[k], mk, vk, a.lr_lat, a.c1, a.c2);
            p[k] = pk;
            m[k] = mk;
            v[k] = vk;
        }
        reinterpret_cast<f32x4*>(a.lat)[e] = p;
        if constexpr (STREAMED) {
            __builtin_nontemporal_store(m, pm);
            __builtin_nontemporal_store(v, pv);
        } else {
            *pm = m;
            *pv = v;
        }
        reinterpret_cast<f32x4*>(a.g_lat)[e] = (f32x4)0.0f;
        return;
    }
    __shared__ float sums[TRAIN_BLOCKS / RGROUP][64];
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int p = (int)blockIdx.x * 64 + lane, ngroups = (a.nblocks + RGROUP - 1) / RGROUP;
    for (int k = wave; k < ngroups; k += UWAVES) {
        float s = 0.0f;
        const int b1 = min(a.nblocks, (k + 1) * RGROUP);
        if (p < PSTRIDE) {
#pragma unroll 16
            for (int b = k * RGROUP; b < b1; ++b) s += a.partial[(int64_t)b * PSTRIDE + p];
        }
        sums[k][lane] = s;
    }
    __syncthreads();
    if (wave != 0 || p >= PSTRIDE) return;
    float s = 0.0f;
    for (int k = 0; k < ngroups; ++k) s += sums[k][lane];
    if (p == NPARAM) {
        if (a.loss) *a.loss = s * a.loss_scale;
    } else if (a.mlp) {
        float pk = a.mlp[p], mk = a.m_mlp[p], vk = a.v_mlp[p];
        adam(pk, s, mk, vk, a.lr_mlp, a.c1, a.c2);
        a.mlp[p] = pk;
        a.m_mlp[p] = mk;
        a.v_mlp[p] = vk;
    } else {
        a.g_mlp[p] = s;
    }
}

__global__ void k_fill(float* __restrict__ p, int64_t n, float v)
{
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) p[e] = v;
}

// Corner quads for inference: entry (y0 + 1, x0 + 1) for every cell
// x0 = -1 .. LW - 1, y0 = -1 .. LH - 1 holds the binary16 latents of its
// clamped corners (x0, y0), (x0 + 1, y0), (x0, y0 + 1), (x0 + 1, y0 + 1), so a
// decode reads one 64-byte quad instead of two rows of the grid.
__global__ void k_to_quads(const float* __restrict__ lat, uint16_t* __restrict__ quad, int32_t LW, int32_t LH)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)(LW + 1) * (LH + 1)) return;
    const int x0 = (int)(e % (LW + 1)) - 1, y0 = (int)(e / (LW + 1)) - 1;
    const int xs[2] = {clampi(x0, LW - 1), clampi(x0 + 1, LW - 1)};
    const int ys[2] = {clampi(y0, LH - 1), clampi(y0 + 1, LH - 1)};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float* src = lat + ((int64_t)ys[k / 2] * LW + xs[k % 2]) * NL;
        uint16_t h[NL];
#pragma unroll
        for (int c = 0; c < NL; ++c) h[c] = __builtin_bit_cast(uint16_t, (_Float16)src[c]);
        reinterpret_cast<uint4*>(quad)[4 * e + k] = __builtin_bit_cast(uint4, h);
    }
}

// ---------------------------------------------------------------------------
// inference
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Operand images: one 8-value A slot per lane for every MFMA.  Layer 1's
// biases enter in its padding slots: each is split exactly into three bf16
// terms held in k-slots 8..10 of the A operand, which meet ones in the same
// slots of the B operand.  Layers 2 and 3 start their accumulation from the
// biases themselves, held in the accumulator's layout.
struct Packed {
    bf16x8 a1[2][64];      // layer 1, M-blocks of 32 hidden units; k 0..7 latent, 8..10 bias terms
    bf16x8 a2[2][4][64];   // layer 2, M-blocks x K-blocks of 16
    bf16x8 a3[2][64];      // layer 3, K-blocks of 32; rows 0..7 the channels, 8..15 the same again
    f32x16 b2[2][2];       // layer 2 biases per lane half and M-block
    f32x4 b3[2];           // layer 3 biases of channels 0..3 and 4..7
};

// Hidden unit held by k-slot kappa = 16 kb + 8 h + j of the B operand when
// the previous layer's accumulator registers are used in place.
__host__ __device__ constexpr int hidden_of_slot(int kb, int h, int j)
{
    return 16 * kb + 8 * (j / 4) + 4 * h + (j % 4);
}

// Hidden/output unit held by accumulator register r of lane half h in M-block mb.
__host__ __device__ constexpr int row_of_acc(int mb, int h, int r)
{
    return 32 * mb + 8 * (r / 4) + 4 * h + (r % 4);
}

// Hidden unit met by slot j of lane group g (of 16 lanes) in layer 3's K-block
// kb2 of 32: layer_3 swaps the odd groups of the even K-block of 16 with the
// even groups of the odd one.
__host__ __device__ constexpr int hidden_of_slot3(int kb2, int g, int j)
{
    return hidden_of_slot(2 * kb2 + g % 2, g / 2, j);
}

struct InferArgs {
    const Packed* pk;
    const uint16_t* quad16;   // (LH + 1) x (LW + 1) corner quads, 4 x 8 binary16 each
    const float* q;          // n x 2 uv
    int32_t n, W, H, LW, LH;
    float rx, ry;
    uint32_t key;
    float* out;              // n x 8
    int32_t* idx;            // n x 2 (stochastic) or null
};

typedef short i16x8 __attribute__((ext_vector_type(8)));
typedef short i16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// ReLU after rounding to bf16, done on the bit patterns: a bf16 whose sign
// bit is set reads as a negative int16, so a signed 16-bit max with zero maps
// it (and -0) to +0 and leaves every other value as it is.  Rounding keeps
// the sign, so this equals rounding the ReLU of the fp32 value.
__device__ __forceinline__ bf16x8 relu_bf16(const f32x16& d, int base)
{
    i16x8 v;
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
        i16x2 p = __builtin_bit_cast(i16x2, __builtin_convertvector((f32x2){d[base + j], d[base + j + 1]}, bf16x2));
        p = __builtin_elementwise_max(p, (i16x2)0);
        v[j] = p[0];
        v[j + 1] = p[1];
    }
    return __builtin_bit_cast(bf16x8, v);
}

// One lane's decode: the tap it stands for, the texel it decodes and the
// tap's filter weight.
struct Decode {
    int sx, sy;
    float w;
    bool fin;
};

// Six times the weight of one cubic B-spline tap, as cubic6 computes it: tap
// is fixed per lane, so its cases are selects on lane masks.
__device__ __forceinline__ float cubic6_tap(int tap, float t)
{
    const bool inner = tap == 1 || tap == 2;
    const float s = 1.0f - t, u = tap < 2 ? s : t;
    const float p = (inner ? 3.0f : u) * u, q = inner ? 1.0f + s * t : u;
    return (inner ? 1.0f : 0.0f) + p * q;
}

template <bool CUBIC, bool STOCH>
__device__ __forceinline__ Decode locate(const InferArgs& a, uint32_t qi, int tap, float2 uv)
{
    Decode d;
    float x = uv.x * (float)a.W - 0.5f, y = uv.y * (float)a.H - 0.5f;
    int cx = 0, cy = 0;
    float tx = 0.0f, ty = 0.0f;
    d.fin = (__builtin_fabsf(x) < TWO24) & (__builtin_fabsf(y) < TWO24);
    (void)cell_of(d.fin ? x : 0.0f, cx, tx);
    (void)cell_of(d.fin ? y : 0.0f, cy, ty);
    d.w = 1.0f;
    if constexpr (STOCH) {
        const uint32_t base = pcg_base(pcg(a.key ^ qi));
        const float mx = hash_m(pcg_from_base(base, 0u)), my = hash_m(pcg_from_base(base, 1u));
        if constexpr (CUBIC) {
            d.sx = cx + choose_cubic_m(tx, mx);
            d.sy = cy + choose_cubic_m(ty, my);
        } else {
            d.sx = cx + choose_linear_m(tx, mx);
            d.sy = cy + choose_linear_m(ty, my);
        }
    } else {
        int ta = tap % 2, tb = tap / 2;
        d.w = (ta ? tx : 1.0f - tx) * (tb ? ty : 1.0f - ty);
        d.sx = cx + ta;
        d.sy = cy + tb;
    }
    d.sx = clampi(d.sx, a.W - 1);
    d.sy = clampi(d.sy, a.H - 1);
    return d;
}

// The latent cell of texel s on one axis (ratio = L / size): the index of its
// lower corner plus one, and the fraction.  With L <= size the corner
// floor(X) lies in -1 .. L - 1.
__device__ __forceinline__ int latent_cell(int s, float ratio, int L, float& f)
{
    const float X = ((float)s + 0.5f) * ratio - 0.5f, x0 = floorf(X);
    f = X - x0;
    return min(max((int)x0, -1), L - 1) + 1;
}

// The corner quad of latent cell (i, j) (its four clamped latent corners,
// 64 contiguous bytes: one cache line) and their bilinear weights.
__device__ __forceinline__ uint32_t latent_quad(const InferArgs& a, int i, int j, float fx, float fy, float (&w)[4])
{
    w[0] = (1.0f - fx) * (1.0f - fy);
    w[1] = fx * (1.0f - fy);
    w[2] = (1.0f - fx) * fy;
    w[3] = fx * fy;
    return __umul24((uint32_t)j, (uint32_t)(a.LW + 1)) + (uint32_t)i;   // sides to 65537, below 2^27 quads
}

// One axis of a cubic tap: its weight (NaN for a non-finite coordinate) and
// the latent cell and fraction of its texel.
struct AxisTap {
    float w, f;
    int i;
};

__device__ __forceinline__ AxisTap locate_axis(float u, int size, int L, float ratio, int tap)
{
    const float x = u * (float)size - 0.5f;
    const bool fin = __builtin_fabsf(x) < TWO24;
    int c = 0;
    float t = 0.0f;
    (void)cell_of(fin ? x : 0.0f, c, t);
    AxisTap d;
    d.w = fin ? cubic6_tap(tap, t) * K6 : __builtin_nanf("");
    d.i = latent_cell(clampi(c - 1 + tap, size - 1), ratio, L, d.f);
    return d;
}

// Layer 3 on a 32-decode batch: the 8 output rows would fill a quarter of a
// 32 x 32 product, so the decodes are split into two blocks of 16 columns
// instead (half the matrix cycles).  Swapping the odd rows of 16 lanes of one
// hidden K-block with the even rows of the next turns two B operands of the
// 32-column layout into one of each block.  The weights' rows 8..15 repeat the
// channels, so that lane groups 0, 1 take the first block's results and groups
// 2, 3 the second's: lane l ends with channels 4 (l / 16 % 2) .. + 3 of decode
// 16 (l / 32) + l % 16.
__device__ __forceinline__ f32x4 layer_3(const bf16x8 (&B3)[4], const bf16x8 (&A3)[2], const f32x4& C3, bool upper)
{
    f32x4 D[2] = {C3, C3};
#pragma unroll
    for (int kb2 = 0; kb2 < 2; ++kb2) {
        const uint4 x = __builtin_bit_cast(uint4, B3[2 * kb2]), y = __builtin_bit_cast(uint4, B3[2 * kb2 + 1]);
        const auto r0 = __builtin_amdgcn_permlane16_swap(x.x, y.x, false, false);
        const auto r1 = __builtin_amdgcn_permlane16_swap(x.y, y.y, false, false);
        const auto r2 = __builtin_amdgcn_permlane16_swap(x.z, y.z, false, false);
        const auto r3 = __builtin_amdgcn_permlane16_swap(x.w, y.w, false, false);
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            const bf16x8 B = __builtin_bit_cast(bf16x8, make_uint4(r0[nb], r1[nb], r2[nb], r3[nb]));
            D[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A3[kb2], B, D[nb], 0, 0, 0);
        }
    }
    f32x4 o;
#pragma unroll
    for (int c = 0; c < 4; ++c) o[c] = upper ? D[1][c] : D[0][c];
    return o;
}

// The decoder MLP on one 32-decode batch: B1 holds the bf16 latents of the
// batch's decodes in k-slots 0..7 (lanes 0..31) and ones in the bias slots
// 8..10 (lanes 32..63).  Returns four channels of one decode per lane (see
// layer_3).
__device__ __forceinline__ f32x4 mlp_batch(const bf16x8& B1, const bf16x8 (&A1)[2], const bf16x8 (&A2)[2][4],
                                           const bf16x8 (&A3)[2], const f32x16* C2, const f32x4& C3, bool upper)
{
    const f32x16 Z = {};
    // A wave in its matrix chain runs at raised issue priority, so the
    // SIMD's other waves fill the gaps with their VALU work (latent
    // interpolation, ReLU conversions, tap sums) instead of contending with
    // it; the chain itself is one dependent sequence per layer.
    __builtin_amdgcn_s_setprio(1);
    // layer 1: 64 x 16 by 16 x 32 (k 0..7 latents, 8..10 bias terms)
    f32x16 D1[2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) D1[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A1[mb], B1, Z, 0, 0, 0);
    bf16x8 B2[4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) B2[kb] = relu_bf16(D1[kb / 2], 8 * (kb % 2));
    // layer 2: bias + 64 x 64 by 64 x 32
    f32x16 D2[2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
        D2[mb] = C2[mb];
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
            D2[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A2[mb][kb], B2[kb], D2[mb], 0, 0, 0);
    }
    bf16x8 B3[4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) B3[kb] = relu_bf16(D2[kb / 2], 8 * (kb % 2));
    const f32x4 o = layer_3(B3, A3, C3, upper);
    __builtin_amdgcn_s_setprio(0);
    return o;
}

// Sum of v over each group of TAPS consecutive lanes (TAPS = 1, 4 or 16),
// left in every lane of the group, by data-parallel-primitive moves within a
// row of 16 lanes: swapping neighbours, then pairs, gives each quad its sum;
// mirroring within 8 lanes adds the neighbouring quad, mirroring within 16
// lanes the other half-row.
template <int TAPS>
__device__ __forceinline__ float tap_sum(float v)
{
    static_assert(TAPS == 1 || TAPS == 4 || TAPS == 16, "taps per query");
    auto dpp = [](float x, int ctrl) {
        switch (ctrl) {   // the control word must be a constant
        case 0:  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, true));
        case 1:  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x4E, 0xF, 0xF, true));
        case 2:  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x141, 0xF, 0xF, true));
        default: return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x140, 0xF, 0xF, true));
        }
    };
    if constexpr (TAPS >= 4) {
        v += dpp(v, 0);   // quad_perm [1,0,3,2]
        v += dpp(v, 1);   // quad_perm [2,3,0,1]
    }
    if constexpr (TAPS >= 16) {
        v += dpp(v, 2);   // row_half_mirror
        v += dpp(v, 3);   // row_mirror
    }
    return v;
}

// Four channels of a decode per lane, weighted: sum the taps of each query and
// store.  A non-finite query carries a NaN weight, so every channel it stores
// is NaN.
template <int TAPS>
__device__ __forceinline__ void emit(const InferArgs& a, const f32x4& D3, float w, uint32_t qi, int tap, int cg)
{
    float o[4] = {D3[0] * w, D3[1] * w, D3[2] * w, D3[3] * w};
#pragma unroll
    for (int c = 0; c < 4; ++c) o[c] = tap_sum<TAPS>(o[c]);
    typedef float f32x4_nt __attribute__((ext_vector_type(4)));   // results are streamed out
    if (qi < (uint32_t)a.n && tap == 0)
        __builtin_nontemporal_store((f32x4_nt){o[0], o[1], o[2], o[3]},
                                    reinterpret_cast<f32x4_nt*>(a.out) + (2 * (size_t)qi + cg));
}

// Lanes with `odd` keep b, the others a: each adds the partner's share of the
// kept value, which CTRL (a swap of lanes that differ in `odd`) brings.
template <int CTRL>
__device__ __forceinline__ float keep_sum(float a, float b, bool odd)
{
    const float keep = odd ? b : a, give = odd ? a : b;
    return keep + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, give), CTRL, 0xF, 0xF, true));
}

// The 16-tap sums of both batches of a pair (a row of 16 lanes holds a query's
// taps): the eight values a lane holds are halved at each step with the lanes
// that share their sum, 8 additions (each with a lane move and two selects
// before it) instead of 32.  Lane l (of those with
// l / 4 even) ends with channel 4 (l / 16 % 2) + l % 4 of query
// 2 (l / 8 % 2) + l / 32 of the pair's four, 128 contiguous bytes per wave.
__device__ __forceinline__ void emit16(const InferArgs& a, const f32x4 (&D3)[2], const float (&w)[2], uint32_t q0,
                                       int lane)
{
    float v[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const float r0 = keep_sum<0xB1>(D3[b][0] * w[b], D3[b][1] * w[b], lane & 1);   // quad_perm [1,0,3,2]
        const float r1 = keep_sum<0xB1>(D3[b][2] * w[b], D3[b][3] * w[b], lane & 1);
        v[b] = keep_sum<0x4E>(r0, r1, lane & 2);                                       // quad_perm [2,3,0,1]
    }
    float r = keep_sum<0x128>(v[0], v[1], lane & 8);   // row_ror:8
    r += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, r), 0x104, 0xF, 0xF, true));   // row_shl:4
    const uint32_t qi = q0 + 2 * (lane / 8 % 2) + lane / 32;
    if (qi < (uint32_t)a.n && (lane & 4) == 0)
        __builtin_nontemporal_store(r, a.out + 8 * (size_t)qi + 4 * (lane / 16 % 2) + lane % 4);
}

// Persistent waves, each handling pairs of 32-decode batches: lane l does the
// per-decode work (latent gather and interpolation) for decode l of the pair,
// so no lane repeats another's; one cross-half swap then lays the two batches'
// latents out as MFMA B operands, each with the bias ones in its upper half.
//
// The large calls run at the clock that the card's power leaves this mix, about
// 1.75 GHz, with the VALU issuing in nine of ten cycles and the matrix cores
// busy in half of them: time goes with the work, however it is interleaved (two
// waves per SIMD with both batches' chains abreast, or no raised priority:
// 890 and 907 us against 870).  What was taken out, for 4M queries of 16 taps
// (948 us before, 870 after): layer 3 as two blocks of 16 columns, layer 2's
// and 3's biases as accumulator starts (17 products of 32 x 32 x 16 per batch,
// now 10 and 4 of half the cycles), each axis of a tap located once instead of
// in every lane of the 4 x 4 block, one reduction for both batches' tap sums,
// stages that swap without moves (390 VALU instructions per pair, now 320).
template <bool CUBIC, bool STOCH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_ntex_infer(InferArgs a)
{
    constexpr int TAPS = STOCH ? 1 : (CUBIC ? 16 : 4);
    constexpr int QPB = 32 / TAPS;   // queries per 32-decode batch
    constexpr int QPP = 2 * QPB;     // queries per pair of batches
    const int lane = threadIdx.x % 64, h = lane / 32;
    const int wave = (blockIdx.x * blockDim.x + threadIdx.x) / 64;
    const int nwaves = gridDim.x * blockDim.x / 64;
    const Packed* __restrict__ pk = a.pk;
    bf16x8 A1[2], A2[2][4], A3[2];
    // The biases of layers 2 and 3 are read where they are needed: held in
    // registers for the whole loop they would not leave room for three waves.
    __shared__ f32x16 C2s[2][2];
    __shared__ f32x4 C3s[2];
    // The wave's first query, the biases and the operand images are asked for
    // together, not one after the other's barrier: 0.1 to 0.2 us of the 3.6 that
    // a small stochastic call takes.
    const int32_t npair = (int32_t)(((int64_t)a.n + QPP - 1) / QPP);
    const uint32_t nq = (uint32_t)a.n;
    auto load_uv = [&](int32_t p) {   // past the end: the last query
        return reinterpret_cast<const float2*>(a.q)[min((uint32_t)p * QPP + lane / TAPS, nq - 1)];
    };
    float2 uv_first = make_float2(0.0f, 0.0f);
    if constexpr (TAPS != 16) uv_first = load_uv(min(wave, npair));
    const float c2 = threadIdx.x < 64 ? reinterpret_cast<const float*>(pk->b2)[threadIdx.x] : 0.0f;
    const float c3 = threadIdx.x < NO ? reinterpret_cast<const float*>(pk->b3)[threadIdx.x] : 0.0f;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
        A1[mb] = pk->a1[mb][lane];
        A3[mb] = pk->a3[mb][lane];
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) A2[mb][kb] = pk->a2[mb][kb][lane];
    }
    if (threadIdx.x < 64) reinterpret_cast<float*>(C2s)[threadIdx.x] = c2;
    if (threadIdx.x < NO) reinterpret_cast<float*>(C3s)[threadIdx.x] = c3;
    __syncthreads();
    // The bias ones as every lane's slots j = 0..2 hold them in the upper
    // half: (1, 1, 1, 0, 0, 0, 0, 0) in bf16, as four 32-bit words.
    const uint32_t ONE_WORDS[4] = {0x3F803F80u, 0x00003F80u, 0u, 0u};

    const uint4* L = reinterpret_cast<const uint4*>(a.quad16);

    // A pair's decode of this lane, its latents in flight.  Every lane loads:
    // the quad index is in the table for any query.
    struct Stage {
        float w, wl[4];   // tap weight, corner weights
        uint4 lat[4];
        int sx, sy;       // texel (stochastic)
    };
    auto load_lat = [&](Stage& st, int i, int j, float fx, float fy) {
        const uint32_t e = latent_quad(a, i, j, fx, fy, st.wl);
#pragma unroll
        for (int k = 0; k < 4; ++k) st.lat[k] = L[4 * (size_t)e + k];
    };
    auto one_pair = [&](int32_t p, const Stage& cur) {
        // ---- latent interpolation of this lane's decode, rounded to bf16
        uint32_t X[4];
#pragma unroll
        for (int wsel = 0; wsel < 4; ++wsel) {
            float v[2];
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const int sh = 16 * half;
                float s = 0.0f;
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    s = __builtin_fmaf(cur.wl[k],
                                       dec_f16((uint16_t)(reinterpret_cast<const uint32_t*>(&cur.lat[k])[wsel] >> sh)), s);
                v[half] = s;
            }
            X[wsel] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){v[0], v[1]}, bf16x2));
        }
        // ---- batch 0 = decodes 0..31, batch 1 = decodes 32..63.  Swapping
        // the upper half of X with the lower half of the ones gives batch 0's
        // B operand in the first result and batch 1's in the second.
        uint32_t B1w[2][4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            auto r = __builtin_amdgcn_permlane32_swap(X[k], ONE_WORDS[k], false, false);
            B1w[0][k] = r[0];
            B1w[1][k] = r[1];
        }
        // decode weights to where layer 3 leaves the decodes: lane l of batch b
        // needs that of decode 32 b + 16 (l / 32) + l % 16
        const uint32_t wb = __builtin_bit_cast(uint32_t, cur.w);
        const auto rows = __builtin_amdgcn_permlane16_swap(wb, wb, false, false);
        const auto rw = __builtin_amdgcn_permlane32_swap(rows[0], rows[1], false, false);
        const float w[2] = {__builtin_bit_cast(float, (uint32_t)rw[0]), __builtin_bit_cast(float, (uint32_t)rw[1])};
        const uint32_t q0 = (uint32_t)p * QPP;
        f32x4 D3[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const bf16x8 B1 = __builtin_bit_cast(bf16x8, make_uint4(B1w[b][0], B1w[b][1], B1w[b][2], B1w[b][3]));
            int at = lane / 16;   // not known to be the same in every turn
            asm volatile("" : "+v"(at));
            D3[b] = mlp_batch(B1, A1, A2, A3, C2s[at / 2], C3s[at % 2], h);
            if constexpr (TAPS != 16)
                emit<TAPS>(a, D3[b], w[b], q0 + b * QPB + (16 * h + lane % 16) / TAPS, lane % TAPS, lane / 16 % 2);
        }
        if constexpr (TAPS == 16) emit16(a, D3, w, q0, lane);
        // selected texel of this lane's own decode (stochastic: one decode per query)
        if (STOCH && a.idx) {
            const uint32_t qi = q0 + lane;
            if (qi < nq) {
                const bool fin = cur.w == cur.w;
                a.idx[2 * (size_t)qi] = fin ? cur.sx : BAD_INDEX;
                a.idx[2 * (size_t)qi + 1] = fin ? cur.sy : BAD_INDEX;
            }
        }
    };

    Stage S0, S1;
    if constexpr (TAPS == 16) {
        // Two neighbouring pairs a turn (one where there are waves for all):
        // the 64 lanes locate the four taps of both axes of their eight
        // queries, and each pair's decodes fetch their two axes from there.
        // While a pair runs its MFMAs, the next one's latents are in flight,
        // and a turn ahead the queries.
        const int both = npair > nwaves ? 2 : 1;
        const int axis = lane / 4 % 2;
        const int from_x = 4 * (8 * (lane / 16) + lane % 4), from_y = 4 * (8 * (lane / 16) + 4 + lane / 4 % 4);
        const int32_t nturn = (npair + both - 1) / both;
        auto load_u = [&](int32_t t) {
            const uint32_t qi = min((uint32_t)t * (both * QPP) + lane / 8, nq - 1);
            return a.q[2 * (size_t)qi + axis];
        };
        auto fetch = [&](const AxisTap& ax, int second, Stage& st) {
            auto from = [&](int at, int v) { return __builtin_amdgcn_ds_bpermute(at + 128 * second, v); };
            auto fromf = [&](int at, float v) { return __builtin_bit_cast(float, from(at, __builtin_bit_cast(int, v))); };
            st.w = fromf(from_x, ax.w) * fromf(from_y, ax.w);
            load_lat(st, from(from_x, ax.i), from(from_y, ax.i), fromf(from_x, ax.f), fromf(from_y, ax.f));
        };
        auto locate_turn = [&](float u) {
            int y = axis;   // selected anew in every turn: four registers fewer in the loop
            asm volatile("" : "+v"(y));
            return locate_axis(u, y ? a.H : a.W, y ? a.LH : a.LW, y ? a.ry : a.rx, lane % 4);
        };
        int32_t t = wave;
        if (t >= nturn) return;
        AxisTap ax = locate_turn(load_u(t));
        float u_next = load_u(min(t + nwaves, nturn - 1));
        fetch(ax, 0, S0);
        for (;; t += nwaves) {
            const int32_t p = t * both;
            if (both == 2) fetch(ax, 1, S1);
            one_pair(p, S0);
            if (both == 1 || p + 1 >= npair) break;
            ax = locate_turn(u_next);
            u_next = load_u(min(t + 2 * nwaves, nturn - 1));
            fetch(ax, 0, S0);
            one_pair(p + 1, S1);
            if (t + nwaves >= nturn) break;
        }
    } else {
        // While pair i runs its MFMAs, the latents of pair i + 1 and the
        // queries of pair i + 2 are in flight; two pairs a turn, so that the
        // stages swap without moves.
        auto stage = [&](int32_t p, float2 uv, Stage& st) {
            const Decode d = locate<CUBIC, STOCH>(a, (uint32_t)p * QPP + lane / TAPS, lane % TAPS, uv);
            st.w = d.fin ? d.w : __builtin_nanf("");
            st.sx = d.sx;
            st.sy = d.sy;
            float fx, fy;
            const int i = latent_cell(d.sx, a.rx, a.LW, fx), j = latent_cell(d.sy, a.ry, a.LH, fy);
            load_lat(st, i, j, fx, fy);
        };
        int32_t p = wave;
        if (p >= npair) return;
        stage(p, uv_first, S0);
        float2 uv_next = load_uv(min(p + nwaves, npair));
        auto turn = [&](const Stage& cur, Stage& nxt) {
            const float2 uv_after = load_uv(min(p + 2 * nwaves, npair));
            stage(p + nwaves, uv_next, nxt);
            uv_next = uv_after;
            one_pair(p, cur);
            p += nwaves;
            return p < npair;
        };
        while (turn(S0, S1) && turn(S1, S0)) {}
    }
}

uint16_t f2bf16_host(float f)
{
    // round to nearest even (finite inputs)
    uint32_t b;
    memcpy(&b, &f, 4);
    b += 0x7fffu + ((b >> 16) & 1u);
    return (uint16_t)(b >> 16);
}

// Exact split of an fp32 value into three bf16 terms: each term takes the
// leading 8 significant bits of what the previous ones left, and 24 bits of
// significand are used up after three.
void split3_bf16(float v, uint16_t (&t)[3])
{
    float rest = v;
    for (int i = 0; i < 3; ++i) {
        t[i] = f2bf16_host(rest);
        uint32_t b = (uint32_t)t[i] << 16;
        float f;
        memcpy(&f, &b, 4);
        rest -= f;
    }
}

void pack_weights(const float* mlp, Packed* pk)
{
    memset(pk, 0, sizeof(Packed));
    auto put = [](bf16x8& dst, int j, float v) {
        uint16_t u = f2bf16_host(v);
        memcpy(reinterpret_cast<char*>(&dst) + 2 * j, &u, 2);
    };
    auto put_bias = [](bf16x8& dst, float v) {   // k-slots 8..10: lanes 32..63, j = 0..2
        uint16_t t[3];
        split3_bf16(v, t);
        memcpy(&dst, t, sizeof t);
    };
    for (int lane = 0; lane < 64; ++lane) {
        int h = lane / 32, m = lane % 32;
        for (int mb = 0; mb < 2; ++mb) {
            if (h == 0)
                for (int j = 0; j < 8; ++j) put(pk->a1[mb][lane], j, mlp[OFF_W1 + (32 * mb + m) * NL + j]);
            else
                put_bias(pk->a1[mb][lane], mlp[OFF_B1 + 32 * mb + m]);
            for (int kb = 0; kb < 4; ++kb)
                for (int j = 0; j < 8; ++j)
                    put(pk->a2[mb][kb][lane], j, mlp[OFF_W2 + (32 * mb + m) * NH + hidden_of_slot(kb, h, j)]);
        }
        for (int kb2 = 0; kb2 < 2; ++kb2)
            for (int j = 0; j < 8; ++j)
                put(pk->a3[kb2][lane], j, mlp[OFF_W3 + (lane % 8) * NH + hidden_of_slot3(kb2, lane / 16, j)]);
    }
    for (int mb = 0; mb < 2; ++mb)
        for (int h = 0; h < 2; ++h)
            for (int r = 0; r < 16; ++r) pk->b2[h][mb][r] = mlp[OFF_B2 + row_of_acc(mb, h, r)];
    for (int c = 0; c < NO; ++c) pk->b3[c / 4][c % 4] = mlp[OFF_B3 + c];
}

bool pow2_ratio(int big, int small)
{
    if (small <= 0 || big < small || big % small) return false;
    int r = big / small;
    return (r & (r - 1)) == 0;
}

}  // namespace

struct stf_neural {
    int32_t W, H, LW, LH;
    int device;
    float* lat;
    float* mlp;
    float* m_lat;
    float* v_lat;
    float* m_mlp;
    float* v_mlp;
    float* g_lat;
    float* g_mlp;
    float* partial;   // TRAIN_BLOCKS rows of PSTRIDE
    int64_t step;
    uint16_t* quad16;
    Packed* packed;
    bool ready;
};

namespace {

int64_t nlat(const stf_neural* nt)
{
    return (int64_t)nt->LW * nt->LH * NL;
}

void free_neural(stf_neural* nt)
{
    if (!nt) return;
    void* ptrs[] = {nt->lat, nt->mlp, nt->m_lat, nt->v_lat, nt->m_mlp, nt->v_mlp,
                    nt->g_lat, nt->g_mlp, nt->partial, nt->quad16, nt->packed};
    for (void* p : ptrs)
        if (p) (void)hipFree(p);
    delete nt;
}

stf_status dalloc(void** p, size_t bytes, const char* what)
{
    hipError_t e = hipMalloc(p, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
        return stf_fail(STF_E_OOM, "hipMalloc of %zu bytes for %s failed", bytes, what);
    }
    return STF_OK;
}

hipError_t fill(float* p, int64_t n, float v, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

// One forward/backward pass over a batch: per-block MLP gradients and losses
// in nt->partial (*blocks rows), the latent gradient accumulated in g_lat.
hipError_t run_fwd_bwd(stf_neural* nt, const float* target, const int32_t* pos, int32_t B, uint32_t kstep,
                       int32_t* blocks, hipStream_t s)
{
    const int32_t tiles = (B - 1) / TS + 1;
    *blocks = tiles < TRAIN_BLOCKS ? tiles : TRAIN_BLOCKS;
    TrainArgs a;
    a.lat = nt->lat;
    a.mlp = nt->mlp;
    a.target = target;
    a.pos = pos;
    a.B = B;
    a.W = nt->W;
    a.H = nt->H;
    a.LW = nt->LW;
    a.LH = nt->LH;
    a.rx = (float)nt->LW / (float)nt->W;
    a.ry = (float)nt->LH / (float)nt->H;
    a.kstep = kstep;
    a.dscale = 2.0f / (8.0f * (float)B);
    a.g_lat = nt->g_lat;
    a.partial = nt->partial;
    hipLaunchKernelGGL(k_ntex_train, dim3(*blocks), dim3(TBLOCK), 0, s, a);
    return hipGetLastError();
}

// Sums a pass's partials: into g_mlp, or (step) straight into Adam steps of
// the MLP and the latents.
hipError_t run_update(stf_neural* nt, int32_t blocks, int32_t B, float* loss, bool step, float lr_lat, float lr_mlp,
                      float c1, float c2, hipStream_t s)
{
    UpdateArgs a = {};
    a.partial = nt->partial;
    a.nblocks = blocks;
    a.g_mlp = nt->g_mlp;
    a.loss = loss;
    a.loss_scale = 1.0f / (8.0f * (float)B);
    if (step) {
        a.mlp = nt->mlp;
        a.m_mlp = nt->m_mlp;
        a.v_mlp = nt->v_mlp;
        a.lat = nt->lat;
        a.g_lat = nt->g_lat;
        a.m_lat = nt->m_lat;
        a.v_lat = nt->v_lat;
        a.nlat4 = (int32_t)(nlat(nt) / 4);   // below 2^28
        a.lr_mlp = lr_mlp;
        a.lr_lat = lr_lat;
        a.c1 = c1;
        a.c2 = c2;
    }
    const dim3 grid((unsigned)(UPDATE_MLP + (a.nlat4 + UBLOCK - 1) / UBLOCK)), block(UBLOCK);
    if (nlat(nt) >= STREAM_FROM) hipLaunchKernelGGL(k_ntex_update<true>, grid, block, 0, s, a);
    else hipLaunchKernelGGL(k_ntex_update<false>, grid, block, 0, s, a);
    return hipGetLastError();
}

stf_status check_neural(const stf_neural* nt)
{
    if (!nt) return stf_fail(STF_E_INVALID, "neural texture is NULL");
    return STF_OK;
}

stf_status check_dev(const void* p, const char* what, size_t align)
{
    if (!p) return stf_fail(STF_E_INVALID, "%s is NULL", what);
    if ((uintptr_t)p % align) return stf_fail(STF_E_INVALID, "%s is not %zu-byte aligned", what, align);
    hipPointerAttribute_t attr;
    hipError_t e = hipPointerGetAttributes(&attr, p);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return stf_fail(STF_E_INVALID, "%s is not a device pointer", what);
    }
    if (attr.type != hipMemoryTypeDevice && attr.type != hipMemoryTypeManaged)
        return stf_fail(STF_E_INVALID, "%s is not device memory", what);
    return STF_OK;
}

}  // namespace

extern "C" {

int32_t stf_ntex_param_count(void)
{
    return NPARAM;
}

stf_status stf_ntex_create(int32_t tex_w, int32_t tex_h, int32_t lat_w, int32_t lat_h, const float* latents_host,
                           const float* mlp_host, stf_neural** out)
{
    stf_clear_error();
    if (!out) return stf_fail(STF_E_INVALID, "out is NULL");
    *out = nullptr;
    if (tex_w < 1 || tex_h < 1 || tex_w > 65536 || tex_h > 65536 || lat_w < 1 || lat_h < 1)
        return stf_fail(STF_E_INVALID, "sizes out of range");
    if (!pow2_ratio(tex_w, lat_w) || !pow2_ratio(tex_h, lat_h))
        return stf_fail(STF_E_UNSUPPORTED, "texture/latent size ratios must be powers of two");
    if ((int64_t)lat_w * lat_h * NL * 2 >= ((int64_t)1 << 31))
        return stf_fail(STF_E_UNSUPPORTED, "latent grid too large");
    if (!latents_host || !mlp_host) return stf_fail(STF_E_INVALID, "initial parameters are NULL");
    stf_neural* nt = new (std::nothrow) stf_neural();
    if (!nt) return stf_fail(STF_E_OOM, "host allocation failed");
    nt->W = tex_w;
    nt->H = tex_h;
    nt->LW = lat_w;
    nt->LH = lat_h;
    (void)hipGetDevice(&nt->device);
    size_t lb = (size_t)nlat(nt) * 4;
    stf_status s = STF_OK;
    float** bufs[] = {&nt->lat, &nt->m_lat, &nt->v_lat, &nt->g_lat};
    for (float** b : bufs)
        if (s == STF_OK) s = dalloc((void**)b, lb, "latents");
    float** mbufs[] = {&nt->mlp, &nt->m_mlp, &nt->v_mlp, &nt->g_mlp};
    for (float** b : mbufs)
        if (s == STF_OK) s = dalloc((void**)b, NPARAM * 4, "MLP parameters");
    if (s == STF_OK)
        s = dalloc((void**)&nt->quad16, (size_t)(lat_w + 1) * (lat_h + 1) * 4 * NL * 2, "binary16 corner quads");
    if (s == STF_OK) s = dalloc((void**)&nt->packed, sizeof(Packed), "packed weights");
    if (s == STF_OK) s = dalloc((void**)&nt->partial, (size_t)TRAIN_BLOCKS * PSTRIDE * 4, "gradient partials");
    if (s == STF_OK) {
        hipError_t e = hipMemcpy(nt->lat, latents_host, lb, hipMemcpyHostToDevice);
        if (e == hipSuccess) e = hipMemcpy(nt->mlp, mlp_host, NPARAM * 4, hipMemcpyHostToDevice);
        if (e == hipSuccess) e = fill(nt->m_lat, nlat(nt), 0.0f, 0);
        if (e == hipSuccess) e = fill(nt->v_lat, nlat(nt), 0.0f, 0);
        if (e == hipSuccess) e = fill(nt->g_lat, nlat(nt), 0.0f, 0);
        if (e == hipSuccess) e = fill(nt->m_mlp, NPARAM, 0.0f, 0);
        if (e == hipSuccess) e = fill(nt->v_mlp, NPARAM, 0.0f, 0);
        if (e == hipSuccess) e = hipDeviceSynchronize();
        if (e != hipSuccess) s = stf_fail(STF_E_DEVICE, "initialising the neural texture failed: %s", hipGetErrorString(e));
    }
    if (s != STF_OK) {
        free_neural(nt);
        return s;
    }
    *out = nt;
    return STF_OK;
}

void stf_ntex_destroy(stf_neural* nt)
{
    free_neural(nt);
}

stf_status stf_ntex_train(stf_neural* nt, const float* target_dev, int32_t steps, int32_t batch, float lr_latent,
                          float lr_mlp, uint64_t seed, float* loss_dev, void* hip_stream)
{
    stf_clear_error();
    stf_status s = check_neural(nt);
    if (s != STF_OK) return s;
    if (steps < 0 || batch < 1) return stf_fail(STF_E_INVALID, "steps = %d, batch = %d", steps, batch);
    if (!(lr_latent >= 0.0f) || !(lr_mlp >= 0.0f)) return stf_fail(STF_E_INVALID, "learning rates must be >= 0");
    if (steps == 0) return STF_OK;
    s = check_dev(target_dev, "target_dev", 16);
    if (s == STF_OK && loss_dev) s = check_dev(loss_dev, "loss_dev", 4);
    if (s != STF_OK) return s;
    hipStream_t st = (hipStream_t)hip_stream;
    uint32_t key = seed_key(seed);
    for (int32_t k = 0; k < steps; ++k) {
        nt->step += 1;
        double c1 = 1.0 / (1.0 - pow(0.9, (double)nt->step)), c2 = 1.0 / (1.0 - pow(0.999, (double)nt->step));
        int32_t blocks = 0;
        hipError_t e = run_fwd_bwd(nt, target_dev, nullptr, batch, pcg(key ^ (uint32_t)nt->step), &blocks, st);
        if (e == hipSuccess)
            e = run_update(nt, blocks, batch, loss_dev ? loss_dev + k : nullptr, true, lr_latent, lr_mlp, (float)c1,
                           (float)c2, st);
        if (e != hipSuccess) return stf_fail(STF_E_DEVICE, "training launch failed: %s", hipGetErrorString(e));
    }
    nt->ready = false;
    return STF_OK;
}

stf_status stf_ntex_gradients(stf_neural* nt, const float* target_dev, const int32_t* positions_dev, int32_t batch,
                              float* grad_latents_dev, float* grad_mlp_dev, float* loss_dev, void* hip_stream)
{
    stf_clear_error();
    stf_status s = check_neural(nt);
    if (s != STF_OK) return s;
    if (batch < 1) return stf_fail(STF_E_INVALID, "batch = %d", batch);
    s = check_dev(target_dev, "target_dev", 16);
    if (s == STF_OK) s = check_dev(positions_dev, "positions_dev", 4);
    if (s == STF_OK) s = check_dev(grad_latents_dev, "grad_latents_dev", 4);
    if (s == STF_OK) s = check_dev(grad_mlp_dev, "grad_mlp_dev", 4);
    if (s == STF_OK && loss_dev) s = check_dev(loss_dev, "loss_dev", 4);
    if (s != STF_OK) return s;
    hipStream_t st = (hipStream_t)hip_stream;
    hipError_t e = fill(nt->g_lat, nlat(nt), 0.0f, st);
    int32_t blocks = 0;
    if (e == hipSuccess) e = run_fwd_bwd(nt, target_dev, positions_dev, batch, 0u, &blocks, st);
    if (e == hipSuccess) e = run_update(nt, blocks, batch, loss_dev, false, 0.0f, 0.0f, 0.0f, 0.0f, st);
    if (e == hipSuccess)
        e = hipMemcpyAsync(grad_latents_dev, nt->g_lat, (size_t)nlat(nt) * 4, hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(grad_mlp_dev, nt->g_mlp, NPARAM * 4, hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess) e = fill(nt->g_lat, nlat(nt), 0.0f, st);
    if (e != hipSuccess) return stf_fail(STF_E_DEVICE, "gradient launch failed: %s", hipGetErrorString(e));
    return STF_OK;
}

stf_status stf_ntex_get_params(const stf_neural* nt, float* latents_host, float* mlp_host)
{
    stf_clear_error();
    stf_status s = check_neural(nt);
    if (s != STF_OK) return s;
    hipError_t e = hipDeviceSynchronize();
    if (e == hipSuccess && latents_host) e = hipMemcpy(latents_host, nt->lat, (size_t)nlat(nt) * 4, hipMemcpyDeviceToHost);
    if (e == hipSuccess && mlp_host) e = hipMemcpy(mlp_host, nt->mlp, NPARAM * 4, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return stf_fail(STF_E_DEVICE, "copying parameters failed: %s", hipGetErrorString(e));
    return STF_OK;
}

stf_status stf_ntex_prepare_inference(stf_neural* nt, void* hip_stream)
{
    stf_clear_error();
    stf_status s = check_neural(nt);
    if (s != STF_OK) return s;
    std::vector<float> mlp(NPARAM);
    hipError_t e = hipDeviceSynchronize();
    if (e == hipSuccess) e = hipMemcpy(mlp.data(), nt->mlp, NPARAM * 4, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return stf_fail(STF_E_DEVICE, "reading the MLP failed: %s", hipGetErrorString(e));
    Packed* pk = new (std::nothrow) Packed;
    if (!pk) return stf_fail(STF_E_OOM, "host allocation failed");
    pack_weights(mlp.data(), pk);
    e = hipMemcpy(nt->packed, pk, sizeof(Packed), hipMemcpyHostToDevice);
    delete pk;
    hipStream_t st = (hipStream_t)hip_stream;
    if (e == hipSuccess) {
        const int64_t nq = (int64_t)(nt->LW + 1) * (nt->LH + 1);
        hipLaunchKernelGGL(k_to_quads, dim3((unsigned)((nq + 255) / 256)), dim3(256), 0, st, nt->lat, nt->quad16, nt->LW,
                           nt->LH);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return stf_fail(STF_E_DEVICE, "preparing inference failed: %s", hipGetErrorString(e));
    nt->ready = true;
    return STF_OK;
}

stf_status stf_ntex_filter(const stf_neural* nt, const float* queries_dev, int64_t n, stf_filter_kind filter,
                           stf_mode mode, uint64_t seed, float* out_dev, int32_t* out_index_dev, void* hip_stream)
{
    stf_clear_error();
    stf_status s = check_neural(nt);
    if (s != STF_OK) return s;
    if (!nt->ready) return stf_fail(STF_E_INVALID, "call stf_ntex_prepare_inference after training");
    if (n < 0 || n > 0x7fffffff) return stf_fail(STF_E_INVALID, "n = %lld out of range", (long long)n);
    if (!valid_filter(filter)) return stf_fail(STF_E_INVALID, "unknown filter");
    if (filter != STF_LINEAR && filter != STF_CUBIC_BSPLINE)
        return stf_fail(STF_E_UNSUPPORTED, "neural textures support the linear and B-spline filters only");
    if (mode != STF_DETERMINISTIC && mode != STF_STOCHASTIC) return stf_fail(STF_E_INVALID, "unknown mode");
    if (mode == STF_DETERMINISTIC && out_index_dev)
        return stf_fail(STF_E_INVALID, "out_index_dev must be NULL in deterministic mode");
    if (n == 0) return STF_OK;
    s = check_dev(queries_dev, "queries_dev", 8);
    if (s == STF_OK) s = check_dev(out_dev, "out_dev", 16);
    if (s == STF_OK && out_index_dev) s = check_dev(out_index_dev, "out_index_dev", 4);
    if (s != STF_OK) return s;
    InferArgs a;
    a.pk = nt->packed;
    a.quad16 = nt->quad16;
    a.q = queries_dev;
    a.n = (int32_t)n;
    a.W = nt->W;
    a.H = nt->H;
    a.LW = nt->LW;
    a.LH = nt->LH;
    a.rx = (float)nt->LW / (float)nt->W;
    a.ry = (float)nt->LH / (float)nt->H;
    a.key = seed_key(seed);
    a.out = out_dev;
    a.idx = out_index_dev;
    int taps = mode == STF_STOCHASTIC ? 1 : (filter == STF_CUBIC_BSPLINE ? 16 : 4);
    int64_t pairs = (n * taps + 63) / 64;   // pairs of 32-decode batches
    // Persistent waves, one resident set (3 per SIMD on 256 CUs): the weights
    // load once per wave.
    int64_t waves = pairs < 3072 ? pairs : 3072;
    // The 16-tap kernel's waves take two pairs a turn where there are more than
    // waves: up to two sets a wave a pair, which leaves no SIMD with six of them
    // while others have three (20,000 queries 8.5 us, 7.9 so).
    if (taps == 16 && pairs <= 2 * 3072) waves = pairs;
    dim3 grid((unsigned)((waves + 3) / 4)), block(256);
    hipStream_t st = (hipStream_t)hip_stream;
    bool cubic = filter == STF_CUBIC_BSPLINE;
    if (mode == STF_STOCHASTIC) {
        if (cubic) hipLaunchKernelGGL((k_ntex_infer<true, true>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((k_ntex_infer<false, true>), grid, block, 0, st, a);
    } else {
        if (cubic) hipLaunchKernelGGL((k_ntex_infer<true, false>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((k_ntex_infer<false, false>), grid, block, 0, st, a);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return stf_fail(STF_E_DEVICE, "kernel launch failed: %s", hipGetErrorString(e));
    return STF_OK;
}

}  // extern "C"
