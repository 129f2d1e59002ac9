// 3x3 / stride-1 backward-filter of small layers, fp32 and bf16, in one launch: no workspace, no atomics, no zero fill.
//
// Such a layer has few outputs (16 x 16 channels: 2304) and a sum over a few hundred to a few thousand pixels, which the general
// kernels walk in one or a handful of workgroups, step by step through LDS with a barrier each, behind a launch that clears dw.
// Here a workgroup takes 16 x 16 channels of one filter row (three taps); its waves share out the pixels in units of 16 bytes of an
// output row, four units an MFMA (v_mfma_f32_16x16x4_f32, v_mfma_f32_16x16x32_bf16): a lane is a channel of dy and of x and holds one
// unit of its dy row, the unit under it of its x row and a column on either side; the three taps are shifts of it in registers.
// What bounds it is the cache lines that a load touches, on the few compute units such a layer has workgroups for: loading, four
// neighbouring lanes are the four units of one channel (16 lines a load; with the MFMA's lanes, whose neighbours are channels, and
// single elements it was 64 lines in two to five times the loads: 2 x 16 x 16x16, 16 channels 11.0 us fp32, 9.9 bf16), and the units
// change lanes through the wave's own LDS.  No barrier before the waves' sums, which meet in LDS in order.
// us a call, before (without workspace; planned with 32 MiB) -> now: 2 x 16 x 16x16, 16 channels fp32 16.6 (17.2) -> 6.5, bf16 21.9
// (15.6) -> 4.4; 1 x 64 x 8x8, 64 channels 10.5 -> 3.6 and 12.1 -> 4.1; 2 x 80 x 24x24, 77 channels 26.7 -> 11.6 and 30.4 (15.5) -> 6.7.
#include <algorithm>
#include <cmath>

#include "sn_internal.h"

namespace sn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int MAXWAVES = 16;

struct SmallWgrad {
    int K, C, H, W, P, Q, ph, pw;
    int ktiles, uq, units;     // units of an output row, of all
    long long x_total, d_total;
};

// PX elements from p + off on, at the element's own alignment (element by element where they are not all in [0, total)).
template <typename T> __device__ inline u32x4 load_unit(const T *p, long long off, long long total)
{
    constexpr int PX = 16 / sizeof(T);
    struct __attribute__((packed, aligned(sizeof(T)))) Any { u32x4 v; };
    if (off >= 0 && off + PX <= total) return reinterpret_cast<const Any *>(p + off)->v;
    T e[PX];
#pragma unroll
    for (int i = 0; i < PX; ++i) e[i] = off + i >= 0 && off + i < total ? p[off + i] : T(0);
    u32x4 v;
    __builtin_memcpy(&v, e, 16);
    return v;
}

// The first n elements, the others zero; the elements lo .. n - 1.
template <typename T> __device__ inline u32x4 keep(u32x4 v, int lo, int n)
{
    constexpr int PX = 16 / sizeof(T);
    T e[PX];
    __builtin_memcpy(e, &v, 16);
#pragma unroll
    for (int i = 0; i < PX; ++i) e[i] = i >= lo && i < n ? e[i] : T(0);
    __builtin_memcpy(&v, e, 16);
    return v;
}

template <typename T>
__global__ void __launch_bounds__(64 * MAXWAVES)
small3x3_wgrad_kernel(const T *__restrict__ x, const T *__restrict__ dy, float *__restrict__ dw, const SmallWgrad p)
{
    constexpr int PX = 16 / sizeof(T);
    extern __shared__ __attribute__((aligned(16))) float sums[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    const int row = lane & 15, g = lane >> 4, r = blockIdx.y;
    // loading, a lane is channel lane / 4 and unit lane % 4 of four: neighbouring lanes read neighbouring units
    const int k = blockIdx.x % p.ktiles * 16 + (lane >> 2), c = blockIdx.x / p.ktiles * 16 + (lane >> 2);

    struct Unit { u32x4 d, x; T left, right; int n; };   // n: elements of the unit inside its row
    auto load = [&](int u, Unit &o) {
        const int line = u / p.uq, q0 = (u - line * p.uq) * PX, n = line / p.P, ph = line - n * p.P, h = ph + r - p.ph, v0 = q0 - p.pw;
        const bool ok = u < p.units, drow = ok && k < p.K, xrow = ok && c < p.C && (unsigned)h < (unsigned)p.H;
        const long long da = drow ? (((long long)n * p.K + k) * p.P + ph) * p.Q + q0 : 0, xa = xrow ? (((long long)n * p.C + c) * p.H + h) * p.W + v0 : 0;
        o.n = ok ? min(p.Q - q0, PX) : 0;
        o.d = keep<T>(load_unit<T>(dy, da, p.d_total), 0, drow ? o.n : 0);
        o.x = keep<T>(load_unit<T>(x, xa + 1, p.x_total), -v0 - 1, xrow ? p.W - v0 - 1 : 0);
        const bool l = xrow && (unsigned)v0 < (unsigned)p.W, rt = xrow && (unsigned)(v0 + PX + 1) < (unsigned)p.W;
        const T lv = x[l ? xa : 0], rv = x[rt ? xa + PX + 1 : 0];
        o.left = l ? lv : T(0);
        o.right = rt ? rv : T(0);
    };
    f32x4 acc[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 *mine = reinterpret_cast<u32x4 *>(sums) + wave * 192;
    auto multiply = [&](const Unit &o) {
        u32x4 ends = {0, 0, (uint32_t)o.n, 0};
        __builtin_memcpy(&ends, &o.left, sizeof(T));
        __builtin_memcpy(reinterpret_cast<char *>(&ends) + 4, &o.right, sizeof(T));
        mine[lane] = o.d;
        mine[64 + lane] = o.x;
        mine[128 + lane] = ends;
        __builtin_amdgcn_wave_barrier();   // (the wave's own LDS, in order: no more than the compiler has to know)
        const int from = 4 * row + g;      // multiplying, a lane is channel lane % 16 and unit lane / 16
        const u32x4 d = mine[from], xm = mine[64 + from], en = mine[128 + from];
        __builtin_amdgcn_wave_barrier();
        T xe[PX + 2], de[PX];
        __builtin_memcpy(de, &d, 16);
        __builtin_memcpy(xe, &en, sizeof(T));
        __builtin_memcpy(xe + 1, &xm, 16);
        __builtin_memcpy(xe + PX + 1, reinterpret_cast<const char *>(&en) + 4, sizeof(T));
        const int n = (int)en[2];
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            // (past the row's end dy is zero, but x may hold a pixel there, which would meet it as an Inf or a NaN)
            T b[PX];
#pragma unroll
            for (int e = 0; e < PX; ++e) b[e] = e < n ? xe[e + s] : T(0);
            if constexpr (sizeof(T) == 2) {
                bf16x8 xb;
                __builtin_memcpy(&xb, b, 16);
                acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, d), xb, acc[s], 0, 0, 0);
            } else {
#pragma unroll
                for (int e = 0; e < PX; ++e) acc[s] = __builtin_amdgcn_mfma_f32_16x16x4f32(de[e], b[e], acc[s], 0, 0, 0);
            }
        }
    };
    Unit u0, u1;
    const int step = 4 * waves;
    int u = 4 * wave;
    if (u < p.units) {
        load(u + (lane & 3), u0);
        for (;;) {
            if (u + step < p.units) load(u + step + (lane & 3), u1);
            multiply(u0);
            if ((u += step) >= p.units) break;
            if (u + step < p.units) load(u + step + (lane & 3), u0);
            multiply(u1);
            if ((u += step) >= p.units) break;
        }
    }
    __syncthreads();
    // register v of a lane: channel 4 * g + v of dy, the lane's channel of x
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int v = 0; v < 4; ++v) sums[(wave * 12 + s * 4 + v) * 64 + lane] = acc[s][v];
    __syncthreads();
    for (int i = threadIdx.x; i < 768; i += blockDim.x) {
        float t = sums[i];
        for (int w = 1; w < waves; ++w) t += sums[w * 768 + i];
        const int s = i >> 8, v = (i >> 6) & 3, ln = i & 63;
        const int ko = blockIdx.x % p.ktiles * 16 + 4 * (ln >> 4) + v, co = blockIdx.x / p.ktiles * 16 + (ln & 15);
        if (ko < p.K && co < p.C) dw[((size_t)ko * p.C + co) * 9 + r * 3 + s] = t;
    }
}

bool problem_of(const ConvGeom &g, SmallWgrad *p)
{
    if (g.R != 3 || g.S != 3 || g.sh != 1 || g.sw != 1) return false;
    const long long sz = g.in_bf16 ? 2 : 4, px = 16 / sz;
    p->K = g.K; p->C = g.C; p->H = g.H; p->W = g.W; p->P = g.P; p->Q = g.Q; p->ph = g.ph; p->pw = g.pw;
    p->ktiles = (g.K + 15) / 16;
    const long long uq = (g.Q + px - 1) / px, units = uq * g.P * g.N;
    if (units > (1 << 30) || (long long)p->ktiles * ((g.C + 15) / 16) > 0x7fffffffLL) return false;
    p->uq = (int)uq;
    p->units = (int)units;
    p->x_total = (long long)g.N * g.C * g.H * g.W;
    p->d_total = (long long)g.N * g.K * g.P * g.Q;
    return true;
}

}  // namespace

// us = start + work * steps on the chip + unit * steps on one compute unit + turn * its workgroups, a step being four units of 16 bytes of a
// row: 4600 layers (1 to 16 images, 8 to 512 channels, planes of 4x4 to 64x64) to 6 % in bf16 and 4 % in fp32 (rms).
double small_wgrad_us(const ConvGeom &g)
{
    SmallWgrad p;
    if (!problem_of(g, &p)) return 1e9;
    const double steps = (p.units + 3) / 4, wgs = 3.0 * p.ktiles * ((g.C + 15) / 16), each = std::ceil(wgs / 256);
    return g.in_bf16 ? 3.6 + 0.033 * steps * wgs / 256 + (0.088 * steps + 0.91) * each : 3.5 + 0.033 * steps * wgs / 256 + (0.109 * steps + 0.68) * each;
}

hipError_t launch_small_wgrad(const void *x, const void *dy, float *dw, const ConvGeom &g, hipStream_t st)
{
    SmallWgrad p;
    if (!problem_of(g, &p)) return hipErrorInvalidValue;
    const int waves = std::max(1, std::min(MAXWAVES, (p.units + 3) / 4));
    const dim3 grid((unsigned)p.ktiles * ((g.C + 15) / 16), 3), block(64 * waves);
    if (g.in_bf16)
        hipLaunchKernelGGL(small3x3_wgrad_kernel<bf16_t>, grid, block, waves * 3072, st, static_cast<const bf16_t *>(x), static_cast<const bf16_t *>(dy), dw, p);
    else
        hipLaunchKernelGGL(small3x3_wgrad_kernel<float>, grid, block, waves * 3072, st, static_cast<const float *>(x), static_cast<const float *>(dy), dw, p);
    return hipGetLastError();
}

}  // namespace sn
