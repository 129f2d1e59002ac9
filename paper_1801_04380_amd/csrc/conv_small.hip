// fp32 3x3 / stride-1 forward and backward-data of problems too small to fill the chip with GEMM tiles, in one launch without workspace.
//
// What bounds these layers is latency: the general kernel gives 2 x 16 x 16x16 (16 channels) 8 workgroups of 64 x 64, each of
// which stages its 144 reduction elements through LDS step by step with nothing else on its compute unit.  Two kernels without a
// barrier in the reduction, whose partial sums meet in LDS in a fixed order:
//   small3x3_kernel, below 16 reduction channels: a wave holds 64 output pixels of four output channels and the four waves of a
//     workgroup share out the channels; per channel a lane has its nine inputs in flight at once and the taps come once per wave.
//   small3x3_mfma_kernel, from 16 on, as the bf16 kernel of such layers (conv_small_bf16.hip): a workgroup takes 16 output channels x a 4 x 4
//     patch of outputs and its waves share out the reduction, 16 channels a step (v_mfma_f32_16x16x4_f32): a lane is an output channel and
//     every fourth reduction channel, whose nine taps lie together in the filter; for the patch it is one of its 36 pixels with their halo, gathers
//     16 channels of it (range-checked: the padding is zeros) into the wave's own LDS, and a tap's operand is an LDS read at a shifted pixel.
// Time of a call, general kernel -> the first: 4 x 32 x 16x16, 32 channels, forward 35 -> 9.6, backward-data 55 -> 9.2 us; 60 layers of 2.2e6 to 15.8e6
// multiplications (1 to 8 images, 4 to 254 channels, planes of 4x4 to 63x63): forward 1.02 to 6.4 times faster, backward-data 1.65 to 9.3 times.
// The first -> the second: 2 x 16 x 16x16, 16 channels forward 5.9 -> 4.0, backward-data 5.7 -> 3.8 us; of 70 such layers those of 16 reduction
// channels and more 1.4 to 7.7 times faster, with 0.7 of the error; of fewer than eight some slower (0.61 times), of eight to fifteen with up to 1.3
// times the error.
#include <algorithm>

#include "sn_internal.h"

namespace sn {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int KO = 4, WAVES = 4;

struct Small3x3 {
    int M, Red, npix;          // output channels, reduction channels, output pixels of all images
    int IH, IW, OH, OW;
    int off_h, off_w;          // input row / column of output pixel (0, 0)'s first tap
    int w_so, w_sr;            // strides of an output / reduction channel in the filter
};

template <bool FLIP>
__global__ void __launch_bounds__(64 * WAVES)
small3x3_kernel(const float *__restrict__ in, const float *__restrict__ w, float *__restrict__ out, const Small3x3 p)
{
    __shared__ float sums[WAVES][KO][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int pix = blockIdx.x * 64 + lane, o0 = blockIdx.y * KO;
    const int ohw = p.OH * p.OW, ihw = p.IH * p.IW;
    const int px = min(pix, p.npix - 1), n = px / ohw, at = px - n * ohw, oh = at / p.OW, ow = at - oh * p.OW;
    int off[9];
    bool in_image[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const int h = oh + p.off_h + t / 3, v = ow + p.off_w + t % 3;
        in_image[t] = (unsigned)h < (unsigned)p.IH && (unsigned)v < (unsigned)p.IW;
        off[t] = in_image[t] ? h * p.IW + v : 0;
    }
    const float *ip = in + (size_t)n * p.Red * ihw;
    float acc[KO];
#pragma unroll
    for (int k = 0; k < KO; ++k) acc[k] = 0.f;
#pragma unroll 2
    for (int c = wave; c < p.Red; c += WAVES) {
        float x[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const float v = ip[(size_t)c * ihw + off[t]];
            x[t] = in_image[t] ? v : 0.f;
        }
#pragma unroll
        for (int k = 0; k < KO; ++k) {
            const float *wp = w + (size_t)min(o0 + k, p.M - 1) * p.w_so + (size_t)c * p.w_sr;
#pragma unroll
            for (int t = 0; t < 9; ++t) acc[k] = __builtin_fmaf(x[t], wp[FLIP ? 8 - t : t], acc[k]);
        }
    }
#pragma unroll
    for (int k = 0; k < KO; ++k) sums[wave][k][lane] = acc[k];
    __syncthreads();
    const int o = o0 + wave;   // wave k finishes output channel k
    if (pix >= p.npix || o >= p.M) return;
    const float v = (sums[0][wave][lane] + sums[1][wave][lane]) + (sums[2][wave][lane] + sums[3][wave][lane]);
    out[((size_t)n * p.M + o) * ohw + at] = v;
}

constexpr int MT = 16, TS = 4, LW = TS + 2, SLOTS = LW * LW, RED = 16, PLANE = 40, MAXWAVES = 8;   // PLANE: floats of a channel's patch
constexpr uint32_t FAR = 0x80000000u;   // an offset outside every tensor: loads bring zeros

struct Patches {
    int M, Red;                // output channels, reduction channels
    int IH, IW, OH, OW;
    int off_h, off_w;          // input row / column of output pixel (0, 0)'s first tap
    int mtiles, tiles_w, tiles;   // channel tiles; patches per row of patches, per image
    int w_so, w_sr;            // strides of an output / reduction channel in the filter
};

template <bool FLIP>
__global__ void __launch_bounds__(64 * MAXWAVES)
small3x3_mfma_kernel(const float *__restrict__ in, const float *__restrict__ w, float *__restrict__ out, const Patches p)
{
    extern __shared__ float lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    const int row = lane & 15, g = lane >> 4;
    const int mt = blockIdx.x % p.mtiles, tile = blockIdx.x / p.mtiles;
    const int n = tile / p.tiles, t = tile - n * p.tiles, h0 = t / p.tiles_w * TS, v0 = t % p.tiles_w * TS;
    const int m = mt * MT + row;
    const uint32_t ihw = (uint32_t)p.IH * p.IW * 4;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(in) + (size_t)n * p.Red * p.IH * p.IW, 0, (uint32_t)p.Red * ihw, 0x00020000);
    uint32_t xoff;
    {
        const int r = lane / LW, c = lane - r * LW, h = h0 + p.off_h + r, v = v0 + p.off_w + c;
        const bool ok = lane < SLOTS && (unsigned)h < (unsigned)p.IH && (unsigned)v < (unsigned)p.IW;
        xoff = ok ? (uint32_t)(h * p.IW + v) * 4 : FAR;
    }
    struct Step { float a[4][9], x[RED]; };
    auto load = [&](int c0, Step &s) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {   // reduction channel c0 + 4 j + g
            const int c = c0 + 4 * j + g;
            const bool ok = m < p.M && c < p.Red;
            const float *q = w + (size_t)min(m, p.M - 1) * p.w_so + (size_t)min(c, p.Red - 1) * p.w_sr;
#pragma unroll
            for (int e = 0; e < 9; ++e) s.a[j][e] = q[e];
#pragma unroll
            for (int e = 0; e < 9; ++e) s.a[j][e] = ok ? s.a[j][e] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < RED; ++i) {
            const int c = c0 + i;   // (past the last: an offset behind the last channel's, so that FAR stays outside)
            s.x[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xr, c < p.Red ? xoff : FAR, (uint32_t)min(c, p.Red - 1) * ihw, 0));
        }
    };
    // (four chains, added up at the end: one of four times the roundings was up to 1.9 times further from the exact result)
    f32x4 part[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) part[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float *patch = lds + wave * RED * PLANE;
    const float *mine = patch + g * PLANE + (row >> 2) * LW + (row & 3);   // the lane's pixel under tap (0, 0), channel g
    auto multiply = [&](const Step &s) {
        if (lane < PLANE) {
#pragma unroll
            for (int i = 0; i < RED; ++i) patch[i * PLANE + lane] = s.x[i];
        }
        __builtin_amdgcn_wave_barrier();   // (the wave's own LDS, in order: no more than the compiler has to know)
#pragma unroll
        for (int e = 0; e < 9; ++e)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                part[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(s.a[j][FLIP ? 8 - e : e], mine[4 * j * PLANE + (e / 3) * LW + e % 3], part[j], 0, 0, 0);
        __builtin_amdgcn_wave_barrier();
    };
    const int step = RED * waves;
    Step s0, s1;
    int c = RED * wave;
    if (c < p.Red) {
        load(c, s0);
        for (;;) {
            if (c + step < p.Red) load(c + step, s1);
            multiply(s0);
            if ((c += step) >= p.Red) break;
            if (c + step < p.Red) load(c + step, s0);
            multiply(s1);
            if ((c += step) >= p.Red) break;
        }
    }
    // register v of a lane is output channel 4 * g + v, the lane's pixel
    const f32x4 acc = (part[0] + part[1]) + (part[2] + part[3]);
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 4; ++v) lds[(wave * 4 + v) * 64 + lane] = acc[v];
    __syncthreads();
    for (int i = threadIdx.x; i < 256; i += blockDim.x) {
        float s = lds[i];
        for (int k = 1; k < waves; ++k) s += lds[k * 256 + i];
        const int v = i >> 6, ln = i & 63, px = ln & 15;
        const int mo = mt * MT + 4 * (ln >> 4) + v, h = h0 + (px >> 2), q = v0 + (px & 3);
        if (mo < p.M && h < p.OH && q < p.OW) out[(((size_t)n * p.M + mo) * p.OH + h) * p.OW + q] = s;
    }
}

}  // namespace

bool small3x3_supported(const ConvGeom &g, bool bwd)
{
    if (g.in_bf16 || g.R != 3 || g.S != 3 || g.sh != 1 || g.sw != 1 || g.P < 1 || g.Q < 1) return false;
    const long long M = bwd ? g.C : g.K, red = bwd ? g.K : g.C, npix = (long long)g.N * (bwd ? g.H * (long long)g.W : g.P * (long long)g.Q);
    const long long inputs = (long long)g.N * red * (bwd ? g.P * (long long)g.Q : g.H * (long long)g.W);
    return M * red * npix * 9 <= SMALL3X3_MACS && M <= 65535LL * KO && inputs < (1LL << 29);   // (KO output channels per grid row; 32-bit byte offsets)
}

hipError_t launch_small3x3(const void *in, const void *w, void *out, const ConvGeom &g, bool bwd, hipStream_t st)
{
    static_assert(KO == WAVES, "wave k finishes output channel k");
    const auto fill = [&](auto &p) {
        p.M = bwd ? g.C : g.K;
        p.Red = bwd ? g.K : g.C;
        p.OH = bwd ? g.H : g.P; p.OW = bwd ? g.W : g.Q;
        p.IH = bwd ? g.P : g.H; p.IW = bwd ? g.Q : g.W;
        p.off_h = bwd ? g.ph - 2 : -g.ph;
        p.off_w = bwd ? g.pw - 2 : -g.pw;
        p.w_so = bwd ? 9 : g.C * 9;
        p.w_sr = bwd ? g.C * 9 : 9;
    };
    const float *a = static_cast<const float *>(in), *b = static_cast<const float *>(w);
    float *o = static_cast<float *>(out);
    if ((bwd ? g.K : g.C) >= RED) {
        Patches p;
        fill(p);
        p.mtiles = (p.M + MT - 1) / MT;
        p.tiles_w = (p.OW + TS - 1) / TS;
        p.tiles = p.tiles_w * ((p.OH + TS - 1) / TS);
        const int waves = std::min(MAXWAVES, (p.Red + RED - 1) / RED);
        const dim3 grid((unsigned)(p.tiles * g.N * p.mtiles)), block(64 * waves);   // (fewer than the products there may be)
        const int lds = waves * RED * PLANE * (int)sizeof(float);                   // patches; the sums take less
        if (bwd) hipLaunchKernelGGL(small3x3_mfma_kernel<true>, grid, block, lds, st, a, b, o, p);
        else hipLaunchKernelGGL(small3x3_mfma_kernel<false>, grid, block, lds, st, a, b, o, p);
        return hipGetLastError();
    }
    Small3x3 p;
    fill(p);
    p.npix = g.N * p.OH * p.OW;
    const dim3 grid((p.npix + 63) / 64, (p.M + KO - 1) / KO), block(64 * WAVES);
    if (bwd) hipLaunchKernelGGL(small3x3_kernel<true>, grid, block, 0, st, a, b, o, p);
    else hipLaunchKernelGGL(small3x3_kernel<false>, grid, block, 0, st, a, b, o, p);
    return hipGetLastError();
}

}  // namespace sn
