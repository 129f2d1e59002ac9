// fp32 3x3 / stride-1 forward and backward-data of problems too small to fill the chip with GEMM tiles: a wave holds 64
// output pixels of four output channels, and the four waves of a workgroup share out the reduction channels.
//
// What bounds these layers is latency: the general kernel gives 2 x 16 x 16x16 (16 channels) 8 workgroups of 64 x 64, each of
// which stages its 144 reduction elements through LDS step by step with nothing else on its compute unit.  Here the same
// layer is 32 workgroups without a barrier in the reduction: per channel a lane has its nine inputs in flight at once
// and the filter taps come once per wave, and the partial sums meet in LDS in a fixed order.
// Time of a call, general kernel -> this one: 2 x 16 x 16x16, 16 channels, forward 19 -> 8 us, backward-data 29 -> 9 us;
// 4 x 32 x 16x16, 32 channels, 35 -> 9.6 and 55 -> 9.2 us.  60 layers of 2.2e6 to 15.8e6 multiplications (1 to 8 images, 4 to 254
// channels, planes of 4x4 to 63x63): forward 1.02 to 6.4 times faster, backward-data 1.65 to 9.3 times.
#include "sn_internal.h"

namespace sn {
namespace {

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

}  // namespace

bool small3x3_supported(const ConvGeom &g, bool bwd)
{
    if (g.in_bf16 || g.R != 3 || g.S != 3 || g.sh != 1 || g.sw != 1 || g.P < 1 || g.Q < 1) return false;
    const long long M = bwd ? g.C : g.K, red = bwd ? g.K : g.C, npix = (long long)g.N * (bwd ? g.H * (long long)g.W : g.P * (long long)g.Q);
    const long long inputs = (long long)g.N * red * (bwd ? g.P * (long long)g.Q : g.H * (long long)g.W);
    return M * red * npix * 9 <= SMALL3X3_MACS && M <= 65535LL * KO && inputs < (1LL << 31);   // (KO output channels per grid row)
}

hipError_t launch_small3x3(const void *in, const void *w, void *out, const ConvGeom &g, bool bwd, hipStream_t st)
{
    static_assert(KO == WAVES, "wave k finishes output channel k");
    Small3x3 p;
    p.M = bwd ? g.C : g.K;
    p.Red = bwd ? g.K : g.C;
    p.OH = bwd ? g.H : g.P; p.OW = bwd ? g.W : g.Q;
    p.IH = bwd ? g.P : g.H; p.IW = bwd ? g.Q : g.W;
    p.npix = g.N * p.OH * p.OW;
    p.off_h = bwd ? g.ph - 2 : -g.ph;
    p.off_w = bwd ? g.pw - 2 : -g.pw;
    p.w_so = bwd ? 9 : g.C * 9;
    p.w_sr = bwd ? g.C * 9 : 9;
    const dim3 grid((p.npix + 63) / 64, (p.M + KO - 1) / KO), block(64 * WAVES);
    const float *a = static_cast<const float *>(in), *b = static_cast<const float *>(w);
    float *o = static_cast<float *>(out);
    if (bwd) hipLaunchKernelGGL(small3x3_kernel<true>, grid, block, 0, st, a, b, o, p);
    else hipLaunchKernelGGL(small3x3_kernel<false>, grid, block, 0, st, a, b, o, p);
    return hipGetLastError();
}

}  // namespace sn
