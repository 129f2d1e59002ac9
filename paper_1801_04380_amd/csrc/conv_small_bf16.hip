// bf16 3x3 / stride-1 forward and backward-data of small layers (a serving loop's, a few images of a deep stage): one launch, no
// workspace.
//
// What bounds such a layer is the chain of dependent launches and, inside one, of dependent loads: the 0.46 GFLOP of 2 x 256 x
// 14x14, 256 channels, are 0.3 us of the matrix cores.  So a workgroup takes MT output channels x an MT / 4 by 4 patch of outputs
// (MT = 32, or 16 where that would be too few workgroups) and its waves share out the reduction, 16 (32) channels a step; nothing
// is shared before the sums meet in LDS, so the reduction has no barrier:
//   * filter: the lane (row, 8-channel octet) of an MFMA operand is also the owner of a contiguous run of the KCRS tensor, 8
//     channels x 9 taps (forward; backward-data: eight runs of 9 taps): nine 16-byte loads, and every tap's operand is cut out of
//     registers with byte permutes.
//   * input: a lane is one of the patch's pixels with its halo and gathers a step's channels (range-checked: the padding is
//     zeros), which go to the wave's own LDS as 16-byte items; a tap's operand is one 16-byte read at a shifted pixel.
//   * the next step's loads are in flight while one is multiplied.  (142 to 162 registers: 12 waves a compute unit.  At 128, 16
//     waves, the loads in flight spill: 400 layers 1.05 to 1.5 times slower.)
// Neighbouring workgroups are neighbouring channel tiles of one patch: with eight of them each XCD keeps one slice of the filter.
// us a call, the kernels that took these layers before (with 8 MiB of workspace; without) -> this one: 2 x 256 x 14x14, 256 channels,
// forward 17.2 (34.6) -> 7.3, backward-data 17.0 (45) -> 10.1; 1 x 512 x 7x7, 512 channels 24 (65) -> 10.5 and 25 (87) -> 11.2;
// 8 x 16 x 16x16, 16 channels 13 (7.7) -> 3.4 and 13 (7.7) -> 3.6.
#include <algorithm>

#include "conv_tile.h"

namespace sn {
namespace {

constexpr int TH = 4, OCTET = 64 * 16;   // rows of a patch; bytes of 8 channels of it
constexpr int MAXWAVES = 12;
constexpr uint32_t FAR = 0x80000000u;   // an offset outside every tensor: loads bring zeros

struct SmallConv {
    int M, Red;                // output channels, reduction channels
    int IH, IW, OH, OW;
    int off_h, off_w;          // input row / column of output pixel (0, 0)'s first tap
    int mtiles, tiles_w, tiles;   // channel tiles; patches per row of patches, per image
    int out_bf16;
};

// TOGETHER: how the filter is loaded, see below.
template <bool BWD, int MT, bool TOGETHER>
__global__ void __launch_bounds__(64 * MAXWAVES)
small3x3_bf16_kernel(const bf16_t *__restrict__ in, const bf16_t *__restrict__ w, void *__restrict__ out, const SmallConv p)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    constexpr int TW = MT / TH, LW = TW + 2, SLOTS = LW * (TH + 2), NOCT = 64 / MT, RED = 8 * NOCT, NACC = MT * MT / 64;
    const int row = lane % MT, g = lane / MT;
    const int mt = blockIdx.x % p.mtiles, tile = blockIdx.x / p.mtiles;
    const int n = tile / p.tiles, t = tile - n * p.tiles, h0 = t / p.tiles_w * TH, v0 = t % p.tiles_w * TW;
    const int m = mt * MT + row;

    // ---- the wave's loads of one step
    const uint32_t ihw = (uint32_t)p.IH * p.IW * 2;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t *>(in) + (size_t)n * p.Red * p.IH * p.IW, 0, (uint32_t)p.Red * ihw, 0x00020000);
    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(w), 0, (uint32_t)p.M * p.Red * 18, 0x00020000);
    uint32_t xoff;
    {
        const int r = lane / LW, c = lane - r * LW, h = h0 + p.off_h + r, v = v0 + p.off_w + c;
        const bool ok = lane < SLOTS && (unsigned)h < (unsigned)p.IH && (unsigned)v < (unsigned)p.IW;
        xoff = ok ? (uint32_t)(h * p.IW + v) * 2 : FAR;
    }
    // Forward, the lane loads its run, 64 cache lines a load; or (TOGETHER) its neighbours do: of the tile's rows, a step's channels are PPR 16-byte
    // pieces each, neighbouring lanes load neighbouring pieces, 12 lines a load, and the pieces change lanes through LDS.
    constexpr int WCD = BWD ? 40 : 36, PPR = 9 * NOCT;
    uint32_t woff[TOGETHER ? 9 : 1];
    if constexpr (TOGETHER) {
#pragma unroll
        for (int j = 0; j < 9; ++j) {
            const int r = (j * 64 + lane) / PPR, pc = (j * 64 + lane) - r * PPR;
            woff[j] = mt * MT + r < p.M ? (uint32_t)(mt * MT + r) * p.Red * 18 + pc * 16 : FAR;
        }
    }
    struct Step { uint32_t a[WCD]; bf16_t x[RED]; };
    auto load = [&](int c0, Step &s) {
        if constexpr (TOGETHER) {
#pragma unroll
            for (int j = 0; j < 9; ++j) {
                // (a last step of fewer channels: the pieces past them are the next row's)
                const bool in = c0 + RED <= p.Red || ((j * 64 + lane) % PPR) * 16 < (p.Red - c0) * 18;
                const u32x4 d = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wr, in ? woff[j] : FAR, (uint32_t)c0 * 18, 0));
                s.a[4 * j] = d.x; s.a[4 * j + 1] = d.y; s.a[4 * j + 2] = d.z; s.a[4 * j + 3] = d.w;
            }
        } else if constexpr (!BWD) {
            const uint32_t o = m < p.M && c0 + 8 * g < p.Red ? ((uint32_t)m * p.Red + c0 + 8 * g) * 18 : FAR;
#pragma unroll
            for (int j = 0; j < 9; ++j) {
                const u32x4 d = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wr, o + 16 * j, 0, 0));
                s.a[4 * j] = d.x; s.a[4 * j + 1] = d.y; s.a[4 * j + 2] = d.z; s.a[4 * j + 3] = d.w;
            }
        } else {
            const int red0 = c0 + 8 * g;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const bool ok = m < p.M && red0 + i < p.Red;
                const bf16_t *q = w + ((size_t)min(red0 + i, p.Red - 1) * p.M + min(m, p.M - 1)) * 9;
                const u32x4 d = load8_any(q);
                const uint32_t last = q[8];
                s.a[5 * i] = ok ? d.x : 0; s.a[5 * i + 1] = ok ? d.y : 0; s.a[5 * i + 2] = ok ? d.z : 0; s.a[5 * i + 3] = ok ? d.w : 0;
                s.a[5 * i + 4] = ok ? last : 0;
            }
        }
#pragma unroll
        for (int i = 0; i < RED; ++i) {
            const int c = c0 + i;   // (past the last: an offset behind the last channel's, so that FAR stays outside)
            s.x[i] = __builtin_amdgcn_raw_buffer_load_b16(xr, c < p.Red ? xoff : FAR, (uint32_t)min(c, p.Red - 1) * ihw, 0);
        }
    };

    typedef float Acc __attribute__((ext_vector_type(NACC)));
    Acc acc;
#pragma unroll
    for (int v = 0; v < NACC; ++v) acc[v] = 0.f;
    constexpr int FILTER = TOGETHER ? 9 * 1024 : 0;   // bytes of a wave's pieces of the filter
    char *patch = lds + wave * (NOCT * OCTET + FILTER);
    const char *mine = patch + g * OCTET + (row / TW * LW + row % TW) * 16;   // the lane's pixel under tap (0, 0)
    auto multiply = [&](Step &s) {
        if constexpr (TOGETHER) {
#pragma unroll
            for (int j = 0; j < 9; ++j)
                *reinterpret_cast<u32x4 *>(patch + NOCT * OCTET + (j * 64 + lane) * 16) = u32x4{s.a[4 * j], s.a[4 * j + 1], s.a[4 * j + 2], s.a[4 * j + 3]};
        }
#pragma unroll
        for (int h = 0; h < NOCT; ++h) {
            u32x4 d;
#pragma unroll
            for (int j = 0; j < 4; ++j) d[j] = (uint32_t)s.x[8 * h + 2 * j] | (uint32_t)s.x[8 * h + 2 * j + 1] << 16;
            *reinterpret_cast<u32x4 *>(patch + h * OCTET + lane * 16) = d;
        }
        __builtin_amdgcn_wave_barrier();   // (the wave's own LDS, in order: no more than the compiler has to know)
        if constexpr (TOGETHER) {
#pragma unroll
            for (int j = 0; j < 9; ++j) {
                const u32x4 d = *reinterpret_cast<const u32x4 *>(patch + NOCT * OCTET + (row * PPR + g * 9 + j) * 16);
                s.a[4 * j] = d.x; s.a[4 * j + 1] = d.y; s.a[4 * j + 2] = d.z; s.a[4 * j + 3] = d.w;
            }
        }
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            u32x4 a;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                a[j] = BWD ? pick2(s.a, 20 * j + 8 - tap, 20 * j + 18 - tap) : pick2(s.a, 18 * j + tap, 18 * j + 9 + tap);
            const u32x4 b = *reinterpret_cast<const u32x4 *>(mine + ((tap / 3) * LW + tap % 3) * 16);
            if constexpr (MT == 32) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
            else acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
        }
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

    // ---- the waves' sums, in order: register v of a lane is output channel 8 * (v / 4) + 4 * g + v % 4, the lane's pixel
    float *sums = reinterpret_cast<float *>(lds);
    __syncthreads();
#pragma unroll
    for (int v = 0; v < NACC; ++v) sums[(wave * NACC + v) * 64 + lane] = acc[v];
    __syncthreads();
    for (int i = threadIdx.x; i < NACC * 64; i += blockDim.x) {
        float s = sums[i];
        for (int k = 1; k < waves; ++k) s += sums[k * NACC * 64 + i];
        const int v = i >> 6, ln = i & 63, px = ln % MT;
        const int mo = mt * MT + 8 * (v >> 2) + 4 * (ln / MT) + (v & 3), h = h0 + px / TW, q = v0 + px % TW;
        if (mo >= p.M || h >= p.OH || q >= p.OW) continue;
        const size_t o = (((size_t)n * p.M + mo) * p.OH + h) * p.OW + q;
        if (p.out_bf16) static_cast<bf16_t *>(out)[o] = f32_to_bf16(s);
        else static_cast<float *>(out)[o] = s;
    }
}

bool problem_of(const ConvGeom &g, bool bwd, int MT, SmallConv *p)
{
    if (!g.in_bf16 || g.R != 3 || g.S != 3 || g.sh != 1 || g.sw != 1) return false;
    p->M = bwd ? g.C : g.K;
    p->Red = bwd ? g.K : g.C;
    p->OH = bwd ? g.H : g.P; p->OW = bwd ? g.W : g.Q;
    p->IH = bwd ? g.P : g.H; p->IW = bwd ? g.Q : g.W;
    p->off_h = bwd ? g.ph - 2 : -g.ph;
    p->off_w = bwd ? g.pw - 2 : -g.pw;
    const int TW = MT / TH;
    p->mtiles = (p->M + MT - 1) / MT;
    p->tiles_w = (p->OW + TW - 1) / TW;
    p->out_bf16 = g.out_bf16;
    const long long tiles = (long long)p->tiles_w * ((p->OH + TH - 1) / TH);
    // forward: a lane's run of the filter starts on 16 bytes; 32-bit offsets with bit 31 to spare
    if (!bwd && g.C % 8 != 0) return false;
    if ((long long)p->M * p->Red * 18 >= (1LL << 31) || (long long)p->Red * p->IH * p->IW * 2 >= (1LL << 31)) return false;
    if (tiles * g.N * p->mtiles > 0x7fffffffLL) return false;
    p->tiles = (int)tiles;
    return true;
}

// Waves of a workgroup: a compute unit holds twelve, of one workgroup or of several, and a workgroup costs its steps and about one
// more for its start and end.
int steps_of(const SmallConv &p, int MT) { return (p.Red * MT + 511) / 512; }
long long workgroups(const ConvGeom &g, const SmallConv &p) { return (long long)p.tiles * g.N * p.mtiles; }

int waves_of(long long wgs, int steps)
{
    const auto cost = [&](int waves) {
        const unsigned fit = 256 * (MAXWAVES / waves);
        return (unsigned long long)(((unsigned)wgs + fit - 1) / fit) * ((unsigned)(steps + waves - 1) / waves + 1);
    };
    int waves = 1;
    unsigned long long least = cost(1);
    for (int v = 2; v <= std::min(MAXWAVES, steps); ++v) {
        const unsigned long long c = cost(v);
        if (c <= least) {
            least = c;
            waves = v;
        }
    }
    return waves;
}

// us = start + chain * a wave's steps, times the rounds of workgroups + work * steps on the chip + unit * steps on one compute unit + MB written and
// read.  A SIMD holds three of these waves, so that a workgroup of five to seven leaves no place for a second.  6500 layers each (1 to 16 images, 8 to 512
// channels, planes of 4x4 to 64x64, either tile) to 6 to 8 % (rms).
struct Cost { double start, chain, work, unit, out, in; };
const Cost kCost[2][2] = {{{4.62, 0.47, 0.068, 0.142, 0.63, 0.16}, {3.88, 0.20, 0.072, 0.224, 0, 0.465}},    // forward: MT = 32, 16
                          {{4.37, 0.83, 0.082, 0.28, 0.35, 0.06}, {3.77, 0.29, 0.047, 0.403, 0, 0.47}}};   // backward-data

double tile_us(const ConvGeom &g, bool bwd, int MT)
{
    SmallConv p;
    if (!problem_of(g, bwd, MT, &p)) return 1e9;
    const Cost &c = kCost[bwd][MT == 16];
    const long long wgs = workgroups(g, p), each = (wgs + 255) / 256;
    const int steps = steps_of(p, MT), waves = waves_of(wgs, steps);
    const long long fit = 256 * (MAXWAVES / 4 / ((waves + 3) / 4));
    const double out = (p.out_bf16 ? 2e-6 : 4e-6) * g.N * p.M * p.OH * p.OW, in = 2e-6 * g.N * p.Red * p.IH * p.IW;
    return c.start + c.chain * ((wgs + fit - 1) / fit * ((steps + waves - 1) / waves)) + c.work * wgs * steps / 256 + c.unit * each * steps + c.out * out + c.in * in;
}

// Long reductions, whose loads add up, load the filter together; in short ones the way through LDS is what counts (350 layers: up to eight steps
// 0.91 to 1.03 of the speed, from nine on 1.0 to 1.22 times; 2 x 256 x 14x14, 256 channels 8.8 -> 7.3 us).
constexpr int TOGETHER_STEPS = 9;

template <bool BWD, int MT, bool TOGETHER>
hipError_t launch_as(const void *in, const void *w, void *out, const ConvGeom &g, const SmallConv &p, hipStream_t st)
{
    const long long wgs = workgroups(g, p);
    const int waves = waves_of(wgs, steps_of(p, MT));
    // LDS, a wave: its patch (MT = 32: two octets of channels, 16: four) and its pieces of the filter, then its sums (4 KB, 1 KB)
    constexpr int each = std::max(4096, 65536 / MT + (TOGETHER ? 9216 : 0));
    typedef Kernel<small3x3_bf16_kernel<BWD, MT, TOGETHER>> K;
    const hipError_t e = K::enable_lds(MAXWAVES * each);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(K::call, dim3((unsigned)wgs), dim3(64 * waves), waves * each, st, static_cast<const bf16_t *>(in),
                       static_cast<const bf16_t *>(w), out, p);
    return hipGetLastError();
}

template <bool BWD, int MT>
hipError_t launch(const void *in, const void *w, void *out, const ConvGeom &g, hipStream_t st)
{
    SmallConv p;
    if (!problem_of(g, BWD, MT, &p)) return hipErrorInvalidValue;
    if constexpr (!BWD)
        if (steps_of(p, MT) >= TOGETHER_STEPS) return launch_as<BWD, MT, true>(in, w, out, g, p, st);
    return launch_as<BWD, MT, false>(in, w, out, g, p, st);
}

}  // namespace

double small_bf16_us(const ConvGeom &g, bool bwd) { return std::min(tile_us(g, bwd, 32), tile_us(g, bwd, 16)); }

hipError_t launch_small_bf16(const void *in, const void *w, void *out, const ConvGeom &g, bool bwd, hipStream_t st)
{
    const bool wide = tile_us(g, bwd, 32) <= tile_us(g, bwd, 16);
    if (bwd) return wide ? launch<true, 32>(in, w, out, g, st) : launch<true, 16>(in, w, out, g, st);
    return wide ? launch<false, 32>(in, w, out, g, st) : launch<false, 16>(in, w, out, g, st);
}

}  // namespace sn
