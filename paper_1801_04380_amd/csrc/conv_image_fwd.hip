// CONV forward of the image layer -- up to four input channels under a filter of 33 products and more with an even column stride (11x11 / 4,
// 7x7 / 2), up to 96 output channels -- on gfx950, bf16 operands, no workspace (definitions in sn.h).
//
// The reduction is cut into octets: eight neighbouring columns of one filter row of one channel, which under output pixel q are eight
// neighbouring elements of an input row, from q sw on.  So the matrix operand of a pixel is 16 bytes of the input row as it lies in
// memory: nothing is unfolded, transposed or copied.  A workgroup keeps the filter in LDS for its life, as operands, two octets an
// MFMA (columns past the filter's are zeros: 363 of 544 products are real ones for 11x11, 147 of 192 for 7x7), and walks blocks of 512
// output pixels; each of its eight waves takes 64 of them x all output channels.  The input rows of the next block are in registers while
// one is multiplied; results leave through LDS in long runs.
// A zero column meets a real element of x; where that is an Inf or a NaN, and the result so is not finite, the wave does its block again
// with those elements cleared.
// Where it runs: filters of up to 16 columns and at least two rows, strides and filter up to 64, whose operands and the input rows of a block (64 or 32
// columns wide, 8 or 16 rows) fit 160 KB of LDS and 4096 pieces of 16 bytes.  7x7 / 2 and 5x5 / 2 over three channels fit at any width; 11x11 / 4 over three
// at any width up to 64 output channels and, with 65 to 96, on images of up to 238 columns (without padding; 161 792 of 163 840 bytes at 227), over
// four channels of up to 206 and 86.  Wider ones, and more than 96 output channels, are the general kernel's.
// Bound by LDS reads (three operands of the filter and two of pixels for six MFMAs) and, half as long, the results' way out.  us, the
// kernels before it (without workspace; with 512 MiB) -> this: 128 x 3 x 227x227, 96 channels 11x11 / 4 241 (110) -> 79, 32 x 3 x 224x224, 64
// channels 7x7 / 2 80 (78) -> 37.  160 layers of 1 to 4 channels, 8 to 96 output channels, 5x5 to 11x11, batch 1 to 128: 0.57 of their time without
// workspace (at most 1.03), 0.51 with.
#include <algorithm>
#include <type_traits>

#include "sn_internal.h"

namespace sn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int LDS_MAX = 160 * 1024, THREADS = 512, NLD = 8;

struct ImageFwd {
    int C, H, W, K, R, S, sh, sw, ph, pw, P, Q;
    int OS, octets, steps;     // octets of a filter row, of the filter, MFMA steps (two each)
    int rows, pieces, pitch;   // input rows of a block and channel, 16-byte pieces of one, its bytes
    int items;                 // pieces of a block
    int bands, strips, blocks; // blocks down and across an image, of all images
    int x_at;                  // bytes of the filter before the input rows
    int out_pitch;             // bytes of an output channel on its way out
    int out_bf16;
    int x_total, w_total;
    uint32_t last;             // the last octet's byte offset in the block's rows
};

// Eight elements at any address.  A run over an end of the tensor is loaded where it ends with it, and moved when it is stored.
struct __attribute__((packed, aligned(2))) Any { u32x4 v; };
__device__ inline int inside(int off, int total) { return min(max(off, 0), total - 8); }
__device__ inline u32x4 load8(const bf16_t *p, int off, int total) { return reinterpret_cast<const Any *>(p + inside(off, total))->v; }
__device__ inline u32x4 moved(u32x4 v, int off, int total)
{
    const int d = off - inside(off, total);   // the element that the run starts with
    if (__any(d != 0)) {
        unsigned __int128 e;
        __builtin_memcpy(&e, &v, 16);
        e = d > 7 || d < -7 ? 0 : d >= 0 ? e >> 16 * d : e << -16 * d;
        __builtin_memcpy(&v, &e, 16);
    }
    return v;
}

// Elements lo .. hi - 1 of eight, the others zero.
__device__ inline u32x4 keep(u32x4 v, int lo, int hi)
{
#pragma unroll
    for (int j = 0; j < 4; ++j)
        v[j] &= (2 * j >= lo && 2 * j < hi ? 0xffffu : 0u) | (2 * j + 1 >= lo && 2 * j + 1 < hi ? 0xffff0000u : 0u);
    return v;
}

// 16 bytes of LDS that start on AL: one access each, as a 16-byte one at such an address takes a cycle per lane (11x11 / 4: 64 cycles,
// as two of 8 bytes 8).
template <int AL> __device__ inline u32x4 lds16(const char *p)
{
    typedef std::conditional_t<AL == 8, uint64_t, uint32_t> Part;
    const volatile __attribute__((address_space(3))) Part *q = (const volatile __attribute__((address_space(3))) Part *)p;
    Part e[16 / AL];
#pragma unroll
    for (int i = 0; i < 16 / AL; ++i) e[i] = q[i];
    u32x4 v;
    __builtin_memcpy(&v, e, 16);
    return v;
}

// A barrier for what is in LDS: the stores of a block's results stay on their way (__syncthreads would wait for them).
__device__ inline void meet()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// MT 32-channel tiles; CT columns of a block: its 512 pixels are 8 rows of 64 or 16 of 32.
template <int MT, int CT, int AL>
__global__ void __launch_bounds__(THREADS, 2)
image_fwd_kernel(const bf16_t *__restrict__ x, const bf16_t *__restrict__ w, void *__restrict__ y, ImageFwd p)
{
    constexpr int RW = 64 / CT, BR = 8 * RW;   // rows of a wave, of a block
    extern __shared__ __align__(16) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;

    // ---- the filter, as operands: lane (row, octet g) of tile mt in step s
    constexpr int AT_ONCE = 7;
    for (int i0 = tid; i0 < p.steps * MT * 64; i0 += AT_ONCE * THREADS) {
        u32x4 v[AT_ONCE];
        int off[AT_ONCE], n[AT_ONCE];
#pragma unroll
        for (int k = 0; k < AT_ONCE; ++k) {
            const int i = i0 + k * THREADS, ln = i & 63, mt = (i >> 6) % MT, s = (i >> 6) / MT, o = 2 * s + (ln >> 5), m = mt * 32 + (ln & 31);
            const int line = p.OS == 2 ? o >> 1 : o, so = p.OS == 2 ? o & 1 : 0;
            n[k] = m < p.K && o < p.octets ? p.S - 8 * so : 0;
            off[k] = n[k] > 0 ? (m * p.C * p.R + line) * p.S + 8 * so : 0;
            v[k] = load8(w, off[k], p.w_total);
        }
#pragma unroll
        for (int k = 0; k < AT_ONCE; ++k)
            if (i0 + k * THREADS < p.steps * MT * 64)
                reinterpret_cast<u32x4 *>(lds)[i0 + k * THREADS] = keep(moved(v[k], off[k], p.w_total), 0, n[k]);
    }

    struct Block { int n, p0, q0; };
    auto block = [&](int b) {
        const int n = b / (p.bands * p.strips), r = b - n * p.bands * p.strips, band = r / p.strips;
        return Block{n, band * BR, (r - band * p.strips) * CT};
    };
    // the thread's pieces of a block's rows [channel][row][piece]
    u32x4 piece[NLD];
    int rel[NLD];        // its first element from the block's first input element on
    uint32_t to[NLD];    // where in LDS (16 bits), input row of the block (8 bits), piece of the row (8 bits)
#pragma unroll
    for (int k = 0; k < NLD; ++k) {
        const int i = min(tid + THREADS * k, p.items - 1), line = i / p.pieces, j = i - line * p.pieces, c = line / p.rows, r = line - c * p.rows;
        rel[k] = (c * p.H + r) * p.W + 8 * j;
        to[k] = (uint32_t)(line * p.pitch + j * 16) | (uint32_t)r << 16 | (uint32_t)j << 24;
    }
    auto first = [&](const Block &b) { return (b.n * p.C * p.H + b.p0 * p.sh - p.ph) * p.W + b.q0 * p.sw - p.pw; };
    auto fetch = [&](const Block &b) {
        const int at = first(b);
#pragma unroll
        for (int k = 0; k < NLD; ++k)
            if (THREADS * k < p.items) piece[k] = load8(x, at + rel[k], p.x_total);
    };
    auto stash = [&](const Block &b) {
        const int at = first(b), h0 = b.p0 * p.sh - p.ph, v0 = b.q0 * p.sw - p.pw;
#pragma unroll
        for (int k = 0; k < NLD; ++k)
            if (THREADS * k < p.items) {   // (the last piece is written by several threads, the same)
                const int h = h0 + (int)(to[k] >> 16 & 0xff), v = v0 + 8 * (int)(to[k] >> 24);
                *reinterpret_cast<u32x4 *>(lds + p.x_at + (to[k] & 0xffff)) =
                    keep(moved(piece[k], at + rel[k], p.x_total), -v, (unsigned)h < (unsigned)p.H ? p.W - v : 0);
            }
    };

    int b = blockIdx.x;
    if (b >= p.blocks) return;
    Block now = block(b);
    fetch(now);
    stash(now);
    __syncthreads();
    uint32_t base[2];   // the lane's pixel of each of the wave's tiles under octet offset 0
#pragma unroll
    for (int f = 0; f < 2; ++f)
        base[f] = p.x_at + (wave * RW + f / (CT / 32)) * p.sh * p.pitch + ((f % (CT / 32)) * 32 + l32) * p.sw * 2;
    for (;;) {
        const int next = b + gridDim.x;
        const bool more = next < p.blocks;
        const Block then = block(more ? next : b);
        if (more) fetch(then);
        f32x16 acc[MT][2];
        auto accumulate = [&](auto cleared) {
            constexpr bool CLEAR = decltype(cleared)::value;
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int f = 0; f < 2; ++f)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][f][v] = 0.f;
            struct Frags { u32x4 a[MT], b[2]; };
            // the lane's octet of a step: two neighbouring ones of a filter row, or of two filter rows; its row and byte offset, from step to step
            int row = p.OS == 2 ? 0 : g, o = g;
            uint32_t off = p.OS == 2 ? 16 * g : g * p.pitch;
            const int down = p.OS == 2 ? 1 : 2;
            auto read = [&](int s, Frags &r) {
                const uint32_t at = min(off, p.last);
#pragma unroll
                for (int i = 0; i < MT; ++i) r.a[i] = *reinterpret_cast<const u32x4 *>(lds + (s * MT + i) * 1024 + lane * 16);
#pragma unroll
                for (int f = 0; f < 2; ++f) {
                    r.b[f] = lds16<AL>(lds + base[f] + at);
                    if (CLEAR) r.b[f] = keep(r.b[f], 0, o < p.octets ? p.S - (p.OS == 2 ? 8 * g : 0) : 0);
                }
                row += down;
                o += 2;
                off += down * p.pitch;
                if (row >= p.R) { row -= p.R; off += (p.rows - p.R) * p.pitch; }
            };
            auto multiply = [&](const Frags &r) {
#pragma unroll
                for (int f = 0; f < 2; ++f)
#pragma unroll
                    for (int i = 0; i < MT; ++i)
                        acc[i][f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, r.a[i]), __builtin_bit_cast(bf16x8, r.b[f]),
                                                                            acc[i][f], 0, 0, 0);
            };
            if constexpr (CLEAR) {
#pragma unroll 1
                for (int s = 0; s < p.steps; ++s) {
                    Frags f;
                    read(s, f);
                    multiply(f);
                }
                return;
            }
            Frags f0, f1;
            read(0, f0);
            for (int s = 0; s < p.steps; s += 2) {   // (an even number of them)
                read(s + 1, f1);
                __builtin_amdgcn_sched_barrier(0);
                multiply(f0);
                __builtin_amdgcn_sched_barrier(0);
                read(min(s + 2, p.steps - 1), f0);   // (past the last step: not used)
                __builtin_amdgcn_sched_barrier(0);
                multiply(f1);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        accumulate(std::false_type());
        float probe = 0.f;
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            const int h = now.p0 + wave * RW + f / (CT / 32), q = now.q0 + (f % (CT / 32)) * 32 + l32;
            if (h < p.P && q < p.Q) {
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int v = 0; v < 16; ++v) probe = __builtin_fmaf(acc[i][f][v], 0.f, probe);   // NaN from then on
            }
        }
        if (__any(probe != probe)) accumulate(std::true_type());

        // ---- results: register v is output channel 8 * (v / 4) + 4 * g + v % 4 of its tile, the lane is the pixel.  bf16: through
        // LDS, where the input rows were, a tile of 32 channels at a time in two buffers, so that a thread stores eight pixels of a run that is as
        // long as memory has it: a row of the block, or where the block is as wide as the output all of its rows.  (Stored from the
        // registers, one pixel or two a store, they were 40 % of the time.)
        if (p.out_bf16) {
            const int cw = min(CT, p.Q - now.q0), nr = min(BR, p.P - now.p0);
            const bool whole = p.strips == 1;
            const int lp = whole ? cw : CT, len = whole ? nr * cw : cw, ppl = (len + 7) >> 3, per = whole ? ppl : nr * ppl;
            meet();
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                char *buf = lds + p.x_at + (i & 1) * 32 * p.out_pitch;
#pragma unroll
                for (int f = 0; f < 2; ++f) {
                    const int q = (f % (CT / 32)) * 32 + l32;
                    if (q < cw) {
                        char *to = buf + 4 * g * p.out_pitch + ((wave * RW + f / (CT / 32)) * lp + q) * 2;
#pragma unroll
                        for (int v = 0; v < 16; v += 2) {
                            const uint32_t d = f32x2_to_bf16x2(acc[i][f][v], acc[i][f][v + 1]);
                            char *t = to + (8 * (v / 4) + v % 4) * p.out_pitch;
                            *reinterpret_cast<bf16_t *>(t) = (bf16_t)d;
                            *reinterpret_cast<bf16_t *>(t + p.out_pitch) = (bf16_t)(d >> 16);
                        }
                    }
                }
                meet();
                const int channels = min(32, p.K - i * 32);
                for (int t = tid; t < channels * per; t += THREADS) {
                    const int ch = t / per, rest = t - ch * per, line = whole ? 0 : rest / ppl, j = rest - line * ppl, n = min(8, len - 8 * j);
                    const u32x4 d = *reinterpret_cast<const u32x4 *>(buf + ch * p.out_pitch + line * lp * 2 + j * 16);
                    bf16_t *o = static_cast<bf16_t *>(y) + (((size_t)now.n * p.K + i * 32 + ch) * p.P + now.p0 + line) * p.Q + now.q0 + 8 * j;
                    if (n == 8) {
                        reinterpret_cast<Any *>(o)->v = d;
                    } else {
#pragma unroll
                        for (int e = 0; e < 7; ++e)
                            if (e < n) o[e] = (bf16_t)(d[e >> 1] >> (16 * (e & 1)));
                    }
                }
            }
        } else {
            uint32_t PQ = (uint32_t)p.P * p.Q;
            asm volatile("" : "+s"(PQ));   // (the channels' places are made here, not kept in registers from block to block)
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                const int h = now.p0 + wave * RW + f / (CT / 32), q = now.q0 + (f % (CT / 32)) * 32 + l32;
                if (h >= p.P || q >= p.Q) continue;
                const uint32_t mine = (4 * g * PQ + (uint32_t)h * p.Q + q) * 4;
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int m = i * 32 + 8 * (v / 4) + v % 4;
                        char *o = static_cast<char *>(y) + ((size_t)now.n * p.K + m) * PQ * 4;
                        if (m + 4 * g < p.K) *reinterpret_cast<float *>(o + mine) = acc[i][f][v];
                    }
            }
        }
        if (!more) break;
        meet();
        stash(then);
        meet();
        b = next;
        now = then;
    }
}

struct Launch { ImageFwd p; int mt, ct, lds; };

bool make_problem(const ConvGeom &g, int ct, Launch *l)
{
    ImageFwd &p = l->p;
    if (!g.in_bf16 || (long long)g.N * g.C * g.H * g.W < 8 || (long long)g.K * g.C * g.R * g.S < 8 || g.C > 4 || g.K > 96 || g.sw % 2 != 0 || g.R * g.S * g.C <= 32) return false;
    p.C = g.C; p.H = g.H; p.W = g.W; p.K = g.K; p.R = g.R; p.S = g.S; p.sh = g.sh; p.sw = g.sw; p.ph = g.ph; p.pw = g.pw; p.P = g.P; p.Q = g.Q;
    p.out_bf16 = g.out_bf16;
    if (g.R > 64 || g.S > 64 || g.sh > 64 || g.sw > 64) return false;
    p.OS = (g.S + 7) / 8;
    p.octets = g.C * g.R * p.OS;
    p.steps = (p.octets + 3) / 4 * 2;
    if (p.OS > 2 || g.R < 2) return false;
    const int br = 512 / ct;
    l->ct = ct;
    l->mt = (g.K + 31) / 32;
    p.rows = (br - 1) * g.sh + g.R;
    // (an only strip is as wide as the output; the lanes past it read what follows in LDS, and write nothing)
    p.pieces = ((std::min(ct, g.Q) - 1) * g.sw + 8 * p.OS + 7) / 8;
    p.pitch = p.pieces * 16;
    p.items = p.C * p.rows * p.pieces;
    p.x_at = p.steps * l->mt * 1024;
    p.out_pitch = (br * std::min(ct, g.Q) * 2 + 15) / 16 * 16 + 16;
    l->lds = p.x_at + std::max(p.C * p.rows * p.pitch + (ct - std::min(ct, g.Q)) * g.sw * 2, 64 * p.out_pitch);
    if (p.items > THREADS * NLD || l->lds > LDS_MAX || p.C * p.rows * p.pitch > 0xffff) return false;
    p.last = (uint32_t)(((g.C - 1) * p.rows + g.R - 1) * p.pitch + (p.OS - 1) * 16);
    p.bands = (g.P + br - 1) / br;
    p.strips = (g.Q + ct - 1) / ct;   // (more than one: CT columns wide all the same, see out_pitch)
    const long long blocks = (long long)p.bands * p.strips * g.N;
    if (blocks > 0x3fffffff) return false;
    p.blocks = (int)blocks;
    // 32-bit element numbers, over either end too; an input row of a block in 8 bits, five planes of y in 32
    const long long xn = (long long)g.N * g.C * g.H * g.W, beyond = (long long)(p.rows + g.ph + 1) * g.W + p.pieces * 8LL + g.pw;
    if (xn + beyond > 0x70000000LL || p.rows > 256 || p.pieces > 256 || (long long)g.P * g.Q > 1 << 27) return false;
    p.x_total = (int)xn;
    p.w_total = g.K * g.C * g.R * g.S;
    return true;
}

int rounds(const Launch &l) { return (l.p.blocks + 255) / 256; }

// Blocks 64 or 32 columns wide: whichever takes fewer rounds of the chip (of 160 layers 0.05 % slower than the better one).
bool choose(const ConvGeom &g, Launch *l)
{
    Launch narrow;
    const bool n = make_problem(g, 32, &narrow);
    if (!make_problem(g, 64, l)) {
        *l = narrow;
        return n;
    }
    if (n && rounds(narrow) < rounds(*l)) *l = narrow;
    return true;
}

}  // namespace

// Of the 160 layers above to 8 % (rms).
double image_fwd_us(const ConvGeom &g)
{
    Launch l;
    if (!choose(g, &l)) return 1e9;
    return 2.9 + rounds(l) * (2.0 + (0.09 * l.p.steps + 1.3) * l.mt + 0.46 * l.p.items / THREADS);
}

hipError_t launch_image_fwd(const void *x, const void *w, void *y, const ConvGeom &g, hipStream_t st)
{
    Launch l;
    if (!choose(g, &l)) return hipErrorInvalidValue;
    auto go = [&](auto kern) -> hipError_t {
        const hipError_t attr = kern.enable_lds(LDS_MAX);
        if (attr != hipSuccess) return attr;
        hipLaunchKernelGGL(kern.call, dim3(std::min(256, l.p.blocks)), dim3(THREADS), l.lds, st, static_cast<const bf16_t *>(x),
                           static_cast<const bf16_t *>(w), y, l.p);
        return hipGetLastError();
    };
#define SN_IMGF(MT_, CT_) (g.sw % 4 == 0 ? go(Kernel<image_fwd_kernel<MT_, CT_, 8>>()) : go(Kernel<image_fwd_kernel<MT_, CT_, 4>>()))
    if (l.ct == 64) return l.mt == 3 ? SN_IMGF(3, 64) : l.mt == 2 ? SN_IMGF(2, 64) : SN_IMGF(1, 64);
    return l.mt == 3 ? SN_IMGF(3, 32) : l.mt == 2 ? SN_IMGF(2, 32) : SN_IMGF(1, 32);
#undef SN_IMGF
}

}  // namespace sn
