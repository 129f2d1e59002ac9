// Kernels of the channels-last implicit GEMM; see conv_chlast.h.
#pragma once
#include <type_traits>
#include "conv_chlast.h"

namespace sn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr uint32_t OUTSIDE = 0x80000000u;   // an offset past any copy: loads bring zeros

// Two fp32 -> two bf16, round to nearest even, a in the low half.
__device__ inline uint32_t pack2(float a, float b)
{
    f32x2 f = {a, b};
    bf16x2 h = __builtin_convertvector(f, bf16x2);
    uint32_t r;
    __builtin_memcpy(&r, &h, 4);
    return r;
}

__device__ inline i32x4 make_rsrc(const void *p, uint32_t bytes)
{
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    i32x4 r = {(int)(uint32_t)a, (int)(uint32_t)(a >> 32), (int)bytes, 0x00020000};
    return r;
}

// 16 bytes per lane from the buffer straight into LDS: lane l's at lds + 16 * l.  In assembly, so that the compiler
// neither counts these loads nor waits for them before LDS reads that do not depend on them: stage_wait does.  (m0 is one
// of the registers that the compiler reserves: that it is not preserved here, which it warns of, is what the clobber says.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ inline void load_lds16(uint32_t lds, uint32_t voff, i32x4 rsrc, uint32_t soff)
{
    asm volatile("s_mov_b32 m0, %0\n\t"
                 "s_nop 0\n\t"
                 "buffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
}
#pragma clang diagnostic pop

// All but the last N of the wave's loads have landed and its LDS reads are done; then the workgroup's barrier.
template <int N>
__device__ inline void stage_wait()
{
    static_assert(N >= 0 && N < 64, "the counter has six bits");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));   // vmcnt(N) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The wave's LDS reads are done (said in a form the compiler counts with: it would wait for later reads as well).
__device__ inline void reads_done() { __builtin_amdgcn_s_waitcnt(0xc07f); }   // lgkmcnt(0)

__device__ inline uint32_t lds_address(const void *p)
{
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)p;
}

// Whether any thread of the workgroup holds an accumulator that is not finite.  `word` is LDS that nobody needs any more (of
// the ring: a word beside it would cost the tiles that take half of a compute unit's LDS their second workgroup).
template <int M, int N>
__device__ inline bool any_not_finite(const f32x16 (&acc)[M][N], char *word)
{
    volatile int *found = reinterpret_cast<volatile int *>(word);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < M; ++i)
#pragma unroll
        for (int f = 0; f < N; ++f)
#pragma unroll
            for (int v = 0; v < 16; ++v) s = __builtin_fmaf(acc[i][f][v], 0.f, s);   // NaN from then on
    __syncthreads();
    if (threadIdx.x == 0) *found = 0;
    __syncthreads();
    if (s != s) *found = 1;
    __syncthreads();
    const bool any = *found;
    __syncthreads();
    return any;
}

// ---- preparation: the channels-last copies and the packed filter ---------------------------------------------
template <typename T> struct Elem;
template <> struct Elem<bf16_t> { static constexpr int PE = 8; };   // elements per 16-byte piece
template <> struct Elem<float> { static constexpr int PE = 4; };

// One workgroup: 64 pixels of the copy x 128 bytes of channels.  A lane gathers one pixel's channels (consecutive
// lanes: consecutive pixels, so every channel's read is one run), packs them into 16-byte pieces in LDS, and the
// pieces go out as 128-byte rows.  Bound by memory: one read and one write of the tensor.
template <typename T>
__device__ void stage_block(const ClStage &s, int blk, char *lds)
{
    constexpr int PE = Elem<T>::PE;
    const T *src = static_cast<const T *>(s.src);
    T *dst = static_cast<T *>(s.dst);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int HpWs = s.Hp * s.Ws;
    int pt = blk % s.ptiles, rest = blk / s.ptiles;
    if (s.Cp <= PE) {   // few channels: a pixel is one store of Cp elements, no transposition
        const int pix = pt * 256 + tid, n = rest % s.nimg, a = rest / s.nimg;
        if (pix >= HpWs) return;
        const int i = pix / s.Ws, w = pix - i * s.Ws - s.pl, h = i * s.sh + a - s.pt;
        const bool in = (unsigned)h < (unsigned)s.H && (unsigned)w < (unsigned)s.W;
        const T *q = src + ((size_t)n * s.C * s.H + h) * s.W + w;
        T v[PE];
#pragma unroll
        for (int c = 0; c < PE; ++c) v[c] = (in && c < s.C) ? q[(size_t)c * s.H * s.W] : T(0);
        T *o = dst + ((size_t)rest * HpWs + pix) * s.Cp;
        if (s.Cp * sizeof(T) == 8) {
            u32x2 d;
            __builtin_memcpy(&d, v, 8);
            *reinterpret_cast<u32x2 *>(o) = d;
        } else {
            u32x4 d;
            __builtin_memcpy(&d, v, 16);
            *reinterpret_cast<u32x4 *>(o) = d;
        }
        return;
    }
    const int ct = rest % s.ctiles;
    rest /= s.ctiles;                       // phase * nimg + image
    const int n = rest % s.nimg, a = rest / s.nimg;
    const int pieces = min(8, s.Cp / PE - ct * 8);
    {
        const int pix = pt * 64 + lane;
        const int i = pix / s.Ws, w = pix - i * s.Ws - s.pl, h = i * s.sh + a - s.pt;
        const bool in = pix < HpWs && (unsigned)h < (unsigned)s.H && (unsigned)w < (unsigned)s.W;
        // range-checked loads: pixels outside the image and channels past the last bring zeros, and all 16 (8) loads
        // of a thread are on their way together.  (An image of less than 2 GiB: the plans see to it.  A channel past the
        // last reads behind the last channel's scalar offset, so that a lane's OUTSIDE never comes back into range.)
        const uint32_t HW = (uint32_t)s.H * s.W * sizeof(T);
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<T *>(src) + (size_t)n * s.C * s.H * s.W, 0, (uint32_t)s.C * HW, 0x00020000);
        const uint32_t v0 = in ? (uint32_t)(h * s.W + w) * sizeof(T) : OUTSIDE;
        T v[2][PE];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int c0 = (ct * 8 + wave + 4 * k) * PE;
#pragma unroll
            for (int c = 0; c < PE; ++c) {
                const uint32_t vo = c0 + c < s.C ? v0 : OUTSIDE, so = (uint32_t)min(c0 + c, s.C - 1) * HW;
                if constexpr (sizeof(T) == 2) v[k][c] = (T)__builtin_amdgcn_raw_buffer_load_b16(rs, vo, so, 0);
                else v[k][c] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, vo, so, 0));
            }
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int pc = wave + 4 * k;
            u32x4 d;
            __builtin_memcpy(&d, v[k], 16);
            if (pc < pieces) *reinterpret_cast<u32x4 *>(lds + lane * 128 + ((pc ^ (lane & 7)) * 16)) = d;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int px = (tid >> 3) + 32 * k, pc = tid & 7;
        if (pc < pieces && pt * 64 + px < HpWs) {
            const u32x4 d = *reinterpret_cast<const u32x4 *>(lds + px * 128 + ((pc ^ (px & 7)) * 16));
            *reinterpret_cast<u32x4 *>(dst + ((size_t)rest * HpWs + pt * 64 + px) * s.Cp + (ct * 8 + pc) * PE) = d;
        }
    }
}

// One 16-byte piece of the packed filter per thread.
template <typename T>
__device__ void pack_block(const ClPack &k, int blk)
{
    constexpr int PE = Elem<T>::PE;
    const int it = blk * 256 + threadIdx.x;
    if (it >= k.pieces) return;
    int ci = 0;
    while (ci + 1 < k.ncls && it >= k.cls[ci + 1].piece0) ++ci;
    const ClPackClass c = k.cls[ci];
    int q = it - c.piece0, m, pr, t;     // output channel, piece of the row, row tap
    const int ppr = c.ncks * 8;
    if (k.mfast) { m = q % k.Mpad; q /= k.Mpad; pr = q % ppr; t = q / ppr; }
    else { pr = q % ppr; q /= ppr; t = q % c.Rt; m = q / c.Rt; }
    const int r = c.r0 + t * c.rstep;
    const T *w = static_cast<const T *>(k.w);
    T v[PE];
    int s = pr * PE / k.Cp, ch = pr * PE - s * k.Cp;
#pragma unroll
    for (int e = 0; e < PE; ++e) {
        const bool ok = m < k.M && s < c.St && ch < k.Red;
        v[e] = ok ? w[(size_t)m * k.w_sm + (size_t)ch * k.w_sr + r * k.S + c.s0 + s * c.sstep] : T(0);
        if (++ch == k.Cp) { ch = 0; ++s; }
    }
    u32x4 d;
    __builtin_memcpy(&d, v, 16);
    const int ck = pr / 8, stage = (ck % c.no * c.Rt + t) * c.ni + ck / c.no;
    char *o = static_cast<char *>(k.dst) + c.a_off + ((size_t)stage * k.Mpad + m) * 128 + (pr & 7) * 16;
    *reinterpret_cast<u32x4 *>(o) = d;
}

template <typename T>
__global__ void __launch_bounds__(256) cl_prep_kernel(ClPrep p)
{
    __shared__ __attribute__((aligned(16))) char lds[64 * 128];
    int b = blockIdx.x;
    if (b < p.pk.blocks) { pack_block<T>(p.pk, b); return; }
    b -= p.pk.blocks;
    if (b < p.st[0].blocks) { stage_block<T>(p.st[0], b, lds); return; }
    b -= p.st[0].blocks;
    if (b < p.st[1].blocks) { stage_block<T>(p.st[1], b, lds); return; }
    b -= p.st[1].blocks;
    int it = b * 256 + threadIdx.x;
    const int first = it < p.zero_items[0] ? 0 : 1;
    if (first) it -= p.zero_items[0];
    if (it < p.zero_items[first]) static_cast<u32x4 *>(p.zero[first])[it] = u32x4{0, 0, 0, 0};
}

// ---- forward and backward-data -------------------------------------------------------------------------------
// BM output channels x BN pixels per workgroup of WM x WN waves; NST stages of 128-byte runs.
// HALF: the runs are an odd number of 4-channel pixels (bf16) and end half way through a 16-byte piece, whose other half is
// the next pixel's.  It meets packed zeros, which is enough unless it is an Inf or a NaN: a tile with a result that is not
// finite is done again with that half cleared (the look at the results costs such layers 1 %, clearing it always 4 %).
template <typename T, int BM, int BN, int WM, int WN, int NST, bool HALF = false>
__global__ void __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(2)))
cl_gemm_kernel(const T *__restrict__ xs, const T *__restrict__ ap, void *__restrict__ y, float *__restrict__ part, ClGemm p)
{
    constexpr int NW = WM * WN, FM = BM / WM / 32, FN = BN / WN / 32;
    constexpr int STG = (BM + BN) * 128;
    constexpr int IA = BM / 8, IB = BN / 8;                       // load instructions per stage
    constexpr int LA = (IA + NW - 1) / NW, LB = IB / NW, LMIN = IA / NW + LB;
    static_assert(IB % NW == 0 && BM % (WM * 32) == 0 && BN % (WN * 32) == 0, "tile");
    extern __shared__ __attribute__((aligned(16))) char lds[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    const int wm = wave % WM, wn = wave / WM;

    // ---- which tile: an XCD (every eighth workgroup) takes a contiguous range of pixel tiles, all channel tiles of one in a row
    const int id = blockIdx.x, xcd = id & 7, slot = id >> 3;
    const int ptl = slot / p.mtiles, mtile = slot - ptl * p.mtiles, ptile = xcd * p.ppx + ptl;
    if (ptile >= p.ptiles) return;
    int ci = 0;
    while (ci + 1 < p.ncls && ptile >= p.cls[ci + 1].tile0) ++ci;
    const ClClass c = p.cls[ci];
    const int m0 = mtile * BM, j0 = (ptile - c.tile0) * BN;

    const i32x4 xr = make_rsrc(xs, p.x_bytes), ar = make_rsrc(ap, p.a_bytes);
    const int psz = p.Cp * (int)sizeof(T);

    // ---- per-lane offsets of the loads: 8 rows of eight pieces per instruction, pieces permuted
    const int lrow = lane >> 3, lpiece = (lane & 7) ^ ((wave & 1) * 4 + (lane >> 4));
    static_assert(NW % 2 == 0, "an instruction's rows keep their parity of eights");
    uint32_t va[LA], vb[LB];
#pragma unroll
    for (int k = 0; k < LA; ++k) va[k] = (uint32_t)(m0 + (wave + NW * k) * 8 + lrow) * 128u + lpiece * 16u;
    const int nimg = c.nh * c.nw;
#pragma unroll
    for (int k = 0; k < LB; ++k) {
        const int j = j0 + (wave + NW * k) * 8 + lrow;
        const int n = j / nimg, rem = j - n * nimg, i = rem / c.nw, w = rem - i * c.nw;
        const uint32_t o = ((uint32_t)(n * p.Hp + i + c.x_row) * p.Ws + w * p.in_sw + c.x_col) * psz + lpiece * 16u;
        vb[k] = j < c.npix ? o : OUTSIDE;
    }
    const uint32_t tailmask = lpiece >= c.tail ? OUTSIDE : 0u;

    const int nsteps = c.Rt * c.ncks;
    int s0 = 0, s1 = nsteps;
    if (p.nsplit > 1) {
        const int per = (nsteps + p.nsplit - 1) / p.nsplit;
        s0 = min((int)blockIdx.y * per, nsteps);
        s1 = min(s0 + per, nsteps);
    }
    const int n = s1 - s0;

    f32x16 acc[FM][FN];
    // operand reads: row l32 of a 32-row block, piece 2t + g of eight, permuted as stored
    const uint32_t ra = (wm * FM * 32 + l32) * 128, rb = BM * 128 + (wn * FN * 32 + l32) * 128;
    const uint32_t q0 = (uint32_t)(g ^ ((l32 >> 1) & 7)) * 16;   // piece 2t + g is at q0 ^ 32 t

    // operands of half a stage (four pieces)
    struct Frags { u32x4 a[2][FM], b[2][FN]; };
    auto fetch = [&](int buf, int half, Frags &r) {
        const char *base = lds + buf * STG;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint32_t q = q0 ^ (uint32_t)(half * 64 + t * 32);
            const char *pa = base + ra + q, *pb = base + rb + q;
#pragma unroll
            for (int i = 0; i < FM; ++i) r.a[t][i] = *reinterpret_cast<const u32x4 *>(pa + i * 4096);
#pragma unroll
            for (int f = 0; f < FN; ++f) r.b[t][f] = *reinterpret_cast<const u32x4 *>(pb + f * 4096);
        }
    };
    auto clear_tail = [&](int half, Frags &r) {   // the second half of the run's last piece
#pragma unroll
        for (int t = 0; t < 2; ++t)
            if (half * 4 + 2 * t + g == c.tail - 1)
#pragma unroll
                for (int f = 0; f < FN; ++f) r.b[t][f][2] = r.b[t][f][3] = 0;
    };
    auto multiply = [&](const Frags &r) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if constexpr (sizeof(T) == 2) {
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int f = 0; f < FN; ++f)
                        acc[i][f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, r.a[t][i]),
                                                                            __builtin_bit_cast(bf16x8, r.b[t][f]), acc[i][f], 0, 0, 0);
            } else {
                // four products of k = {element e of piece 2t, element e of piece 2t + 1}
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < FM; ++i)
#pragma unroll
                        for (int f = 0; f < FN; ++f)
                            acc[i][f] = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(f32x4, r.a[t][i])[e],
                                                                             __builtin_bit_cast(f32x4, r.b[t][f])[e], acc[i][f], 0, 0, 0);
            }
        }
    };

    auto accumulate = [&](auto clear) {
        constexpr bool CUT = decltype(clear)::value;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int f = 0; f < FN; ++f)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][f][v] = 0.f;

        // ---- the running position of the loads: channel block, row tap, run within it
        const int ni = max(c.ni, 1), per_block = max(c.Rt * ni, 1);
        int co = s0 / per_block, tap = (s0 - co * per_block) / ni, ri = s0 - co * per_block - tap * ni;
        int mo = co, mleft = per_block - (s0 - co * per_block);   // and of the multiplications: block, stages left in it
        int plane = tap % p.sh;
        const uint32_t rowb = (uint32_t)p.Ws * psz;
        uint32_t prow = (uint32_t)(tap / p.sh) * rowb;
        uint32_t asoff = c.a_off + (uint32_t)s0 * p.Mpad * 128u;
        const uint32_t lbase = lds_address(lds);
        auto issue = [&](int buf) {
            const uint32_t lb = lbase + buf * STG + wave * 1024;
            const int ck = ri * c.no + co;
            const uint32_t xsoff = plane * p.plane_bytes + prow + ck * 128u;
            const uint32_t tm = ck == c.ncks - 1 ? tailmask : 0u;
#pragma unroll
            for (int k = 0; k < LA; ++k)
                if (IA % NW == 0 || wave + NW * k < IA) load_lds16(lb + k * NW * 1024, va[k], ar, asoff);
#pragma unroll
            for (int k = 0; k < LB; ++k) load_lds16(lb + IA * 1024 + k * NW * 1024, vb[k] | tm, xr, xsoff);
            asoff += p.Mpad * 128u;
            if (++ri == ni) {
                ri = 0;
                if (++plane == p.sh) { plane = 0; prow += rowb; }
                if (++tap == c.Rt) { tap = 0; plane = 0; prow = 0; ++co; }
            }
        };

        // Trip i, two halves: the second half of stage i is read while the first is multiplied; then, when stage i + 1
        // has landed and everybody has read stage i, its buffer takes stage i + NST, and the first half of stage i + 1 is
        // read while the second of stage i is multiplied (unless the run ends in the first half).
        Frags f0, f1;
        for (int i = 0; i < NST && i < n; ++i) issue(i);
        if (n >= NST) stage_wait<(NST - 1) * LMIN>();
        else stage_wait<0>();
        fetch(0, 0, f0);
        int buf = 0;
        for (int i = 0; i < n; ++i) {
            const bool both = c.tail > 4 || mo != c.no - 1;   // (a short run is its block's only one)
            const bool cut = CUT && mo == c.no - 1;
            if (--mleft == 0) { mleft = per_block; ++mo; }
            reads_done();
            fetch(buf, 1, f1);
            __builtin_amdgcn_sched_barrier(0);
            if (cut) clear_tail(0, f0);
            multiply(f0);
            __builtin_amdgcn_sched_barrier(0);
            if (i + NST - 1 < n) stage_wait<(NST - 2) * LMIN>();
            else stage_wait<0>();
            const int free = buf;
            buf = buf + 1 == NST ? 0 : buf + 1;
            fetch(buf, 0, f0);   // (past the last stage: whatever is there, not used)
            if (i + NST < n) issue(free);
            __builtin_amdgcn_sched_barrier(0);
            if (cut) clear_tail(1, f1);
            if (both) multiply(f1);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    accumulate(std::false_type());
    if constexpr (HALF)
        if (any_not_finite(acc, lds)) accumulate(std::true_type());

    // ---- epilogue: register v is output channel 8 * (v / 4) + 4 * g + v % 4 of its block, the lane is the pixel
    const size_t OHW = (size_t)p.OH * p.OW;
#pragma unroll
    for (int f = 0; f < FN; ++f) {
        const int j = j0 + (wn * FN + f) * 32 + l32;
        const bool ok = j < c.npix;
        if (p.nsplit > 1) {
            float *o = part + ((size_t)blockIdx.y * p.M) * p.nptot + j;
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int m = m0 + (wm * FM + i) * 32 + 8 * (v / 4) + 4 * g + v % 4;
                    if (ok && m < p.M) o[(size_t)m * p.nptot] = acc[i][f][v];
                }
            continue;
        }
        const int nn = j / nimg, rem = j - nn * nimg, ii = rem / c.nw, ww = rem - ii * c.nw;
        const size_t base = (size_t)nn * p.M * OHW + (size_t)(c.oh0 + ii * p.osh) * p.OW + c.ow0 + ww * p.osw;
        if (p.pair) {   // bf16, neighbouring lanes are neighbouring pixels of one image: lane pairs trade halves
            const int odd = lane & 1;
            bf16_t *o = static_cast<bf16_t *>(y) + base - odd;
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int v = 0; v < 16; v += 2) {
                    const int m = m0 + (wm * FM + i) * 32 + 8 * (v / 4) + 4 * g + v % 4 + odd;
                    const float send = odd ? acc[i][f][v] : acc[i][f][v + 1];
                    const float got = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(send), 0xB1, 0xf, 0xf, true));
                    const uint32_t d = odd ? pack2(got, acc[i][f][v + 1]) : pack2(acc[i][f][v], got);
                    if (ok && m < p.M) *reinterpret_cast<uint32_t *>(o + (size_t)m * OHW) = d;
                }
        } else if (p.out_bf16) {
            bf16_t *o = static_cast<bf16_t *>(y) + base;
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int m = m0 + (wm * FM + i) * 32 + 8 * (v / 4) + 4 * g + v % 4;
                    if (ok && m < p.M) o[(size_t)m * OHW] = (bf16_t)pack2(acc[i][f][v], 0.f);
                }
        } else {
            float *o = static_cast<float *>(y) + base;
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int m = m0 + (wm * FM + i) * 32 + 8 * (v / 4) + 4 * g + v % 4;
                    if (ok && m < p.M) o[(size_t)m * OHW] = acc[i][f][v];
                }
        }
    }
}

// y[n][m][px] = sum over the slices, in order (one class, whole planes).
template <bool BF16>
__global__ void __launch_bounds__(256) cl_reduce_kernel(const float *__restrict__ part, void *__restrict__ y, int M, int npix,
                                                        int OHW, int nsplit)
{
    const int j = blockIdx.x * 256 + threadIdx.x, m = blockIdx.y;
    if (j >= npix) return;
    const float *q = part + (size_t)m * npix + j;
    const size_t pitch = (size_t)M * npix;
    float s = 0.f;
    for (int z = 0; z < nsplit; ++z) s += q[z * pitch];
    const int n = j / OHW, px = j - n * OHW;
    const size_t o = ((size_t)n * M + m) * OHW + px;
    if (BF16) static_cast<bf16_t *>(y)[o] = (bf16_t)pack2(s, 0.f);
    else static_cast<float *>(y)[o] = s;
}

// ---- backward-filter -----------------------------------------------------------------------------------------
// BM output channels x BN columns (r, s, c) per workgroup; stages of 32 flat pixels (16 for fp32).
// Where the copies' pitch leaves flat pixels that are no output pixel (p.holes), dy is zero, but x may hold a real pixel there.
// Zero products, unless that pixel is an Inf or a NaN: a tile with a result that is not finite is done again without x's
// loads at such pixels (the look at the results costs 1 %, leaving them out always 9 to 18 %).
template <typename T, int BM, int BN, int WM, int WN, int NST>
__global__ void __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(2)))
cl_wgrad_kernel(const T *__restrict__ ds, const T *__restrict__ xs, float *__restrict__ part, ClWgrad p)
{
    constexpr int NW = WM * WN, FM = BM / WM / 32, FN = BN / WN / 32;
    constexpr int SZ = sizeof(T), PE = 16 / SZ, PIX = SZ == 2 ? 32 : 16;
    constexpr int PA = BM / PE, PB = BN / PE;                     // pieces per row
    constexpr int STG = PIX * (BM + BN) * SZ;
    constexpr int IA = PIX * PA / 64, IB = PIX * PB / 64;         // load instructions per stage
    constexpr int LA = (IA + NW - 1) / NW, LB = (IB + NW - 1) / NW, LMIN = IA / NW + IB / NW;
    static_assert(PIX * PA % 64 == 0 && PIX * PB % 64 == 0, "tile");
    extern __shared__ __attribute__((aligned(16))) char lds[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    const int wm = wave % WM, wn = wave / WM;

    // ---- which tile: the tiles of one slice on one XCD, so that the slice's pixels come from memory once
    const int tiles = p.ktiles * p.jtiles;
    int slice, tile;
    if (p.nsl % 8 == 0) {
        const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
        slice = (slot / tiles) * 8 + xcd;
        tile = slot % tiles;
    } else {
        slice = blockIdx.x / tiles;
        tile = blockIdx.x % tiles;
    }
    const int kt = tile % p.ktiles, jt = tile / p.ktiles;
    const int k0 = kt * BM, c0 = jt * BN;

    const i32x4 dr = make_rsrc(ds, p.d_bytes), xr = make_rsrc(xs, p.x_bytes);

    // the XOR that spreads the rows of a transposing read over the banks
    auto perm = [](int row, int pieces) { return SZ == 4 || (pieces & (pieces - 1)) ? 0 : pieces >= 16 ? (row & 3) * 4 : (row & 3) * 2; };
    uint32_t va[LA], vb[LB];
#pragma unroll
    for (int k = 0; k < LA; ++k) {
        const int it = (wave + NW * k) * 64 + lane, row = it / PA, piece = (it % PA) ^ perm(row, PA);
        const int kk = k0 + piece * PE;
        va[k] = kk < p.Kp ? (uint32_t)(row * p.Kp + kk) * SZ : OUTSIDE;
    }
#pragma unroll
    for (int k = 0; k < LB; ++k) {
        const int it = (wave + NW * k) * 64 + lane, row = it / PB, piece = (it % PB) ^ perm(row, PB);
        const int col = c0 + piece * PE, r = col / p.SC, rem = col - r * p.SC;
        const uint32_t o = (uint32_t)(r % p.sh) * p.plane_bytes +
                           ((uint32_t)(r / p.sh) * p.Ws * p.Cp + rem + (uint32_t)row * p.in_sw * p.Cp) * SZ;
        vb[k] = col < p.ncols ? o : OUTSIDE;
    }
    const int s0 = slice * p.sps, n = min(p.sps, p.steps - s0);
    const uint32_t dstep = (uint32_t)PIX * p.Kp * SZ, xstep = (uint32_t)PIX * p.in_sw * p.Cp * SZ;
    const uint32_t lbase = lds_address(lds);
    f32x16 acc[FM][FN];
    // operand reads.  bf16: lane i of 16 addresses row i / 4, columns 4 * (i % 4) .. + 3 and receives column i of the
    // four rows; rows 8g .. 8g + 3 and the four after them make the eight reduction elements of the lane's column.
    uint32_t ra[FM], rb[FN];
    const int i16 = lane & 15, half = (lane >> 4) & 1;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        const int blk = (wm * FM + i) * 32;
        if (SZ == 2) {
            const int row = 8 * g + (i16 >> 2), piece = blk / 8 + 2 * half + ((i16 & 3) >> 1);
            ra[i] = row * (BM * SZ) + ((piece ^ perm(row, PA)) * 16) + (i16 & 1) * 8;
        } else {
            ra[i] = g * (BM * SZ) + (blk + l32) * 4;
        }
    }
#pragma unroll
    for (int f = 0; f < FN; ++f) {
        const int blk = (wn * FN + f) * 32;
        if (SZ == 2) {
            const int row = 8 * g + (i16 >> 2), piece = blk / 8 + 2 * half + ((i16 & 3) >> 1);
            rb[f] = PIX * BM * SZ + row * (BN * SZ) + ((piece ^ perm(row, PB)) * 16) + (i16 & 1) * 8;
        } else {
            rb[f] = PIX * BM * SZ + g * (BN * SZ) + (blk + l32) * 4;
        }
    }
    auto tr8 = [](const char *q, int pitch4) {   // rows 0 .. 3 and 4 .. 7 behind q
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)q);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(q + pitch4));
        const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
        const u32x4 d = {l2[0], l2[1], h2[0], h2[1]};
        return __builtin_bit_cast(bf16x8, d);
    };
    constexpr int NT = SZ == 2 ? 2 : 8;   // reduction steps per stage
    struct Frags {
        std::conditional_t<SZ == 2, bf16x8, float> a[NT][FM], b[NT][FN];
    };
    auto fetch = [&](int buf, Frags &r) {
        const char *base = lds + buf * STG;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            if constexpr (SZ == 2) {
#pragma unroll
                for (int i = 0; i < FM; ++i) r.a[t][i] = tr8(base + ra[i] + t * 16 * BM * SZ, 4 * BM * SZ);
#pragma unroll
                for (int f = 0; f < FN; ++f) r.b[t][f] = tr8(base + rb[f] + t * 16 * BN * SZ, 4 * BN * SZ);
            } else {
#pragma unroll
                for (int i = 0; i < FM; ++i) r.a[t][i] = *reinterpret_cast<const float *>(base + ra[i] + t * 2 * BM * SZ);
#pragma unroll
                for (int f = 0; f < FN; ++f) r.b[t][f] = *reinterpret_cast<const float *>(base + rb[f] + t * 2 * BN * SZ);
            }
        }
    };
    auto multiply = [&](const Frags &r) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int f = 0; f < FN; ++f) {
                    if constexpr (SZ == 2) acc[i][f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(r.a[t][i], r.b[t][f], acc[i][f], 0, 0, 0);
                    else acc[i][f] = __builtin_amdgcn_mfma_f32_32x32x2f32(r.a[t][i], r.b[t][f], acc[i][f], 0, 0, 0);
                }
    };

    auto accumulate = [&](auto masked) {
        constexpr bool MASK = decltype(masked)::value;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int f = 0; f < FN; ++f)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][f][v] = 0.f;
        int fq[LB], fp[LB];   // column and row of the pitch of each load's pixel
#pragma unroll
        for (int k = 0; k < LB; ++k) {
            const int px = s0 * PIX + ((wave + NW * k) * 64 + lane) / PB, row = px / p.Qp;
            fq[k] = px - row * p.Qp;
            fp[k] = row % p.Pp;
        }
        uint32_t dsoff = s0 * dstep, xsoff = s0 * xstep;
        auto issue = [&](int buf) {
            const uint32_t lb = lbase + buf * STG + wave * 1024;
            uint32_t vo[LB];
#pragma unroll
            for (int k = 0; k < LB; ++k) {
                vo[k] = vb[k];
                if (MASK) {
                    if (fq[k] >= p.Q || fp[k] >= p.P) vo[k] = OUTSIDE;
                    fq[k] += p.dq;
                    fp[k] += p.dp;
                    if (fq[k] >= p.Qp) { fq[k] -= p.Qp; ++fp[k]; }
                    if (fp[k] >= p.Pp) fp[k] -= p.Pp;
                }
            }
#pragma unroll
            for (int k = 0; k < LA; ++k)
                if (IA % NW == 0 || wave + NW * k < IA) load_lds16(lb + k * NW * 1024, va[k], dr, dsoff);
#pragma unroll
            for (int k = 0; k < LB; ++k)
                if (IB % NW == 0 || wave + NW * k < IB) load_lds16(lb + IA * 1024 + k * NW * 1024, vo[k], xr, xsoff);
            dsoff += dstep;
            xsoff += xstep;
        };

        // the loop of cl_gemm_kernel
        Frags fr[2];
        for (int i = 0; i < NST && i < n; ++i) issue(i);
        if (n >= NST) stage_wait<(NST - 1) * LMIN>();
        else stage_wait<0>();
        fetch(0, fr[0]);
        int buf = 0;
        auto trip = [&](int i, const Frags &cur, Frags &nxt) {
            if (i + NST - 1 < n) stage_wait<(NST - 2) * LMIN>();
            else stage_wait<0>();
            const int free = buf;
            buf = buf + 1 == NST ? 0 : buf + 1;
            reads_done();
            fetch(buf, nxt);
            if (i + NST < n) issue(free);
            __builtin_amdgcn_sched_barrier(0);
            multiply(cur);
            __builtin_amdgcn_sched_barrier(0);
        };
        // fp32: a chain of 128 pixels (CHAIN stages) at a time, the chains' sums added up: one long chain's roundings made the result up to 1.7 times
        // further from the exact one than the general kernel's slices did (8 x 256 x 56x56, 256 channels 3x3: 5.0e-7; chains of 128 pixels 1.7e-7, of 256
        // 2.1e-7).  The additions cost 2 % (269 -> 274 us a call there; six other layers 1.3 to 2.1 %).
        f32x16 whole[FM][FN];
        constexpr int CHAIN = 8;
        auto add_up = [&](bool last) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int f = 0; f < FN; ++f)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        whole[i][f][v] += acc[i][f][v];
                        acc[i][f][v] = last ? whole[i][f][v] : 0.f;
                    }
        };
        if constexpr (SZ == 4) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int f = 0; f < FN; ++f)
#pragma unroll
                    for (int v = 0; v < 16; ++v) whole[i][f][v] = 0.f;
        }
        for (int i = 0; i < n; i += 2) {
            trip(i, fr[0], fr[1]);
            if (i + 1 < n) trip(i + 1, fr[1], fr[0]);
            if constexpr (SZ == 4)
                if (i % CHAIN == CHAIN - 2) add_up(false);
        }
        if constexpr (SZ == 4) add_up(true);
    };
    accumulate(std::false_type());
    if (p.holes && any_not_finite(acc, lds)) accumulate(std::true_type());

    float *o = part + (size_t)(p.slice0 + slice) * p.K * p.ncols;
#pragma unroll
    for (int f = 0; f < FN; ++f) {
        const int col = c0 + (wn * FN + f) * 32 + l32;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int k = k0 + (wm * FM + i) * 32 + 8 * (v / 4) + 4 * g + v % 4;
                if (col < p.ncols && k < p.K) o[(size_t)k * p.ncols + col] = acc[i][f][v];
            }
    }
}

// dw[k][c][r][s] = sum over the slices.  A workgroup takes 256 / G columns of one k; its G groups of threads take every
// G-th slice and are added in order (many slices in one chain would be all latency, few do not need the groups).
template <int G>
__global__ void __launch_bounds__(256) cl_wgrad_reduce_kernel(const float *__restrict__ part, float *__restrict__ dw, int K, int C,
                                                              int R, int S, int Cp, int SC, int ncols, int nsl)
{
    constexpr int COLS = 256 / G;
    __shared__ float sums[G][COLS];
    const int lane = threadIdx.x % COLS, grp = threadIdx.x / COLS;
    const int col = blockIdx.x * COLS + lane, k = blockIdx.y;
    const float *q = part + (size_t)k * ncols + min(col, ncols - 1);
    const size_t pitch = (size_t)K * ncols;
    float v = 0.f;
    int z = grp;
    for (; z + 3 * G < nsl; z += 4 * G) {
        const float a = q[z * pitch], b = q[(z + G) * pitch], c = q[(z + 2 * G) * pitch], d = q[(z + 3 * G) * pitch];
        v += (a + b) + (c + d);
    }
    for (; z < nsl; z += G) v += q[z * pitch];
    if (G > 1) {
        sums[grp][lane] = v;
        __syncthreads();
        if (grp) return;
        v = sums[0][lane];
#pragma unroll
        for (int i = 1; i < G; ++i) v += sums[i][lane];
    }
    if (col >= ncols) return;
    const int r = col / SC, rem = col - r * SC, s = rem / Cp, c = rem - s * Cp;
    if (s < S && c < C) dw[(((size_t)k * C + c) * R + r) * S + s] = v;
}

}  // namespace
}  // namespace sn
