// CONV 3x3 / stride-1 over at most 64 reduction channels, bf16 (forward: input channels; backward-data: output channels), on
// gfx950, at any workspace (it needs none).
//
// With so few channels a tile of outputs is over after four 16-channel chunks, and a kernel that starts afresh for every tile
// spends its time in prologues and epilogues.  Here the filter stays in registers for the workgroup's life and the image
// runs past it: a wave owns 32 output channels (9 taps x 64 channels: 144 registers) and a band of rows 32 pixels wide,
// and takes one input row a step.  The row is multiplied with all three filter rows at once, into the three output rows
// that are open; the first of them is then complete and stored.  An operand read from LDS serves three matrix products,
// each input row is read once per band, and there are no vertical halos but the two rows at a band's ends.
//   A workgroup is 8 waves: 4 bands x 2 halves of 64 output channels; the two waves of a band share its rows in LDS, laid out
// [pixel][channel] (a pixel's pitch is an odd number of 16-byte units: neither operands read nor turned pixels written meet in a bank,
// measured alone).  Rows come from memory straight into LDS three steps ahead, and a step ahead of their use they are turned with byte
// permutes, 8 channels x 4 pixels a lane; the reads for that, 8 bytes at strides of 192, are what conflicts: 29 % of the kernel's LDS cycles.  All this,
// and storing the row completed before, is cut into pieces between the matrix products: done before and after them it cost
// 10 to 15 % (54 steps: 139 us, like this 125).  One barrier a step.  BN statistics are summed as rows are stored, a triple per
// workgroup and channel.
//   Bound by the step's chain, not by a unit: 36 products of 32 cycles a wave and step, two waves on a SIMD, fill 49 % of 4400
// cycles; memory moves 313 MB in 125 us.  32 x 64 x 224x224 -> 64: 185 -> 130 us with a workspace (the tiles of conv_tile.h),
// 222 and 238 (backward-data) -> 145 and 138 without; 64 x 64 x 56x56 -> 64: 32 -> 25 and 33 -> 26; 32 x 32 x 112x112 -> 64:
// 35 -> 28 and 41 -> 28.  A launch starts with the filter's way into registers: small layers stay with the tiles.
#include <algorithm>
#include <cmath>

#include "conv_tile.h"

namespace sn {
namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int BW = 32;        // output columns of a band
constexpr int LCOLS = 48;     // columns of a row in LDS: from 8 before the band to 8 past it
constexpr int WG_BANDS = 4;
constexpr uint32_t OUTSIDE = 0x80000000u;   // an offset no tensor reaches

// LDS: two rows of each band, and DEPTH rows on their way, 4 x 1 KB a wave; at the start the filter
constexpr int DEPTH = 3;
constexpr int band_rows_lds(int NC) { return WG_BANDS * 2 * LCOLS * (NC * 32 + 16); }
constexpr int band_lds(int NC) { return band_rows_lds(NC) + 8 * DEPTH * 4096; }

struct BandProblem {
    int N, Cin, Hin, Win, Kout, Pout, Qout, padh, padw;
    int w_sm, w_sr;       // strides of w over output and reduction channels
    int strips, bands, rows;   // 32-column strips of an image, bands of a strip, output rows of a band
    int units;            // N * strips * bands
    int nub;              // workgroups per 64 output channels, and those of an XCD
    int per_xcd;
    int nkt;
    uint32_t in_bytes, out_bytes;
    float *stats;
};

struct BandPlan {
    BandProblem p;
    int NC;
};

// The row a step works on: `t` counts the input rows of unit `u`.
struct RowIter {
    int u, t, n, band, q0;
    __device__ void decode(const BandProblem &p)
    {
        const int v = u / p.strips;
        q0 = (u - v * p.strips) * BW;
        n = v / p.bands;
        band = v - n * p.bands;
        t = 0;
    }
    __device__ bool next(const BandProblem &p)   // true: a new unit
    {
        if (++t < p.rows + 2) return false;
        u += p.nub * WG_BANDS;
        decode(p);
        return true;
    }
};

__device__ inline i32x4 make_rsrc(const void *p, uint32_t bytes)
{
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    const i32x4 r = {(int)(uint32_t)a, (int)(uint32_t)(a >> 32) & 0xffff, (int)bytes, 0x00020000};
    return r;
}

__device__ inline uint32_t lds_address(const void *p)
{
    return (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const void *)p);
}

// 16 bytes a lane from memory to LDS, lane l's at lds + 16 l.  (m0 is one of the registers that the compiler reserves: that it is not
// preserved here, which it warns of, is what the clobber says.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ inline void load_lds16(uint32_t lds, uint32_t voff, i32x4 rsrc)
{
    asm volatile("s_mov_b32 m0, %0\n\t"
                 "s_nop 0\n\t"
                 "buffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(lds), "v"(voff), "s"(rsrc) : "memory", "m0");
}
#pragma clang diagnostic pop

// All but the last N of the wave's loads and stores are done.
template <int N>
__device__ inline void wait_loads()
{
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

template <int NC, bool TFLIP, bool STATS>
__global__ void __launch_bounds__(512, 2)
band3x3_kernel(const bf16_t *__restrict__ in, const bf16_t *__restrict__ w, bf16_t *__restrict__ out, BandProblem p)
{
    constexpr int PITCH = NC * 32 + 16, ROW = LCOLS * PITCH;
    extern __shared__ __align__(16) unsigned char lds[];
    static_assert(band_lds(NC) <= 160 * 1024 && band_lds(NC) >= 2 * NC * 9 * 64 * 16, "the filter");
    static_assert(band_rows_lds(NC) >= 8 * 32 * 3 * (int)sizeof(float), "the statistics' triples");

    const int xcd = blockIdx.x % 8, jx = blockIdx.x / 8, kt = jx % p.nkt, ub = xcd * p.per_xcd + jx / p.nkt;
    if (ub >= p.nub) return;   // uniform for the workgroup, before any barrier
    const int lane = threadIdx.x % 64, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int band = wave % WG_BANDS, kh = wave / WG_BANDS, l32 = lane % 32, g = lane / 32;
    const int k = kt * 64 + kh * 32 + l32;
    const bool k_on = k < p.Kout;
    const uint32_t kout = (uint32_t)k * (uint32_t)(p.Pout * p.Qout) * 2u;   // k < Kout: below 2^31

    // The wave's filter: lane (k, half g) holds channels 16 c + 8 g .. + 7 of every tap.  The four waves of the same output
    // channels gather a chunk each -- 16-byte pieces 1152 bytes apart, a request to the cache per lane -- and share it through LDS.
    bf16x8 wf[NC][9];
    {
        bf16x8 *const share = reinterpret_cast<bf16x8 *>(lds) + kh * NC * 9 * 64 + lane;
        if (band < NC) {
            const int kc = min(k, p.Kout - 1), ch = 16 * band + 8 * g;
            uint32_t wc[TFLIP ? 40 : 36];
            if (ch < p.Cin) {
                const bf16_t *src = w + (size_t)kc * p.w_sm + (size_t)ch * p.w_sr;
                if constexpr (!TFLIP) {   // eight channels x nine taps: one run
#pragma unroll
                    for (int j = 0; j < 9; ++j) {
                        const u32x4 v = load8_any(src + 8 * j);
                        wc[4 * j] = v.x; wc[4 * j + 1] = v.y; wc[4 * j + 2] = v.z; wc[4 * j + 3] = v.w;
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const bf16_t *run = src + (size_t)i * p.w_sr;
                        const u32x4 v = load8_any(run);
                        wc[5 * i] = v.x; wc[5 * i + 1] = v.y; wc[5 * i + 2] = v.z; wc[5 * i + 3] = v.w;
                        wc[5 * i + 4] = run[8];
                    }
                }
            } else {
#pragma unroll
                for (int i = 0; i < (TFLIP ? 40 : 36); ++i) wc[i] = 0;
            }
            static_for<9>([&](auto tc) {
                constexpr int tap = decltype(tc)::value;
                u32x4 d;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int h0 = TFLIP ? 2 * j * 10 + 8 - tap : 2 * j * 9 + tap;
                    const int h1 = TFLIP ? (2 * j + 1) * 10 + 8 - tap : (2 * j + 1) * 9 + tap;
                    d[j] = pick2(wc, h0, h1);
                }
                share[(band * 9 + tap) * 64] = __builtin_bit_cast(bf16x8, d);
            });
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int tap = 0; tap < 9; ++tap) wf[c][tap] = share[(c * 9 + tap) * 64];
        __syncthreads();
    }

    // ---- rows into LDS: a lane moves 4 channels x 8 pixels; the band's two waves share its channels
    constexpr int QUADS = NC * 2;   // channel quads of a wave
    const int blk = lane % 6, quad = kh * QUADS + lane % (6 * QUADS) / 6;   // lanes left over repeat another's
    unsigned char *const mine = lds + band * 2 * ROW;
    // turned: a lane takes 8 channels x 4 pixels of the columns 4 .. 43, neighbours the next channels (written without bank conflicts)
    const int turn = lane % (10 * NC), tcol = 4 + turn / NC * 4, oct = turn % NC;
    const uint32_t tsrc = (oct * 12 + tcol / 8) * 16 + tcol % 8 * 2;
    const uint32_t wr = tcol * PITCH + (kh * NC + oct) * 16;
    const uint32_t chan = (uint32_t)p.Hin * p.Win * 2;
    uint32_t voff = OUTSIDE;
    auto strip = [&](const RowIter &it) {
        const int lcol = it.q0 - 8 + 8 * blk;   // all eight pixels lie in the row, or none
        const bool ok = quad * 4 < p.Cin && lcol >= 0 && lcol < p.Win;
        voff = ok ? quad * 4 * chan + lcol * 2u : OUTSIDE;
    };
    // Memory to LDS, a lane's four 16-byte pieces at its place in the wave's slot: no register holds a row on its way.  Slots and
    // waits are counted, not tracked: step T waits for row T + 1 of T + DEPTH, with NST stores between them.
    constexpr int NST = 2, YOUNGER = (DEPTH - 1) * 4 + DEPTH * NST;
    static_assert(YOUNGER < 64, "the counter has six bits");
    const uint32_t raw0 = band_rows_lds(NC) + wave * DEPTH * 4096;
    const uint32_t raw_m0 = __builtin_amdgcn_readfirstlane(lds_address(lds) + raw0);
    uint32_t lat = 0;
    bool lok = false;
    auto load_row = [&](const RowIter &it) {   // where the next row lies
        const int h = it.band * p.rows - p.padh + it.t;
        lok = it.u < p.units && h >= 0 && h < p.Hin;
        lat = lok ? (uint32_t)(it.n * p.Cin * p.Hin + h) * (uint32_t)p.Win * 2u : 0u;
    };
    auto load_piece = [&](int slot, int i) {   // channel i of the lane's four: the image's row moved by i channels (there are eight at least)
        const uint32_t at = lat + i * chan;
        load_lds16(raw_m0 + slot * 4096 + i * 1024, voff, make_rsrc(reinterpret_cast<const unsigned char *>(in) + at, lok ? p.in_bytes - at : 0u));
    };
    uint2 tv[8];
    auto fetch = [&](int slot) {
        const unsigned char *own = lds + raw0 + slot * 4096 + tsrc;
#pragma unroll
        for (int j = 0; j < 8; ++j) tv[j] = *reinterpret_cast<const uint2 *>(own + j % 4 * 1024 + j / 4 * 96);
    };
    auto turn_pixel = [&](uint32_t buf, auto pixel) {
        constexpr int px = decltype(pixel)::value;
        constexpr uint32_t sel = px % 2 ? 0x07060302u : 0x05040100u;
        u32x4 v;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            v[j] = px < 2 ? __builtin_amdgcn_perm(tv[2 * j + 1].x, tv[2 * j].x, sel) : __builtin_amdgcn_perm(tv[2 * j + 1].y, tv[2 * j].y, sel);
        *reinterpret_cast<u32x4 *>(mine + buf + wr + px * PITCH) = v;
    };
    auto barrier = [&]() {   // the wave's LDS accesses are done; its global ones stay in flight
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };

    RowIter ld, cp;   // of the row to load next; of the last row multiplied
    ld.u = ub * WG_BANDS + band;
    ld.decode(p);
    cp = ld;
    cp.t = -1;
    strip(ld);
    auto load_next = [&](int slot) {
        load_row(ld);
#pragma unroll
        for (int i = 0; i < 4; ++i) load_piece(slot, i);
        if (ld.next(p)) strip(ld);
    };
    static_assert(DEPTH == 3, "slots are numbered as steps are");
    load_next(0);
    load_next(1);
    load_next(2);
    wait_loads<0>();   // the rows of the first two steps, too, from where on the count is right
    fetch(0);
    static_for<4>([&](auto px) { turn_pixel(0, px); });
    load_next(0);
    barrier();

    const int rounds = (p.units + p.nub * WG_BANDS - 1) / (p.nub * WG_BANDS);
    const int steps = rounds * (p.rows + 2);
    const uint32_t rd = (l32 + 8 - p.padw) * PITCH + g * 16;
    uint32_t buf = 0;
    f32x16 acc[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) acc[i] = f32x16{};
    int cnt = 0;   // whole rows: the same in every lane
    float shift = 0.f, s1 = 0.f, s2 = 0.f;
    // The row that the last step completed, as it is stored: pixels 8 (j / 2) + 4 g + 2 (j % 2) and one more are u[j].
    uint32_t u[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    bool real = false;
    int cols = 0;
    uint32_t oat = 0;
    auto finish_row = [&]() {
        const int row = cp.band * p.rows + cp.t - 2;
        cols = p.Qout - cp.q0;
        real = cp.t >= 2 && cp.u < p.units && row < p.Pout;
        oat = real ? (uint32_t)(cp.n * p.Kout * p.Pout + row) * (uint32_t)p.Qout * 2u : 0u;
    };
    auto finish_stats = [&]() {
        if constexpr (STATS) {
            if (real) {
                if (cnt == 0) shift = __uint_as_float(u[0] << 16);
                float a1 = 0.f, a2 = 0.f;
                if (cols >= BW) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const float d0 = __uint_as_float(u[j] << 16) - shift, d1 = __uint_as_float(u[j] & 0xffff0000u) - shift;
                        a1 += d0; a2 = __builtin_fmaf(d0, d0, a2);
                        a1 += d1; a2 = __builtin_fmaf(d1, d1, a2);
                    }
                    cnt += BW / 2;
                } else {
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        if (8 * (j / 2) >= cols) continue;   // the width is a multiple of eight
                        const float d0 = __uint_as_float(u[j] << 16) - shift, d1 = __uint_as_float(u[j] & 0xffff0000u) - shift;
                        a1 += d0; a2 = __builtin_fmaf(d0, d0, a2);
                        a1 += d1; a2 = __builtin_fmaf(d1, d1, a2);
                    }
                    cnt += cols / 2;
                }
                s1 += a1;
                s2 += a2;
            }
        }
    };
    auto finish_half = [&](auto half) {
        constexpr int h = decltype(half)::value;
        // halves of the wave swap, so that a lane has eight pixels in a row; always a store, for the waits: what must not be
        // written has an offset outside
        const __amdgpu_buffer_rsrc_t ors = __builtin_amdgcn_make_buffer_rsrc(
            reinterpret_cast<unsigned char *>(out) + oat, 0, real ? p.out_bytes - oat : 0u, 0x00020000);
        const auto e0 = __builtin_amdgcn_permlane32_swap(u[4 * h], u[4 * h + 2], false, false);
        const auto e1 = __builtin_amdgcn_permlane32_swap(u[4 * h + 1], u[4 * h + 3], false, false);
        const u32x4 v = {e0[0], e1[0], e0[1], e1[1]};
        const int left = k_on ? cols - 16 * h - 8 * g : 0;   // of the lane's eight columns
        __builtin_amdgcn_raw_buffer_store_b128(v, ors, left > 0 ? kout + (uint32_t)(cp.q0 + 16 * h + 8 * g) * 2u : OUTSIDE, 0, 0);
    };
    // A step: the row in `buf` multiplied, the next one turned and written beside it, the one DEPTH after it loaded, and the row
    // that the step before completed stored.  The moves are cut into pieces between the products, which they run under.
    auto step = [&](auto slot) {
        constexpr int S0 = decltype(slot)::value, S1 = (S0 + 2) % 3, S2 = (S0 + 1) % 3;   // rows opened now, one and two steps ago
        constexpr int NG = 3 * NC, RS = (S0 + 1) % DEPTH;
        const unsigned char *src = mine + buf + rd;
        const uint32_t other = ROW - buf;
        bf16x8 a[2];
        a[0] = *reinterpret_cast<const bf16x8 *>(src);
        finish_row();
        load_row(ld);
        static_for<NG>([&](auto idx) {
            constexpr int i = decltype(idx)::value, c = i / 3, s = i % 3, nx = i + 1;
            // six places for the pieces: after groups 0, NG/6, ...
            constexpr auto at = [](int piece) { return piece * (NG - 1) / 5; };
            if constexpr (nx < NG) a[nx % 2] = *reinterpret_cast<const bf16x8 *>(src + nx % 3 * PITCH + nx / 3 * 32);
            acc[S2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i % 2], wf[c][6 + s], acc[S2], 0, 0, 0);
            acc[S1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i % 2], wf[c][3 + s], acc[S1], 0, 0, 0);
            if constexpr (i == 0) acc[S0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i % 2], wf[c][s], f32x16{}, 0, 0, 0);
            else acc[S0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i % 2], wf[c][s], acc[S0], 0, 0, 0);
            if constexpr (i == at(0)) {
                finish_half(std::integral_constant<int, 0>{});
                finish_half(std::integral_constant<int, 1>{});
            }
            if constexpr (i == at(1)) {
                wait_loads<YOUNGER>();
                fetch(RS);
                if constexpr (STATS) finish_stats();
            }
            if constexpr (i == at(2)) {
                turn_pixel(other, std::integral_constant<int, 0>{});
                turn_pixel(other, std::integral_constant<int, 1>{});
            }
            if constexpr (i == at(3)) {
                turn_pixel(other, std::integral_constant<int, 2>{});
                turn_pixel(other, std::integral_constant<int, 3>{});
            }
            if constexpr (i == at(4)) {
                load_piece(RS, 0);
                load_piece(RS, 1);
                load_piece(RS, 2);
                load_piece(RS, 3);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
#pragma unroll
        for (int j = 0; j < 8; ++j) u[j] = f32x2_to_bf16x2(acc[S2][2 * j], acc[S2][2 * j + 1]);
        cp.next(p);
        if (ld.next(p)) strip(ld);
        buf = other;
        barrier();
    };
    // whole rounds of three steps: those beyond the last row load, multiply and store nothing of a unit
    for (int t = 0; t < steps; t += 3) {
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
        step(std::integral_constant<int, 2>{});
    }
    finish_row();
    finish_half(std::integral_constant<int, 0>{});
    finish_half(std::integral_constant<int, 1>{});
    if constexpr (STATS) finish_stats();
    wait_loads<0>();   // rows past the last one are on their way into LDS: not past the workgroup's end

    if constexpr (STATS) {
        TileMoments m;
        m.n = (float)cnt;
        m.mean = cnt > 0 ? shift + s1 / m.n : 0.f;
        m.m2 = cnt > 0 ? fmaxf(s2 - s1 * s1 / m.n, 0.f) : 0.f;
        TileMoments o;
        o.n = __shfl_xor(m.n, 32);
        o.mean = __shfl_xor(m.mean, 32);
        o.m2 = __shfl_xor(m.m2, 32);
        float *red = reinterpret_cast<float *>(lds);   // every step ended with a barrier
        if (g == 0) {
            m = moments_join(m, o);
            float *e = red + (wave * 32 + l32) * 3;
            e[0] = m.n; e[1] = m.mean; e[2] = m.m2;
        }
        __syncthreads();
        if (band == 0 && g == 0 && k_on) {
#pragma unroll
            for (int b = 1; b < WG_BANDS; ++b) {
                const float *e = red + ((wave + b) * 32 + l32) * 3;
                o = {e[0], e[1], e[2]};
                m = moments_join(m, o);
            }
            float *e = p.stats + ((size_t)k * p.nub + ub) * 3;
            e[0] = m.n; e[1] = m.mean; e[2] = m.m2;
        }
    }
}

bool band_plan(const ConvGeom &g, bool bwd_data, BandPlan *pl)
{
    if (g.R != 3 || g.S != 3 || g.sh != 1 || g.sw != 1 || !g.in_bf16 || !g.out_bf16) return false;
    if (g.ph > 2 || g.pw > 2 || g.ph < 0 || g.pw < 0) return false;
    BandProblem &p = pl->p;
    p.N = g.N;
    if (!bwd_data) {
        p.Cin = g.C; p.Hin = g.H; p.Win = g.W; p.Kout = g.K; p.Pout = g.P; p.Qout = g.Q; p.padh = g.ph; p.padw = g.pw;
        p.w_sm = g.C * 9; p.w_sr = 9;
    } else {
        p.Cin = g.K; p.Hin = g.P; p.Win = g.Q; p.Kout = g.C; p.Pout = g.H; p.Qout = g.W; p.padh = 2 - g.ph; p.padw = 2 - g.pw;
        p.w_sm = 9; p.w_sr = g.C * 9;
    }
    // rows of whole 16-byte pieces, channels in runs of eight
    if (p.Cin > 64 || p.Cin % 8 || p.Win % 8 || p.Qout % 8) return false;
    const unsigned long long lim = 0x80000000ull;
    if (2ull * p.N * p.Cin * p.Hin * p.Win > lim || 2ull * p.N * p.Kout * p.Pout * p.Qout > lim) return false;
    pl->NC = p.Cin <= 32 ? 2 : p.Cin <= 48 ? 3 : 4;
    p.strips = (p.Qout + BW - 1) / BW;
    p.nkt = (p.Kout + 63) / 64;
    p.per_xcd = std::max(1, 32 / p.nkt);
    p.nub = 8 * p.per_xcd;
    // Bands of a strip, of four rows at least, so that the rounds of bands that the workgroups' slots take have the fewest steps in all.
    // For a number of rounds that is as many bands as fit; more rounds, with two rows of halo each, only make up for rows that do
    // not divide evenly, and none can do with fewer steps than all rows over the slots and its halos.
    const long long each = (long long)p.N * p.strips, at = (long long)p.nub * WG_BANDS;
    const long long most = std::min<long long>(std::max(1, p.Pout / 4), 0x3fffffff / each);
    long long best = -1;
    for (long long rounds = (each + at - 1) / at, b = 0; most > 0; rounds = std::max(rounds + 1, ((b + 1) * each + at - 1) / at)) {
        if (best >= 0 && (p.Pout * each + at - 1) / at + 2 * rounds >= best) break;
        b = std::min(most, rounds * at / each);
        const int rows = (int)((p.Pout + b - 1) / b), bands = (p.Pout + rows - 1) / rows;
        const long long units = each * bands, steps = (units + at - 1) / at * (rows + 2);
        if (best < 0 || steps < best) {
            best = steps;
            p.bands = bands; p.rows = rows; p.units = (int)units;
        }
        if (b == most) break;
    }
    if (best < 0 || best > 0x3fffffff) return false;
    p.nub = std::min(p.nub, (p.units + WG_BANDS - 1) / WG_BANDS);
    p.per_xcd = (p.nub + 7) / 8;
    p.in_bytes = (uint32_t)(2ull * p.N * p.Cin * p.Hin * p.Win);
    p.out_bytes = (uint32_t)(2ull * p.N * p.Kout * p.Pout * p.Qout);
    p.stats = nullptr;
    return true;
}

template <int NC, bool TFLIP, bool STATS>
hipError_t launch(const void *in, const void *w, void *out, const BandProblem &p, hipStream_t st)
{
    auto kern = band3x3_kernel<NC, TFLIP, STATS>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, band_lds(NC));
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(kern, dim3(8 * p.per_xcd * p.nkt), dim3(512), band_lds(NC), st, static_cast<const bf16_t *>(in),
                       static_cast<const bf16_t *>(w), static_cast<bf16_t *>(out), p);
    return hipGetLastError();
}

template <int NC>
hipError_t launch_nc(const void *in, const void *w, void *out, const BandProblem &p, bool bwd_data, hipStream_t st)
{
    if (bwd_data) return launch<NC, true, false>(in, w, out, p, st);
    return p.stats ? launch<NC, false, true>(in, w, out, p, st) : launch<NC, false, false>(in, w, out, p, st);
}

}  // namespace

// Estimate in us: steps of a workgroup, rounds of workgroups, bytes; fitted to 1600 layers (1 to 64 images, 8 to 64 reduction and 8 to 520
// output channels, planes of 7x7 to 230x224, either direction), which it reproduces to 8 % (rms).
double band_conv_us(const ConvGeom &g, bool bwd_data)
{
    BandPlan pl;
    if (!band_plan(g, bwd_data, &pl)) return 1e9;
    const BandProblem &p = pl.p;
    const long long at = (long long)p.nub * WG_BANDS, steps = (p.units + at - 1) / at * (p.rows + 2);
    const double share = p.nub * p.nkt / 256.0;
    return 6.8 + steps * (0.204 + 0.337 * pl.NC + 0.14 * std::min(1.0, share)) * std::max(1.0, std::ceil(share)) + 0.058e-6 * ((double)p.in_bytes + p.out_bytes);
}

int band_conv_stats_tiles(const ConvGeom &g)
{
    BandPlan pl;
    return band_plan(g, false, &pl) ? pl.p.nub : 0;
}

hipError_t launch_band_conv(const void *in, const void *w, void *out, const ConvGeom &g, bool bwd_data, hipStream_t st, float *stats)
{
    BandPlan pl;
    if (!band_plan(g, bwd_data, &pl) || (stats && bwd_data)) return hipErrorInvalidValue;
    pl.p.stats = stats;
    const BandProblem &p = pl.p;
    if (pl.NC == 2) return launch_nc<2>(in, w, out, p, bwd_data, st);
    if (pl.NC == 3) return launch_nc<3>(in, w, out, p, bwd_data, st);
    return launch_nc<4>(in, w, out, p, bwd_data, st);
}

}  // namespace sn
