// CONV backward-filter of the image layer -- up to four input channels under a large filter (11x11 / stride 4,
// 7x7 / stride 2) -- on gfx950, bf16 operands, at any workspace (definitions in sn.h).
//
// The layer is a product dw[k][(c,r,s)] = sum over (n,p,q) of dy[n][k][p][q] * x[n][c][p sh + r - ph][q sw + s - pw] with
// a few hundred columns and a reduction of hundreds of thousands of pixels, which dy has contiguous and x, under a
// strided filter, does not.  An unfolded copy of x would be 30 to 40 times x in memory; here it exists in LDS only,
// one output row of 64 pixels at a time: row (c, h, s) of the ring below holds x[c][h][q sw + s - pw] for 64 consecutive q,
// which is what a lane of the matrix operand reads 16 bytes of.  An input row's share does not depend on the
// output row it is used for, so going down a strip of 64 output columns only the sh input rows that the next output row
// adds are unfolded (11x11 / 4: 12 of 33 (c, r) rows).
//   A workgroup owns 32 MT output channels (all of them up to 96) x every (c, r, s) and walks its share of the output rows;
// its twelve waves take a tile of 32 columns each, or where there are at most six tiles share one, each with its part
// of the pixels, and add up through LDS at the end.  Loads run two output rows ahead in registers (one row multiplies for half the latency of
// memory), one barrier per row.  The workgroups' sums go to slices of the workspace that a reduction in slice order adds,
// or without workspace to dw by atomics.
//   Bound by instruction issue: a row's 144 matrix products take 1150 cycles, its unfolding, addresses and operand reads
// twice that.  128 x 3 x 227x227, 96 channels 11x11 / 4 (27 GFLOP): general kernel 203 -> 69 us, the channels-last product
// with 300 MiB 140; 22 x 3 x 82x66, 38 channels 7x7 / 2: forward and backward-filter 64 -> 36 us.
#include <algorithm>
#include <cmath>

#include "sn_internal.h"

namespace sn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int WAVES = 12, THREADS = WAVES * 64;
constexpr int LDS_MAX = 160 * 1024;

struct ImageProblem {
    int N, C, H, W, K, R, S, sh, sw, ph, pw, P, Q;
    int CRS;
    int nqb;       // strips per image: PX-pixel blocks of an output row
    int steps;     // steps of a strip: P output rows, 64 / PX at a time
    int rows;      // N * nqb * steps
    int gr;        // input rows of a group: those a step adds
    int G;         // groups under a step; the ring holds one more
    int xn, dyn;   // elements of x and dy
};

// Four elements at any address.  What lies outside a row is masked when the run is stored, not when it is loaded, so that nothing
// waits for a load before its turn; a run over an end of the tensor is loaded where it ends with it, and shifted.
struct __attribute__((packed, aligned(2))) Any8 { uint64_t v; };
__device__ inline uint64_t load4(const bf16_t *base, int at)
{
    return reinterpret_cast<const Any8 *>(reinterpret_cast<const char *>(base) + (uint32_t)at * 2u)->v;
}
__device__ inline int clamped(int at, int n) { return min(max(at, 0), n - 4); }   // where the run at `at` of n elements is loaded

// elements lo .. hi - 1 of four
__device__ inline uint64_t elements(int lo, int hi)
{
    const uint64_t h = hi >= 4 ? ~0ull : hi <= 0 ? 0ull : (1ull << (16 * hi)) - 1;
    return lo <= 0 ? h : lo >= 4 ? 0ull : h & ~((1ull << (16 * lo)) - 1);
}

// One stage: group gam of input rows of a strip, and the step whose last group it is (-1: none yet).
struct Stage { int n, q0, gam, step; };

// The stages of a workgroup's share [row, row + left) of all strips' steps, in order: for each strip G - 1 groups before its first
// step, then one per step.
struct Walk {
    int n, qb, pb, pe, gam, left;
    __device__ Walk(const ImageProblem &p, int row, int rows)
    {
        const int strip = row / p.steps;
        n = strip / p.nqb;
        qb = strip - n * p.nqb;
        left = rows;
        begin(p, row - strip * p.steps);
    }
    __device__ void begin(const ImageProblem &p, int first)
    {
        pb = gam = first;
        pe = min(p.steps, first + left);
        left -= pe - pb;
    }
    __device__ bool live() const { return pe > pb; }
    __device__ Stage next(const ImageProblem &p, int px)   // the stage, and on to the one behind it; past the last one live() is false
    {
        const Stage s = {n, qb * px, gam, gam - (p.G - 1) >= pb ? gam - (p.G - 1) : -1};
        if (++gam > pe - 1 + p.G - 1) {
            if (++qb == p.nqb) { qb = 0; ++n; }
            begin(p, 0);
        }
        return s;
    }
};

// MT 32-channel tiles of dw; NL runs of four elements hold a filter row; PX pixels of an output row per step: 64, or 32
// of two output rows; NROW passes of a wave over the (channel, input row) pairs of a group.  Every stage issues the
// same loads, needed or not: their number is what lets a wait leave the newest in flight.  KS waves share a column tile.
// What bounds a stage is the instructions issued around its 12 matrix products per wave, hence a filter row padded to 4 NL rows of
// the ring instead of a test per write, masks kept from stage to stage of a strip, and addresses that are a sum of a thread's and a stage's part.
template <int MT, int NL, int PX, int NROW, int KS>
__global__ void __launch_bounds__(THREADS, 3)
image_wgrad_kernel(const bf16_t *__restrict__ x, const bf16_t *__restrict__ dy, float *__restrict__ out, int use_atomics,
                   ImageProblem p)
{
    extern __shared__ __align__(16) char smem[];
    constexpr int PITCH = PX * 2 + 16;    // bytes per row of the ring: so that rows spread over the banks
    constexpr int DPITCH = 64 * 2 + 16, DYB = 32 * MT * DPITCH;
    constexpr int PER = 64 / PX;          // (channel, input row) pairs a wave unfolds at once, and output rows of a step
    constexpr int NG = (32 * MT * 16 + THREADS - 1) / THREADS;   // runs of dy per thread
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int k0 = blockIdx.y * 32 * MT;
    const int gbytes = p.gr * p.C * 4 * NL * PITCH, nring = p.G + 1;   // a group of the ring, and how many there are
    char *const ring = smem, *const dyb = smem + nring * gbytes;

    // this wave's column tile, and its share of the four 16-pixel steps: part, part + KS, ...
    const int ntiles = (p.CRS + 31) / 32, tile = wave / KS, part = wave % KS;
    // where its operand's columns (c, r, s) are, for each output row of the step: in which group of the ring, and where in it
    int b_grp[PER], b_off[PER];
#pragma unroll
    for (int h = 0; h < PER; ++h) {
        const int crs = min(tile * 32 + (lane & 31), p.CRS - 1);
        const int c = crs / (p.R * p.S), rs = crs - c * p.R * p.S, r0 = rs / p.S, s = rs - r0 * p.S;
        const int r = r0 + (KS == 4 ? (PX == 32 ? part >> 1 : 0) : h) * p.sh, g = r / p.gr;
        b_grp[h] = g + 2;   // see multiply
        b_off[h] = (((r - g * p.gr) * p.C + c) * 4 * NL + s) * PITCH + (lane >> 5) * 16 + (PX == 64 ? part * 32 : (part & 1) * 32);
    }
    const int a_off = (lane & 31) * DPITCH + (lane >> 5) * 16 + part * 32;

    f32x16 acc[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[m][v] = 0.f;

    // A wave unfolds PER (channel, input row) pairs of a group at a time; a lane the S elements under its pixel.
    const int npair = p.gr * p.C, px = lane % PX;
    int u_hr[NROW], u_row[NROW], u_lds[NROW];   // this lane's pairs: input row of the group, element offset, place in the group
#pragma unroll
    for (int i = 0; i < NROW; ++i) {
        const int pair = (wave + i * WAVES) * PER + (PX == 32 ? lane >> 5 : 0);
        const int hr = pair / p.C, c = pair - hr * p.C;
        u_hr[i] = pair < npair ? hr : 0x40000000;   // no input row of any image
        u_row[i] = pair < npair ? (c * p.H + hr) * p.W : 0;
        u_lds[i] = min(pair, npair) * 4 * NL * PITCH + px * 2;
    }
    // A thread brings a run of four pixels of dy for NG channels, THREADS / 16 apart.
    const int run = (t & 15) * 4, sub = run / PX, rq = run % PX;   // of output row sub of the step, pixels rq on
    uint64_t xr[2][NROW][NL], gr[2][NG];
    int g_off[NG];
#pragma unroll
    for (int m = 0; m < NG; ++m) g_off[m] = (min(k0 + m * (THREADS / 16) + (t >> 4), p.K - 1) * p.P + sub) * p.Q + rq;
    const int xpx = px * p.sw - p.pw, ximg = p.C * p.H * p.W, gimg = p.K * p.P * p.Q;
    const auto x_of = [&](const Stage &s, int i) {   // element under the filter's first column, or 0 outside the rows of the image
        const int h0 = s.gam * p.gr - p.ph, at = s.n * ximg + h0 * p.W + s.q0 * p.sw;
        return (unsigned)(h0 + u_hr[i]) < (unsigned)p.H ? at + (u_row[i] + xpx) : 0;
    };
    const auto dy_of = [&](const Stage &s, int m) { return s.n * gimg + max(s.step, 0) * PER * p.Q + s.q0 + g_off[m]; };
    const auto load = [&](const Stage &s, uint64_t (&xv)[NROW][NL], uint64_t (&gv)[NG]) {
#pragma unroll
        for (int i = 0; i < NROW; ++i) {
            const int at = x_of(s, i);
#pragma unroll
            for (int l = 0; l < NL; ++l) xv[i][l] = load4(x, clamped(at + 4 * l, p.xn));
        }
#pragma unroll
        for (int m = 0; m < NG; ++m) gv[m] = load4(dy, clamped(dy_of(s, m), p.dyn));
    };
    // what of this lane's runs is inside its rows, for strip mq0
    int mq0 = -1;
    uint64_t mask[NL], dmask = 0;
    // pixels past the row's end are zeros on both sides: nothing from outside a row is ever multiplied
    const auto store = [&](const Stage &s, const uint64_t (&xv)[NROW][NL], const uint64_t (&gv)[NG], int slot, int buf) {
        const int h0 = s.gam * p.gr - p.ph;
        if (s.q0 != mq0) {
            mq0 = s.q0;
            const int v0 = mq0 * p.sw + xpx;
#pragma unroll
            for (int l = 0; l < NL; ++l) mask[l] = mq0 + px < p.Q ? elements(-v0 - 4 * l, p.W - v0 - 4 * l) : 0ull;
            dmask = elements(0, p.Q - mq0 - rq);
        }
        // where a run with something in its row may have been moved
        const bool ends = (s.n == 0 && max(h0, 0) * p.W < p.pw) || (s.n == p.N - 1 && (p.H - h0 - p.gr) * p.W < p.pw + 16);
#pragma unroll
        for (int i = 0; i < NROW; ++i) {
            if ((wave + i * WAVES) * PER >= npair) break;
            uint64_t d[NL];
#pragma unroll
            for (int l = 0; l < NL; ++l) d[l] = xv[i][l];
            if (ends) {
                const int at = x_of(s, i);
#pragma unroll
                for (int l = 0; l < NL; ++l) {
                    const int over = at + 4 * l - clamped(at + 4 * l, p.xn);
                    d[l] = over > 3 || over < -3 ? 0 : over >= 0 ? d[l] >> (16 * over) : d[l] << (-16 * over);
                }
            }
            const bool in = (unsigned)(h0 + u_hr[i]) < (unsigned)p.H;
            char *dst = ring + slot * gbytes + u_lds[i];
            if (PX == 64 || u_hr[i] < 0x40000000) {
#pragma unroll
                for (int l = 0; l < NL; ++l) {
                    d[l] &= in ? mask[l] : 0ull;
#pragma unroll
                    for (int e = 0; e < 4; ++e) *reinterpret_cast<bf16_t *>(dst + (4 * l + e) * PITCH) = (bf16_t)(d[l] >> (16 * e));
                }
            }
        }
        if (s.step < 0) return;
        const bool dends = s.n == p.N - 1 && (p.P - (s.step + 1) * PER) * p.Q < 4;
#pragma unroll
        for (int m = 0; m < NG; ++m) {
            const int row = m * (THREADS / 16) + (t >> 4);
            uint64_t d = gv[m];
            if (dends) d >>= 16 * min(max(dy_of(s, m) - (p.dyn - 4), 0), 3);
            d = k0 + row < p.K ? d & dmask : 0ull;
            if (NG * (THREADS / 16) == 32 * MT || row < 32 * MT) *reinterpret_cast<uint64_t *>(dyb + buf * DYB + row * DPITCH + run * 2) = d;
        }
    };
    // groups slot - G + 1 .. slot of the ring, dy buffer buf, `rows` output rows of the step: one past the image's last is left out --
    // dy is another row's there, and x is inside the image (an Inf times zero is no zero either)
    const auto multiply = [&](int slot, int buf, int rows) {
        const char *a = dyb + buf * DYB + a_off;
        const char *b[PER];
#pragma unroll
        for (int h = 0; h < PER; ++h) {
            int g = slot + b_grp[h];   // slot - (G - 1) + the group, modulo the G + 1 groups
            g -= g >= nring ? nring : 0;
            b[h] = ring + g * gbytes + b_off[h];
        }
#pragma unroll
        for (int ks = 0; ks < 4; ks += KS) {   // (+ part)
            if (PX == 32 && (KS == 4 ? part >> 1 : ks / 2) >= rows) break;
            const bf16x8 bv = *reinterpret_cast<const bf16x8 *>(PX == 64 ? b[0] + ks * 32 : b[KS == 4 ? 0 : ks / 2] + (ks & 1) * 32);
            bf16x8 av[MT];
#pragma unroll
            for (int m = 0; m < MT; ++m) av[m] = *reinterpret_cast<const bf16x8 *>(a + m * 32 * DPITCH + ks * 32);
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[m], bv, acc[m], 0, 0, 0);
        }
    };

    const int per = p.rows / (int)gridDim.x, rest = p.rows - per * (int)gridDim.x;
    const int row0 = (int)blockIdx.x * per + min((int)blockIdx.x, rest), rows = per + ((int)blockIdx.x < rest ? 1 : 0);
    Walk walk(p, row0, rows);
    // Stages tau (in LDS), tau + 1 (in registers, set (tau + 1) & 1) and tau + 2 (being loaded), from tau = -2 on.
    Stage s0 = {0, 0, 0, -1}, s1 = s0;
    bool l0 = false, l1 = false, l2 = true;
    int slot = p.G;   // of tau: stage 0 goes to slot 1 % nring
    while (l0 || l1 || l2) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            Stage s2 = s1;
            l2 = walk.live();
            if (l2) s2 = walk.next(p, PX);
            load(s2, xr[u], gr[u]);
            if (l0 && s0.step >= 0 && tile < ntiles) multiply(slot, u, p.P - s0.step * PER);
            slot = slot + 1 == nring ? 0 : slot + 1;
            if (l1) store(s1, xr[u ^ 1], gr[u ^ 1], slot, u ^ 1);
            __syncthreads();
            s0 = s1; l0 = l1;
            s1 = s2; l1 = l2;
        }
    }

    // acc[m][v]: column lane & 31 of the tile, row 32 m + 8 (v / 4) + 4 (lane / 32) + v % 4 of the workgroup's channels
    const int cols = ntiles * 32;
    float *const red = reinterpret_cast<float *>(smem);   // [32 rows][cols]
    float *const mine = red + 4 * (lane >> 5) * cols + tile * 32 + (lane & 31);
    float *const dst = out + (use_atomics ? (size_t)0 : (size_t)blockIdx.x * p.K * p.CRS);
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        for (int h = 0; h < KS; ++h) {
            if (part == h && tile < ntiles)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    float *e = mine + (8 * (v / 4) + v % 4) * cols;
                    *e = h == 0 ? acc[m][v] : *e + acc[m][v];
                }
            __syncthreads();
        }
        const int n = min(32, p.K - k0 - 32 * m) * cols;
        for (int e = t; e < n; e += THREADS) {
            const int row = e / cols, col = e - row * cols;
            if (col >= p.CRS) continue;
            float *o = dst + (size_t)(k0 + 32 * m + row) * p.CRS + col;
            if (use_atomics) unsafeAtomicAdd(o, red[e]);
            else *o = red[e];
        }
        __syncthreads();
    }
}

struct ImageLaunch {
    ImageProblem p;
    int px, mt, nl, nrow, ks, ktiles;
    size_t lds;
};

bool make_problem(const ConvGeom &g, ImageLaunch *l)
{
    if (!g.in_bf16 || g.C > 4 || g.S > 12 || g.R > 384 || g.sw > 64) return false;
    const int crs = g.C * g.R * g.S;
    if (crs <= 32 || crs > 384) return false;
    ImageProblem &p = l->p;
    p.N = g.N; p.C = g.C; p.H = g.H; p.W = g.W; p.K = g.K; p.R = g.R; p.S = g.S;
    p.sh = g.sh; p.sw = g.sw; p.ph = g.ph; p.pw = g.pw; p.P = g.P; p.Q = g.Q;
    p.CRS = crs;
    // rows whose last block of 64 pixels would be half empty: blocks of 32, two output rows at a time
    l->px = (g.Q + 31) / 32 % 2 != 0 ? 32 : 64;
    const int per = 64 / l->px;
    p.nqb = (g.Q + l->px - 1) / l->px;
    p.steps = (g.P + per - 1) / per;
    const long long rows = (long long)g.N * p.nqb * p.steps;
    if (rows > 0x7fffffffLL || (long long)g.sh * g.C > 2 * WAVES) return false;
    p.rows = (int)rows;
    p.gr = g.sh * per;
    p.G = (g.R + (per - 1) * g.sh + p.gr - 1) / p.gr;
    // 32-bit element numbers, beyond either end too; a run never longer than an image
    const long long xn = (long long)g.N * g.C * g.H * g.W, dyn = (long long)g.N * g.K * g.P * g.Q, lim = 0x70000000LL;
    const long long beyond = (long long)(g.ph + g.R + p.gr * (p.G + 1)) * g.W + (g.Q + 64LL) * g.sw + g.pw;
    if (xn + beyond > lim || dyn > lim || (long long)g.C * g.H * g.W < 4 || (long long)g.K * g.P * g.Q < 4) return false;
    p.xn = (int)xn;
    p.dyn = (int)dyn;
    l->ktiles = (g.K + 95) / 96;
    if (l->ktiles > 65535) return false;
    l->mt = g.K <= 64 ? 2 : 3;
    l->nl = g.S <= 8 ? 2 : 3;
    l->nrow = g.sh * g.C <= WAVES ? 1 : 2;
    const int ntiles = (crs + 31) / 32;
    l->ks = ntiles <= 3 ? 4 : ntiles <= 6 ? 2 : 1;
    l->lds = std::max((size_t)(p.G + 1) * p.gr * g.C * 4 * l->nl * (l->px * 2 + 16) + (size_t)2 * 32 * l->mt * 144,
                      (size_t)32 * ntiles * 32 * sizeof(float));
    return l->lds <= LDS_MAX;
}

// us of a stage, and of a slice's way into dw: with partial sums fitted to 1900 timings (1100 layers of 1 to 4 channels, 33 to 384 products,
// strides 1 to 4, planes of 16 to 300 on a side, 8 to 1024 channels of dy; 400 of them over their slices), which they reproduce to 8 % (rms); atomics
// to 13 % of 400 layers'.
double stage_us(const ImageLaunch &l, bool partial)
{
    return partial ? 0.41 + 0.035 * l.mt / l.ks + 0.16 * l.nl * l.nrow + 0.047 * (l.mt - 2) : 0.42 + 0.09 * l.mt / l.ks + 0.15 * l.nl * l.nrow;
}
double slice_us(const ImageLaunch &l, bool partial) { return (double)l.p.K * l.p.CRS * 4e-6 * (partial ? 0.51 : 0.8); }

// Slices of the sum: with partial sums a workgroup per compute unit, or as many as the workspace holds.  Atomics cost more than a
// reduction reads, so without them as many as balance the two terms above (2 x 3 x 97x91, 1024 channels 11x11 / 4: 23 slices 44 us, 6
// 32; 6 x 3 x 44x44, 256 channels 11x11: 85 slices 52, 21 42; 400 layers: 7 % on average).
int slices_of(const ImageLaunch &l, int cap, bool partial)
{
    const int most = std::max(1, std::min(l.p.rows, 256 / l.ktiles));   // a workgroup per compute unit
    if (!partial) return std::max(1, std::min(most, (int)std::sqrt(l.p.rows * stage_us(l, false) / slice_us(l, false))));
    return cap > 0 ? std::min(most, cap) : most;
}

}  // namespace

bool image_wgrad_supported(const ConvGeom &g)
{
    ImageLaunch l;
    return make_problem(g, &l);
}

int image_wgrad_slices(const ConvGeom &g, int cap)
{
    ImageLaunch l;
    return make_problem(g, &l) ? slices_of(l, cap, true) : 0;
}

double image_wgrad_us(const ConvGeom &g, bool partial, int cap)
{
    ImageLaunch l;
    if (!make_problem(g, &l)) return 1e9;
    const int slices = slices_of(l, cap, partial), steps = (l.p.rows + slices - 1) / slices;
    const int strips = (steps + l.p.steps - 1) / l.p.steps;   // each starts with G - 1 groups that no step ends with
    const int ntiles = (l.p.CRS + 31) / 32;
    const double base = partial ? 9.7 + 2.4 * (l.mt - 2) + 0.03 * ntiles * l.mt / l.ks : 9.8 + 0.8e-5 * l.p.K * l.p.CRS;
    return base + (steps + (l.p.G - 1.0) * strips + 2) * stage_us(l, partial) + slices * slice_us(l, partial);
}

hipError_t launch_image_wgrad(const void *x, const void *dy, float *dw, const ConvGeom &g, float *partial, hipStream_t st, int cap)
{
    ImageLaunch l;
    if (!make_problem(g, &l)) return hipErrorInvalidValue;
    const int slices = slices_of(l, cap, partial != nullptr);
    const size_t nw = (size_t)g.K * l.p.CRS;
    const bool alone = slices == 1;   // no sum over workgroups: straight into dw
    if (!partial && !alone) {
        const hipError_t e = launch_fill_zero(dw, nw, st);
        if (e != hipSuccess) return e;
    }
    float *out = partial && !alone ? partial : dw;
    const int atomics = !partial && !alone;
    auto go = [&](auto kern) -> hipError_t {
        const hipError_t attr = kern.enable_lds(LDS_MAX);
        if (attr != hipSuccess) return attr;
        hipLaunchKernelGGL(kern.call, dim3(slices, l.ktiles), dim3(THREADS), l.lds, st, static_cast<const bf16_t *>(x),
                           static_cast<const bf16_t *>(dy), out, atomics, l.p);
        return hipGetLastError();
    };
    hipError_t e = hipErrorInvalidValue;
#define SN_IMG_K(MT_, NL_, PX_, NR_) \
    (l.ks == 1 ? go(Kernel<image_wgrad_kernel<MT_, NL_, PX_, NR_, 1>>()) : l.ks == 2 ? go(Kernel<image_wgrad_kernel<MT_, NL_, PX_, NR_, 2>>()) \
                                                                           : go(Kernel<image_wgrad_kernel<MT_, NL_, PX_, NR_, 4>>()))
#define SN_IMG_R(MT_, NL_, PX_) (l.nrow == 1 ? SN_IMG_K(MT_, NL_, PX_, 1) : SN_IMG_K(MT_, NL_, PX_, 2))
#define SN_IMG_P(MT_, NL_) (l.px == 64 ? SN_IMG_R(MT_, NL_, 64) : SN_IMG_R(MT_, NL_, 32))
#define SN_IMG(MT_) (l.nl == 2 ? SN_IMG_P(MT_, 2) : SN_IMG_P(MT_, 3))
    e = l.mt == 2 ? SN_IMG(2) : SN_IMG(3);
#undef SN_IMG
#undef SN_IMG_P
#undef SN_IMG_R
#undef SN_IMG_K
    if (e != hipSuccess) return e;
    return partial && !alone ? launch_reduce_partials(partial, dw, nw, slices, false, st) : hipSuccess;
}

}  // namespace sn
