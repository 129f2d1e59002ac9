// Host side of the channels-last implicit GEMM (see conv_chlast.h): geometry of the copies, choice of tile and
// slices, workspace needs, launches.
#include <algorithm>
#include <cmath>
#include <new>
#include "conv_chlast_kernels.h"

namespace sn {
namespace {

constexpr size_t WS_ALIGN = 256;
constexpr size_t COPY_MAX = (size_t)1 << 30;   // bytes of one pass's copy: 32-bit offsets, bit 31 marks "outside"
constexpr int GRID_Y = 65535;                  // output channels of the kernels that add up slices are rows of their grid
constexpr size_t IMAGE_MAX = (size_t)1 << 31;  // below this, bytes of a source image: likewise (a stride may leave most of it out of the copy)

// Tiles, and what they take: a workgroup alone on its compute unit needs `alone` us per stage of its reduction; with
// more workgroups than compute units, a compute unit gets through one workgroup's stage in `busy` us (fp32 first, bf16
// second).  Fitted to 2000 timings over 70 shapes (batch 1 to 128, 3 to 900 channels, planes of 7x7 to 227x227, filters
// 1x1 to 11x11), which they reproduce to 12 %; the tile picked by them is within 3 % of the best one.
struct Tile { int bm, bn, occ; double alone[2], busy[2]; };
constexpr double NEVER = 1e9;
const Tile kTile[] = {{128, 128, 2, {0.08, 0.708}, {1.96, 0.432}},
                      {64, 256, 2, {NEVER, 0.832}, {NEVER, 0.465}},
                      {64, 64, 3, {0.527, 0.217}, {0.507, 0.159}},
                      {256, 256, 1, {NEVER, 1.69}, {NEVER, 1.475}},
                      {128, 128, 1, {NEVER, 0.543}, {NEVER, 0.117}}};
constexpr int NTILE = 5;
const Tile kWTile[] = {{128, 128, 2, {NEVER, 0.279}, {NEVER, 0.210}},
                       {64, 128, 2, {NEVER, 0.011}, {NEVER, 0.183}},   // (fp32: 0.55 busy, more than two 64 x 64)
                       {64, 64, 3, {0.304, 0.154}, {0.257, 0.103}},
                       {256, 256, 1, {NEVER, 0.689}, {NEVER, 0.080}}};
constexpr int NWTILE = 4;
// us: launches; bytes per us: copies in and out, partial sums written and read, results written
constexpr double LAUNCH_US = CHLAST_LEAST_US, COPY_RATE = 5.0e6, PART_RATE = 4.6e6, OUT_RATE = 1.4e6;

double loop_us(const Tile &t, int bf16, double wgs, double steps)
{
    const double n = wgs / 256;
    return steps * std::max(t.alone[bf16] * std::ceil(n / t.occ), t.busy[bf16] * std::ceil(n));
}

struct FwdPlan {
    int Cr, M, Cp, sz;                    // reduction / output channels
    int planes, Hp, Ws, pt, pl, nimg;     // the copy; images per pass
    int ncls;
    ClClass cls[CL_MAXCLS];
    ClPackClass pcls[CL_MAXCLS];
    int in_sw, in_sh, osh, osw, OH, OW, SH, SW;   // SH, SW: source plane
    int cfg, nsplit, Mpad;
    size_t packed_bytes, copy_bytes, part_bytes;
    double us;
};

int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Geometry that does not depend on the tile.
bool fwd_geometry(const ConvGeom &g, bool bwd, FwdPlan *f)
{
    f->sz = g.in_bf16 ? 2 : 4;
    f->Cr = bwd ? g.K : g.C;
    f->M = bwd ? g.C : g.K;
    const int pe = 16 / f->sz;
    f->Cp = f->Cr <= 4 ? 4 : ceil_div(f->Cr, pe) * pe;
    if (g.in_bf16 && f->Cr > 4 && f->Cr <= 8) f->Cp = 8;
    if (!bwd) {
        f->planes = std::min(g.sh, g.R);
        f->in_sh = g.sh;
        f->in_sw = g.sw;
        f->Hp = g.P - 1 + (g.R - 1) / g.sh + 1;
        f->Ws = (g.Q - 1) * g.sw + g.S;
        f->pt = g.ph; f->pl = g.pw;
        f->SH = g.H; f->SW = g.W;
        f->OH = g.P; f->OW = g.Q;
        f->osh = f->osw = 1;
        f->ncls = 1;
        ClClass &c = f->cls[0];
        c.Rt = g.R;
        c.x_row = c.x_col = 0;
        c.nh = g.P; c.nw = g.Q;
        c.oh0 = c.ow0 = 0;
        ClPackClass &k = f->pcls[0];
        k.Rt = g.R; k.St = g.S; k.r0 = 0; k.rstep = 1; k.s0 = 0; k.sstep = 1;
        return true;
    }
    if (g.sh * g.sw > CL_MAXCLS) return false;
    f->planes = 1;
    f->in_sh = f->in_sw = 1;
    f->SH = g.P; f->SW = g.Q;
    f->OH = g.H; f->OW = g.W;
    f->osh = g.sh; f->osw = g.sw;
    int pt = 0, pl = 0, bottom = 1, right = 1;   // rows / columns of dy the classes reach: -pt .. bottom - 1
    f->ncls = 0;
    for (int pass = 0; pass < 2; ++pass) {
        for (int a = 0; a < std::min(g.sh, g.H); ++a)
            for (int b = 0; b < std::min(g.sw, g.W); ++b) {
                const int r0 = (a + g.ph) % g.sh, s0 = (b + g.pw) % g.sw;
                const int Rt = r0 < g.R ? (g.R - 1 - r0) / g.sh + 1 : 0, St = s0 < g.S ? (g.S - 1 - s0) / g.sw + 1 : 0;
                const int nh = ceil_div(g.H - a, g.sh), nw = ceil_div(g.W - b, g.sw);
                // ascending dy rows: filter rows r0 + (Rt - 1) * sh down to r0
                const int rt = r0 + (Rt - 1) * g.sh, st = s0 + (St - 1) * g.sw;
                const int o = Rt ? (a + g.ph - rt) / g.sh : 0, u = St ? (b + g.pw - st) / g.sw : 0;
                if (pass == 0) {
                    if (!Rt || !St) continue;
                    pt = std::max(pt, -o);
                    pl = std::max(pl, -u);
                    bottom = std::max(bottom, nh - 1 + o + Rt);
                    right = std::max(right, nw - 1 + u + St);
                    continue;
                }
                ClClass &c = f->cls[f->ncls];
                ClPackClass &k = f->pcls[f->ncls++];
                c.Rt = St ? Rt : 0;
                c.x_row = c.Rt ? o + pt : 0;
                c.x_col = c.Rt ? u + pl : 0;
                c.nh = nh; c.nw = nw;
                c.oh0 = a; c.ow0 = b;
                k.Rt = c.Rt; k.St = St; k.r0 = rt; k.rstep = -g.sh; k.s0 = st; k.sstep = -g.sw;
            }
    }
    f->pt = pt; f->pl = pl;
    f->Hp = pt + bottom;
    f->Ws = pl + right;
    return true;
}

void finish_classes(FwdPlan *f, int nimg)
{
    const int bm = kTile[f->cfg].bm, bn = kTile[f->cfg].bn, run = 128 / f->sz, pe = 16 / f->sz;
    f->nimg = nimg;
    f->Mpad = ceil_div(f->M, bm) * bm;
    size_t a = 0;
    int tile = 0;
    for (int i = 0; i < f->ncls; ++i) {
        ClClass &c = f->cls[i];
        ClPackClass &k = f->pcls[i];
        const int elems = k.St * f->Cp;
        c.ncks = c.Rt ? ceil_div(elems, run) : 0;
        c.tail = c.Rt ? (ceil_div(elems, pe) - 1) % 8 + 1 : 8;
        c.npix = nimg * c.nh * c.nw;
        c.a_off = (unsigned)a;
        c.tile0 = tile;
        tile += ceil_div(c.npix, bn);
        // whole channel blocks per run: the taps of a filter row that read the same channels follow one another
        const bool blocks = f->Cp % run == 0;
        c.no = blocks ? f->Cp / run : c.ncks;
        c.ni = blocks ? k.St : 1;
        if (!c.Rt) c.no = c.ni = 0;
        k.ncks = c.ncks;
        k.no = std::max(c.no, 1);
        k.ni = c.ni;
        k.a_off = c.a_off;
        k.piece0 = (int)(a / 16);
        a += (size_t)c.Rt * c.ncks * f->Mpad * 128;
    }
    f->packed_bytes = align_up(a, WS_ALIGN);
    f->copy_bytes = align_up((size_t)f->planes * nimg * f->Hp * f->Ws * f->Cp * f->sz + 256, WS_ALIGN);
}

// Tile and slices for nimg images: the least estimated time (us, for one pass).
void choose(FwdPlan *f, int nimg, size_t part_limit)
{
    const int bf16 = f->sz == 2, run = 128 / f->sz;
    f->us = -1;
    for (int c = 0; c < NTILE; ++c) {
        const Tile &k = kTile[c];
        if (k.alone[bf16] >= NEVER) continue;
        const int mt = ceil_div(f->M, k.bm);
        double work = 0, wgs = 0, npix = 0, longest = 0;   // work: workgroup stages, a half stage counted as half
        int most = 0;
        for (int i = 0; i < f->ncls; ++i) {
            const int elems = f->pcls[i].St * f->Cp, Rt = f->cls[i].Rt;
            const double half = Rt * ceil_div(elems, run / 2) * 0.5, np = (double)nimg * f->cls[i].nh * f->cls[i].nw;
            const double t = std::ceil(np / k.bn) * mt;
            wgs += t;
            npix += np;
            work += t * half;
            longest = std::max(longest, half);
            most = std::max(most, Rt * ceil_div(elems, run));
        }
        const double copy = (double)nimg * (f->Cr * (double)f->SH * f->SW + (double)f->planes * f->Hp * f->Ws * f->Cp) * f->sz;
        for (int s = 1; s <= 16; s = s < 4 ? s + 1 : s * 2) {
            if (s > 1 && (f->ncls > 1 || most / s < 4 || f->M > GRID_Y)) break;
            const double pb = s > 1 ? (double)s * f->M * npix * 4 : 0;
            if (pb > part_limit) break;
            double t = std::max(loop_us(k, bf16, wgs * s, work / wgs / s), 0.9 * longest / s * k.alone[bf16]);
            t += LAUNCH_US + copy / COPY_RATE + f->M * npix * f->sz / OUT_RATE;
            if (s > 1) t += 2 + 2 * pb / PART_RATE;
            if (f->us < 0 || t < f->us) { f->us = t; f->cfg = c; f->nsplit = s; }
        }
    }
}

size_t fwd_bytes(FwdPlan *f, int nimg)
{
    finish_classes(f, nimg);
    f->part_bytes = f->nsplit > 1 ? align_up((size_t)f->nsplit * f->M * f->cls[0].npix * 4, WS_ALIGN) : 0;
    return f->packed_bytes + f->copy_bytes + f->part_bytes;
}

// The plan under a budget: the fewest passes that fit (halving); false if not even one image does.
bool fwd_plan(const ConvGeom &g, bool bwd, size_t budget, FwdPlan *f)
{
    if (!fwd_geometry(g, bwd, f) || (size_t)f->Cr * f->SH * f->SW * f->sz >= IMAGE_MAX) return false;
    const size_t per = (size_t)f->planes * f->Hp * f->Ws * f->Cp * f->sz;
    if (per > COPY_MAX) return false;
    const int cap = (int)std::min<size_t>(g.N, COPY_MAX / per);
    for (int parts = ceil_div(g.N, cap);; parts = std::min(g.N, 2 * parts)) {   // passes of equal size
        const int nimg = ceil_div(g.N, parts);
        for (size_t limit = (size_t)64 << 20;; limit = 0) {   // with partial sums if they fit, else without
            choose(f, nimg, limit);
            if (fwd_bytes(f, nimg) <= budget) {
                f->us *= ceil_div(g.N, nimg);
                return f->packed_bytes < ((size_t)1 << 31);
            }
            if (limit == 0) break;
        }
        if (nimg == 1) return false;
    }
}

ClStage stage_job(const void *src, void *dst, int C, int H, int W, int nimg, int planes, int sh, int pt, int pl, int Hp, int Ws,
                  int Cp, int sz)
{
    ClStage s;
    s.src = src; s.dst = dst;
    s.C = C; s.H = H; s.W = W; s.nimg = nimg; s.sh = sh; s.pt = pt; s.pl = pl; s.Hp = Hp; s.Ws = Ws; s.Cp = Cp;
    const int pe = 16 / sz;
    const long long px = (long long)Hp * Ws;
    if (Cp <= pe) { s.ptiles = (int)((px + 255) / 256); s.ctiles = 1; }
    else { s.ptiles = (int)((px + 63) / 64); s.ctiles = ceil_div(Cp / pe, 8); }
    s.blocks = s.ptiles * s.ctiles * nimg * planes;
    return s;
}

template <typename T, int BM, int BN, int WM, int WN, int NST, bool HALF>
hipError_t launch_gemm_as(const void *xs, const void *ap, void *y, float *part, const ClGemm &p, hipStream_t st)
{
    constexpr int lds = NST * (BM + BN) * 128;
    auto kern = cl_gemm_kernel<T, BM, BN, WM, WN, NST, HALF>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(kern, dim3(8 * p.ppx * p.mtiles, p.nsplit), dim3(64 * WM * WN), lds, st, static_cast<const T *>(xs),
                       static_cast<const T *>(ap), y, part, p);
    return hipGetLastError();
}

template <typename T, int BM, int BN, int WM, int WN, int NST>
hipError_t launch_gemm(const void *xs, const void *ap, void *y, float *part, const ClGemm &p, int half, hipStream_t st)
{
    if constexpr (sizeof(T) == 2)
        if (half) return launch_gemm_as<T, BM, BN, WM, WN, NST, true>(xs, ap, y, part, p, st);
    return launch_gemm_as<T, BM, BN, WM, WN, NST, false>(xs, ap, y, part, p, st);
}

template <typename T>
hipError_t launch_cfg(int cfg, const void *xs, const void *ap, void *y, float *part, const ClGemm &p, int half, hipStream_t st)
{
    if (cfg == 0) return launch_gemm<T, 128, 128, 2, 2, 2>(xs, ap, y, part, p, half, st);
    if (cfg == 2) return launch_gemm<T, 64, 64, 2, 2, 3>(xs, ap, y, part, p, half, st);
    if constexpr (sizeof(T) == 2) {
        if (cfg == 1) return launch_gemm<T, 64, 256, 1, 4, 2>(xs, ap, y, part, p, half, st);
        if (cfg == 3) return launch_gemm<T, 256, 256, 2, 4, 2>(xs, ap, y, part, p, half, st);
        if (cfg == 4) return launch_gemm<T, 128, 128, 2, 4, 4>(xs, ap, y, part, p, half, st);
    }
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t run_fwd(const void *in, const void *w, void *out, const ConvGeom &g, bool bwd, FwdPlan &f, void *ws, hipStream_t st)
{
    char *packed = static_cast<char *>(ws), *copy = packed + f.packed_bytes;
    float *part = reinterpret_cast<float *>(copy + f.copy_bytes);
    const int chunk = f.nimg, T_ = g.R * g.S;
    for (int n0 = 0; n0 < g.N; n0 += chunk) {
        const int nimg = std::min(chunk, g.N - n0);
        fwd_bytes(&f, nimg);   // tile counts of this pass (the layout is the full pass's)
        ClPrep pr = {};
        const size_t src_img = (size_t)f.Cr * f.SH * f.SW * f.sz, dst_img = (size_t)f.M * f.OH * f.OW * (g.out_bf16 ? 2 : 4);
        pr.st[0] = stage_job(static_cast<const char *>(in) + n0 * src_img, copy, f.Cr, f.SH, f.SW, nimg, f.planes, f.in_sh, f.pt, f.pl,
                             f.Hp, f.Ws, f.Cp, f.sz);
        if (n0 == 0) {
            ClPack &k = pr.pk;
            k.w = w; k.dst = packed;
            k.M = f.M; k.Red = f.Cr; k.Cp = f.Cp; k.Mpad = f.Mpad;
            k.w_sm = bwd ? T_ : g.C * T_;
            k.w_sr = bwd ? g.C * T_ : T_;
            k.R = g.R; k.S = g.S;
            k.ncls = f.ncls;
            k.mfast = bwd;
            k.pieces = 0;
            for (int i = 0; i < f.ncls; ++i) {
                k.cls[i] = f.pcls[i];
                k.pieces += f.cls[i].Rt * f.cls[i].ncks * f.Mpad * 8;
            }
            k.blocks = ceil_div(k.pieces, 256);
        }
        hipLaunchKernelGGL(cl_prep_kernel<T>, dim3(pr.pk.blocks + pr.st[0].blocks), dim3(256), 0, st, pr);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        ClGemm p = {};
        p.M = f.M; p.Mpad = f.Mpad;
        p.mtiles = f.Mpad / kTile[f.cfg].bm;
        p.ncls = f.ncls;
        long long np = 0;
        for (int i = 0; i < f.ncls; ++i) {
            p.cls[i] = f.cls[i];
            np += f.cls[i].npix;
        }
        const ClClass &last = f.cls[f.ncls - 1];
        p.ptiles = last.tile0 + ceil_div(last.npix, kTile[f.cfg].bn);
        p.ppx = ceil_div(p.ptiles, 8);
        p.Hp = f.Hp; p.Ws = f.Ws; p.Cp = f.Cp; p.in_sw = f.in_sw; p.sh = f.in_sh;
        p.plane_bytes = (unsigned)((size_t)nimg * f.Hp * f.Ws * f.Cp * f.sz);
        p.x_bytes = (unsigned)((size_t)f.planes * p.plane_bytes);
        p.a_bytes = (unsigned)f.packed_bytes;
        p.OH = f.OH; p.OW = f.OW; p.osh = f.osh; p.osw = f.osw;
        p.out_bf16 = g.out_bf16;
        p.pair = g.out_bf16 && f.ncls == 1 && f.osh == 1 && f.osw == 1 && (f.OH * f.OW) % 2 == 0;
        int half = 0;   // a run ends half way through a piece (4 channels per pixel, bf16)
        for (int i = 0; i < f.ncls; ++i) half |= f.pcls[i].St * f.Cp % (16 / f.sz) != 0;
        p.nsplit = f.nsplit;
        p.nptot = (int)np;
        char *o = static_cast<char *>(out) + n0 * dst_img;
        e = launch_cfg<T>(f.cfg, copy, packed, o, part, p, half, st);
        if (e != hipSuccess) return e;
        if (f.nsplit > 1) {
            const dim3 grid((unsigned)((np + 255) / 256), f.M);
            if (g.out_bf16) hipLaunchKernelGGL(cl_reduce_kernel<true>, grid, dim3(256), 0, st, part, o, f.M, (int)np, f.OH * f.OW, f.nsplit);
            else hipLaunchKernelGGL(cl_reduce_kernel<false>, grid, dim3(256), 0, st, part, o, f.M, (int)np, f.OH * f.OW, f.nsplit);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

// ---- backward-filter -----------------------------------------------------------------------------------------
struct WPlan {
    int sz, Cp, Kp, SC, ncols, planes, Pp, Qp, Ws, pix;
    int nimg, passes, nflat, steps, want, nsl, sps, cfg;
    size_t x_bytes, x_all, d_bytes, d_all, part_bytes;
    double us;
};

bool w_geometry(const ConvGeom &g, WPlan *f)
{
    f->sz = g.in_bf16 ? 2 : 4;
    const int pe = 16 / f->sz;
    f->pix = g.in_bf16 ? 32 : 16;
    f->Cp = g.C <= 4 ? 4 : ceil_div(g.C, pe) * pe;
    f->Kp = ceil_div(g.K, pe) * pe;
    f->SC = ceil_div(g.S * f->Cp, pe) * pe;
    f->ncols = g.R * f->SC;
    f->planes = std::min(g.sh, g.R);
    const int rows = (g.P - 1) * g.sh + g.R, cols = (g.Q - 1) * g.sw + g.S;
    // With one row phase an image's rows below its last one may be the next image's padding above its first; with
    // several they are stored.  Columns to the right of a row may always be the next row's padding on its left.
    const int hs = g.sh == 1 ? std::max(std::min(g.H + g.ph, rows), rows - g.ph) : rows;
    const int ws = std::max(std::min(g.W + g.pw, cols), cols - g.pw);
    f->Pp = std::max(g.P, ceil_div(hs, g.sh));
    f->Qp = std::max(g.Q, ceil_div(ws, g.sw));
    f->Ws = f->Qp * g.sw;
    return true;
}

size_t w_bytes(const ConvGeom &g, WPlan *f, int nimg)
{
    f->nimg = nimg;
    f->passes = ceil_div(g.N, nimg);
    f->nflat = nimg * f->Pp * f->Qp;
    f->steps = ceil_div(f->nflat, f->pix);
    const size_t plane = (size_t)nimg * f->Pp * f->Ws * f->Cp * f->sz;
    f->x_bytes = plane * f->planes;
    const size_t slack = ((size_t)((g.R - 1) / g.sh) * f->Ws * f->Cp + f->SC + (size_t)f->pix * g.sw * f->Cp) * f->sz + 16;
    f->x_all = align_up(f->x_bytes + slack, WS_ALIGN);
    f->d_bytes = (size_t)f->nflat * f->Kp * f->sz;
    f->d_all = align_up(f->d_bytes + (size_t)f->pix * f->Kp * f->sz, WS_ALIGN);
    int want = std::min(f->want, std::max(1, f->steps / 4));
    if (want > 8) want = want / 8 * 8;
    f->sps = ceil_div(f->steps, want);
    f->nsl = want;
    while (f->nsl > 1 && (long long)(f->nsl - 1) * f->sps >= f->steps) --f->nsl;
    f->part_bytes = align_up((size_t)f->passes * f->nsl * g.K * f->ncols * 4, WS_ALIGN);
    return f->x_all + f->d_all + f->part_bytes;
}

// Tile, slices and passes over parts of the batch: the least estimated time among those that fit (small passes leave room
// for partial sums).
bool w_plan(const ConvGeom &g, size_t budget, WPlan *f)
{
    if (g.K > GRID_Y || !w_geometry(g, f) || std::max((size_t)g.C * g.H * g.W, (size_t)g.K * g.P * g.Q) * f->sz >= IMAGE_MAX) return false;
    const size_t per = (size_t)f->planes * f->Pp * f->Ws * f->Cp * f->sz, dper = (size_t)f->Pp * f->Qp * f->Kp * f->sz;
    if (std::max(per, dper) > COPY_MAX) return false;
    const int cap = (int)std::min<size_t>(g.N, COPY_MAX / std::max(per, dper)), bf16 = f->sz == 2;
    WPlan best = *f;
    best.us = -1;
    int tried = 0;
    for (int parts = ceil_div(g.N, cap); tried < 3; parts = std::min(g.N, parts * 2)) {
        const int nimg = ceil_div(g.N, parts);
        for (int c = 0; c < NWTILE; ++c) {
            const Tile &k = kWTile[c];
            if (k.alone[bf16] >= NEVER) continue;
            const double tiles = (double)ceil_div(g.K, k.bm) * ceil_div(f->ncols, k.bn);
            for (int want = 1; want <= 256; want *= 2) {
                f->cfg = c;
                f->want = want;
                if (w_bytes(g, f, nimg) > budget) break;
                const double copy = (double)nimg * (g.C * (double)g.H * g.W + g.K * (double)g.P * g.Q) * f->sz + f->x_bytes + f->d_bytes;
                const double t = f->passes * (LAUNCH_US + copy / COPY_RATE + loop_us(k, bf16, tiles * f->nsl, f->sps)) +
                                 2.0 * f->part_bytes / PART_RATE + 1.5;
                if (best.us < 0 || t < best.us) { best = *f; best.us = t; }
                if (f->nsl < want) break;
            }
        }
        if (best.us >= 0) ++tried;
        if (parts == g.N) break;
    }
    *f = best;
    return best.us >= 0;
}

template <typename T, int BM, int BN, int WM, int WN, int NST>
hipError_t launch_wgemm(const void *ds, const void *xs, float *part, const ClWgrad &p, hipStream_t st)
{
    constexpr int lds = NST * (sizeof(T) == 2 ? 32 : 16) * (BM + BN) * (int)sizeof(T);
    auto kern = cl_wgrad_kernel<T, BM, BN, WM, WN, NST>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(kern, dim3(p.ktiles * p.jtiles * p.nsl), dim3(64 * WM * WN), lds, st, static_cast<const T *>(ds),
                       static_cast<const T *>(xs), part, p);
    return hipGetLastError();
}

template <typename T>
hipError_t run_wgrad(const void *x, const void *dy, float *dw, const ConvGeom &g, WPlan &f, void *ws, hipStream_t st)
{
    char *xs = static_cast<char *>(ws), *ds = xs + f.x_all;
    float *part = reinterpret_cast<float *>(ds + f.d_all);
    const int chunk = f.nimg;
    int slices = 0;
    for (int n0 = 0; n0 < g.N; n0 += chunk) {
        const int nimg = std::min(chunk, g.N - n0), full_nsl = f.nsl;
        WPlan q = f;
        if (nimg != chunk) {
            w_bytes(g, &q, nimg);
            if (q.nsl > full_nsl) { q.nsl = full_nsl; q.sps = ceil_div(q.steps, q.nsl); }
        }
        ClPrep pr = {};
        pr.st[0] = stage_job(static_cast<const char *>(x) + (size_t)n0 * g.C * g.H * g.W * f.sz, xs, g.C, g.H, g.W, nimg, f.planes, g.sh,
                             g.ph, g.pw, f.Pp, f.Ws, f.Cp, f.sz);
        pr.st[1] = stage_job(static_cast<const char *>(dy) + (size_t)n0 * g.K * g.P * g.Q * f.sz, ds, g.K, g.P, g.Q, nimg, 1, 1, 0, 0, f.Pp,
                             f.Qp, f.Kp, f.sz);
        pr.zero[0] = xs + q.x_bytes;   // (a copy of few channels may end half way through an item)
        pr.zero_items[0] = (int)((q.x_all - q.x_bytes) / 16);
        pr.zero[1] = ds + q.d_bytes;
        pr.zero_items[1] = (int)((q.d_all - q.d_bytes) / 16);
        const int zb = ceil_div(pr.zero_items[0] + pr.zero_items[1], 256);
        hipLaunchKernelGGL(cl_prep_kernel<T>, dim3(pr.st[0].blocks + pr.st[1].blocks + zb), dim3(256), 0, st, pr);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        ClWgrad p = {};
        p.K = g.K; p.ncols = f.ncols; p.Kp = f.Kp; p.Cp = f.Cp; p.SC = f.SC; p.in_sw = g.sw; p.sh = g.sh; p.Ws = f.Ws;
        p.plane_bytes = (unsigned)(q.x_bytes / f.planes);
        p.x_bytes = (unsigned)q.x_all;
        p.d_bytes = (unsigned)q.d_all;
        p.P = g.P; p.Q = g.Q; p.Pp = f.Pp; p.Qp = f.Qp;
        p.holes = f.Pp != g.P || f.Qp != g.Q;
        p.dp = f.pix / f.Qp % f.Pp; p.dq = f.pix % f.Qp;
        p.steps = q.steps; p.sps = q.sps; p.nsl = q.nsl;
        p.ktiles = ceil_div(g.K, kWTile[f.cfg].bm);
        p.jtiles = ceil_div(f.ncols, kWTile[f.cfg].bn);
        p.slice0 = slices;
        slices += q.nsl;
        e = hipErrorInvalidValue;
        if (f.cfg == 2) e = launch_wgemm<T, 64, 64, 2, 2, 4>(ds, xs, part, p, st);
        if constexpr (sizeof(T) == 2) {
            if (f.cfg == 1) e = launch_wgemm<T, 64, 128, 2, 2, 4>(ds, xs, part, p, st);
            else if (f.cfg == 0) e = launch_wgemm<T, 128, 128, 2, 2, 4>(ds, xs, part, p, st);
            else if (f.cfg == 3) e = launch_wgemm<T, 256, 256, 2, 4, 4>(ds, xs, part, p, st);
        }
        if (e != hipSuccess) return e;
    }
    if (slices > 8)
        hipLaunchKernelGGL(cl_wgrad_reduce_kernel<4>, dim3(ceil_div(f.ncols, 64), g.K), dim3(256), 0, st, part, dw, g.K, g.C, g.R, g.S, f.Cp,
                           f.SC, f.ncols, slices);
    else
        hipLaunchKernelGGL(cl_wgrad_reduce_kernel<1>, dim3(ceil_div(f.ncols, 256), g.K), dim3(256), 0, st, part, dw, g.K, g.C, g.R, g.S, f.Cp,
                           f.SC, f.ncols, slices);
    return hipGetLastError();
}

}  // namespace

static_assert(sizeof(FwdPlan) <= sizeof(ChlastPlan::mem) && sizeof(WPlan) <= sizeof(ChlastPlan::mem), "plans fit their opaque form");

bool chlast_plan(const ConvGeom &g, int dir, size_t budget, ChlastPlan *plan)
{
    if (dir == SN_CONV_BWD_FILTER) {
        WPlan &f = *new (plan->mem) WPlan;
        if (!w_plan(g, budget, &f)) return false;
        plan->bytes = f.x_all + f.d_all + f.part_bytes;
        plan->passes = f.passes;
        plan->us = f.us;
        return true;
    }
    FwdPlan &f = *new (plan->mem) FwdPlan;
    if (!fwd_plan(g, dir == SN_CONV_BWD_DATA, budget, &f)) return false;
    plan->bytes = f.packed_bytes + f.copy_bytes + f.part_bytes;
    plan->passes = ceil_div(g.N, f.nimg);
    plan->us = f.us;
    return true;
}

void chlast_config(const ChlastPlan &plan, int dir, int *tile_m, int *tile_n, int *threads, int *slices)
{
    const bool w = dir == SN_CONV_BWD_FILTER;
    const WPlan &f = *reinterpret_cast<const WPlan *>(plan.mem);
    const FwdPlan &d = *reinterpret_cast<const FwdPlan *>(plan.mem);
    const int cfg = w ? f.cfg : d.cfg;
    const Tile &t = w ? kWTile[cfg] : kTile[cfg];
    *tile_m = t.bm;
    *tile_n = t.bn;
    *threads = cfg >= 3 ? 512 : 256;
    *slices = w ? f.nsl : d.nsplit;
}

hipError_t launch_chlast(const void *a, const void *b, void *out, const ConvGeom &g, int dir, void *ws, ChlastPlan *plan, hipStream_t st)
{
    if (dir == SN_CONV_BWD_FILTER) {
        WPlan &f = *reinterpret_cast<WPlan *>(plan->mem);
        return g.in_bf16 ? run_wgrad<bf16_t>(a, b, static_cast<float *>(out), g, f, ws, st)
                         : run_wgrad<float>(a, b, static_cast<float *>(out), g, f, ws, st);
    }
    FwdPlan &f = *reinterpret_cast<FwdPlan *>(plan->mem);
    const bool bwd = dir == SN_CONV_BWD_DATA;
    return g.in_bf16 ? run_fwd<bf16_t>(a, b, out, g, bwd, f, ws, st) : run_fwd<float>(a, b, out, g, bwd, f, ws, st);
}

}  // namespace sn
