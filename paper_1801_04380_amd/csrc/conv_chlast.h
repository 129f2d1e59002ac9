// Implicit GEMM over a channels-last copy of the input (gfx950): the kernels.  Host side in conv_chlast.hip.
//
// The NCHW tensor puts the pixels of a channel next to each other; the MFMA wants runs of reduction
// elements (channels) per pixel.  Everything the other kernels do to bridge that -- patches cut out and
// transposed in LDS, tap by tap, for one filter size and stride 1 -- is done here once, by a copy of the
// input (forward), of dy (backward-data) or of both (backward-filter) in the caller's workspace:
//   [row phase h mod stride][image][row][column][channel], zero padded all around.
// After it every convolution is a matrix product whose operand rows are plain addresses:
//   * Output pixel j and filter row r: the S * Cp elements under the filter row are ONE contiguous run of the
//     copy, starting at an address that is linear in (pixel, r).  The reduction is cut into runs of 128 bytes of
//     it, walked channel block by channel block with all taps of a block in a row, so that the taps' overlapping
//     reads meet in the caches; a lane's offset is a constant per pixel, the filter row and the run are one scalar offset.  No tap
//     is an exception (padding is real zeros), no filter size or stride has a kernel of its own, and channel
//     counts only round up to a multiple of 8 (4 for fp32 and for images of up to 4 channels).
//   * Operands travel global memory -> LDS without passing through registers (16 bytes per lane), into a ring of
//     stages; a row's eight 16-byte pieces are permuted by XOR with bits of the row number (on the global side, as
//     the LDS side is fixed lane order), so that the 16-byte operand reads spread over all banks.
//   * One barrier per stage: wait for the wave's own loads of the stage, barrier, issue the loads of the stage
//     NST - 1 ahead into the buffer everyone has just left, multiply.
//   * Backward-data with strides: the input pixels of one residue class (h mod sh, w mod sw) share their taps, and
//     are a stride-1 problem over dy; all classes run in one launch.
//   * Backward-filter: dy and x in copies of the same pitch, so that one flat pixel index addresses both: dw[k][r,s,c]
//     = sum over the flat index of dy[i][k] * x[i + tap][c], a product with the reduction along the rows of
//     both copies.  bf16 operands come out of LDS through the transposing read (ds_read_b64_tr_b16).
#pragma once
#include "sn_internal.h"

namespace sn {

constexpr int CL_MAXCLS = 16;   // residue classes of a strided backward-data

struct ClStage {                // one copy job: NCHW -> the channels-last copy
    const void *src;
    void *dst;
    int C, H, W;                // source planes
    int nimg;
    int sh;                     // row phases
    int pt, pl;                 // rows above / columns left of the image in the copy
    int Hp, Ws;                 // rows per phase and image, columns
    int Cp;                     // channels per pixel, rounded up
    int blocks;                 // workgroups of the job
    int ptiles, ctiles;         // pixel tiles per (phase, image), channel tiles
};

struct ClPackClass {            // one class's filter taps
    int Rt, St;                 // taps along rows / columns
    int r0, rstep, s0, sstep;   // filter row of row tap t: r0 + t * rstep, column likewise
    int ncks, no, ni;           // runs per row tap, as ClClass
    unsigned a_off;             // bytes into the packed filter
    int piece0;                 // first 16-byte item of the class
};

struct ClPack {                 // filter packing: [class][stage][Mpad][128 bytes]
    const void *w;
    void *dst;
    int M, Red, Cp, Mpad;       // output channels, reduction channels
    int w_sm, w_sr, R, S;       // strides of an output / reduction channel in w, in elements; filter size
    int ncls, pieces, blocks, mfast;
    ClPackClass cls[CL_MAXCLS];
};

struct ClPrep {
    ClStage st[2];
    ClPack pk;
    void *zero[2];              // the ends of the backward-filter's copies: what the last stages read past the pixels
    int zero_items[2];          // 16-byte items
};

struct ClClass {
    int Rt, ncks, tail;         // row taps, runs per row tap, valid 16-byte pieces of the last run
    int no, ni;                 // stages: for o < no, for row taps, for i < ni: run i * no + o
    unsigned a_off;             // packed filter of the class
    int x_row, x_col;           // copy row / column of output pixel (0, 0)'s first tap
    int nh, nw, npix;           // output pixels per image of the class, over all images of the pass
    int oh0, ow0;               // first output pixel
    int tile0;                  // first pixel tile of the class
};

struct ClGemm {
    int M, Mpad, mtiles, ptiles, ppx;   // ppx: pixel tiles per XCD
    int ncls;
    ClClass cls[CL_MAXCLS];
    int Hp, Ws, Cp, in_sw, sh;          // the copy; in_sw: copy columns per output column, sh: row phases
    unsigned plane_bytes;
    unsigned x_bytes, a_bytes;
    int OH, OW, osh, osw;               // output plane and the spacing of a class's pixels in it
    int out_bf16, pair;                 // pair: 4-byte stores of two neighbouring bf16 pixels
    int nsplit, nptot;                  // reduction slices; row length of a slice's partial sums
};

struct ClWgrad {
    int K, ncols;               // rows of dw, columns R * S * Cp
    int Kp;                     // channels per pixel of the dy copy
    int Cp, SC;                 // of the x copy; S * Cp
    int in_sw, sh;
    int Ws;                     // columns of the x copy
    unsigned plane_bytes, x_bytes, d_bytes;
    int P, Q, Pp, Qp;           // output plane, and its pitch in the copies
    int holes, dp, dq;          // whether the pitch is larger; rows (mod Pp) and columns of the pitch that a stage's pixels are
    int steps, sps;             // reduction stages in all, per slice
    int ktiles, jtiles, nsl;    // tiles, slices of this launch
    int slice0;                 // first slice's number among all partial sums
};

}  // namespace sn
