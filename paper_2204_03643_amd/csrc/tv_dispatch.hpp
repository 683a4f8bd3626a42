// Every size at which the library switches from one kernel mapping to another, in one place,
// each with the measurement that set it (one MI355X; times in microseconds, forward unless
// noted).  They are crossover points of two ways to compute the same minimiser: results agree to
// rounding, not bit for bit.  The values are variables so that the benchmark can time both sides
// of a threshold at the threshold (tv_dispatch_override); nothing else writes them.
#pragma once
#include <stdint.h>

namespace tvd {

struct Threshold {
    const char *name;
    int64_t     value;
    const char *what;
};

// Index constants of `table` below.
enum {
    kStreamBytes = 0,
    kOrderMinRows,
    kFused32FullPlanes,
    kFused32FullPlanesK2,
    kFused32FullPlanesK3,
    kFused32RaggedPlanes,
    kFused16OneSweepPlanes,
    kFused16DensePlanes,
    kPlanePerGroupPlanes,
    kPlanePerGroup64Planes,
    kPlanePerGroup64PlanesK2,
    kPlanePerGroup64FullPlanesK2,
    kPlanePerGroup64FullPlanesK3,
    kPlanePerGroup64FullPlanesK5,
    kPair2dPlanes,
    kPair2dManyPlanes,
    kPlanePerGroupBwdPlanes,
    kPlanePerGroup64BwdPlanes,
    kPlanePerGroup64BwdRaggedPlanes,
    kPlanePerGroup64BwdRaggedPlanesK2,
    kFusedKeepsPasses,
    kChunkCodesBytes,
    kThreadPerSampleWideRows,
    kThreadPerSample1dRows,
    kPair1dRows,
    kPair1dLongRows,
    kWavePerRowRows,
    kOneLambdaTriSide,
    kMlMinLength,
    kMlCoarsest,
    kBwdFewColumns,
    kCount
};

inline Threshold table[kCount] = {
    // A tensor of this many bytes or more is touched once per call and does not survive in the
    // 256 MB last-level cache until the next call; its 16-byte accesses are marked non-temporal.
    // 128 MiB tensors, forward + backward: 147 -> 136 with the hint; 64 MiB: 104 with it against 100
    // without; 32 MiB: 74 against 72; 16 MiB tensors (the 2D workloads, re-read by the next pass):
    // 3-9 % slower with it.
    {"stream_bytes", (int64_t)96 << 20, "non-temporal accesses from this tensor size on"},
    // The slot order of the row-per-lane forward kernel costs a 5 us kernel of one workgroup and
    // shortens the drain of the main kernel.  It paid while single rows of a wave could take 16
    // Newton iterations; since clipped trial points are polished and rows stop on their Newton
    // decrement, the slowest wave of a slot is no longer far from the others, and the order gains
    // about 1 us: 2^20 rows x 32, forward + backward alternating, 124 natural order / 128 with
    // the slot order; with the lambdas sorted along the slots 121 / 126 (ascending), 119 / 130
    // (descending); with the expensive slots last 125 / 129.  The library still computes the
    // order whenever it is handed the workspace; the layer (layer.py) would hand it over from
    // this many rows on, and the value means "never".
    {"order_min_rows", (int64_t)1 << 40, "the layer passes the slot-order workspace from this many rows on"},
    // 2D, planes of 17-32 samples a side: the one-launch forward with two lanes a row (tv_pair.hpp, four
    // waves per SIMD) against pass by pass.  N(0, 1), lambda 10^U(-1.3, 0), forward:
    //   32 x 32, K = 1: 4096 planes 33 / 53,  8192: 59 / 71, 65 536: 393 / 429;  K = 2: 65 536 planes 696 / 864;
    //   28 x 28, K = 1: 16 384 planes 98 / 111, 65 536: 348 / 392;  20 x 20, K = 1: 16 384 planes 61 / 76.
    // So for planes that fill, or nearly fill, their square the one launch wins at every count, and with two sweeps or
    // more it does for every plane: the first three values mean "always".
    {"fused32_full_planes", (int64_t)1 << 40, "2D planes of 17-32 a side, the shorter at least 15/16 of the longer, one sweep: all passes in one launch up to this many planes"},
    {"fused32_full_planes_k2", (int64_t)1 << 40, "2D planes of 32 x 32, two sweeps: one launch up to this many planes"},
    {"fused32_full_planes_k3", (int64_t)1 << 40, "... three sweeps or more"},
    // Other planes leave lanes idle, a wave being a plane whatever it holds, and with one sweep there is
    // little to save.  K = 1, one launch / pass by pass, and / pass by pass with a row per lane:
    //   20 000 planes:  1 x 32: 83 / 22 / 28,  8 x 32: 112 / 41 / 49,  32 x 16: 146 / 66 / 83,  10 x 20: 75 / - / 68,  20 x 28: 0.87 of it;
    //   12 288 planes: 24 x 32 0.93 / 1.24 of it, 20 x 28 0.95 / 1.42, 16 x 20 0.69 / 1.81, 1 x 32 0.34 / 1.33;
    //   80 000 planes:  1 x 32: 295 / 44 / 47,  16 x 24: 0.47 / 0.98 of it,  20 x 32: 0.76 / 0.80.
    // (The line is where it was with a row per lane; for the thinnest planes it could lie lower.)
    {"fused32_ragged_planes", 12288, "2D planes with a longer side of 17-32 and a shorter below 15/16 of it (or below 17), one sweep: one launch up to this many planes"},
    // 2D, planes of 9-16 samples a side, single sweep, forward + backward, one launch against pass
    // by pass: 16 x 16, 24 576 planes 67 / 73, 49 152: 101 / 107, 98 304: 178 / 180, 262 144: 445 / 500;
    // 14 x 14, 49 152 planes 111 / 118, 262 144: 507 / 579 (the value means "always").
    {"fused16_one_sweep_planes", (int64_t)1 << 40, "2D planes of at most 16 x 16, one sweep: one launch up to this many planes"},
    // ... and from this many planes on the one-launch kernel for planes of 9-16 a side is the
    // variant held to 128 VGPRs, four waves per SIMD (planes that do not fill their square take 129
    // left alone; 16 384 planes of 14 x 14, K = 4: 101 us against 78).  The crossover is where the
    // waves, 4 planes each, outnumber three per SIMD.
    {"fused16_dense_planes", 12288, "2D planes of 9-16 a side in one launch: the four-waves-per-SIMD variant from this many planes on"},
    // 2D, small batches: one plane per workgroup of 512 threads, resident in LDS for all passes,
    // 16 threads x 2 samples per row (sides of 17-32) or 8 x 8 (sides of 33-64); tv_plane2d.hpp.
    // A lone wave per SIMD of a kernel with few lanes a row issues an instruction every 9 cycles, and
    // pass by pass a small batch pays a launch and a trip through memory per pass; this mapping has 4x the
    // waves of two lanes a row, short chains and one launch.  Its time is set by the slowest row of each
    // pass (a barrier between passes), so it stops paying once the other kernels fill the chip.  Sides of
    // 17-32, this kernel / two lanes a row, N(0, 1), lambda 0.3 and 10^U(-1.3, 0), forward:
    //   32 x 32, K = 1: 512 planes 13 / 16, 16 / 20,   768: 16 / 16, 20 / 21,  1024: 19 / 16, 25 / 21;
    //            K = 4: 768 planes 42 / 48, 52 / 58,  1024: 51 / 47, 63 / 57;
    //   28 x 28, K = 1: 512 planes 12 / 14, 15 / 19,   768: 16 / 15, 20 / 19;
    //            K = 4: 768 planes 41 / 41, 49 / 55,  1024: 49 / 41, 59 / 55;
    //   20 x 30, K = 4: 1024 planes 46 / 51, 54 / 60, 1280: 57 / 58, 68 / 70.
    // (With two sweeps or more the library takes a third more planes than the value says.)
    // Planes with one side of 29-32 that are no squares take three quarters more: two lanes a row lie in halves of
    // 16 and leave what the shorter side lacks idle.  This kernel / two lanes a row:
    //   1 x 32, K = 1: 800 planes 11 / 15, 1200: 14 / 15, 1536: 16 / 17;  8 x 32: 800: 16 / 18, 1000: 17 / 18, 1300: 22 / 23;
    //   32 x 16: 800 planes 20 / 23, 1200: 24 / 25;  K = 4: 1000: 47 / 53, 1200: 0.96 of it, 1536: 1.07 of it;
    //   20 x 32: 1000 planes 21 / 23, 1300: 1.04 of it;  28 x 32, K = 4: 1000: 0.91 of it, 1200: 0.95, 1536: 1.11.
    {"plane_per_group_planes", 768, "2D planes of 17-32 a side: one launch, a plane per workgroup, up to this many planes (a third more: two sweeps and more; three quarters more: one side of 29-32, no square)"},
    //   64 x 64, K = 1:  512 planes  47 /  50,  768:  67 /  60, 1024:  78 /  73, 1536: 109 / 94;
    //   48 x 48, K = 1:  512 planes  35 /  38,  768:  55 /  54, 1024:  64 /  57.
    // (With row masks, forward + reverse sweep: 600 planes of 45 x 45 59 / 57, 560 of 64 x 64 57 / 61.)
    {"plane_per_group64_planes", 512, "2D planes of 33-64 a side, one sweep: one launch, a plane per workgroup, up to this many planes"},
    // Several sweeps, forward + reverse sweep, ratio of this kernel to pass by pass on post-ReLU
    // maps and on N(0, 1) data:
    //   48 x 48, K = 2: 1024 planes 0.95 1.01, 1280: 1.02 1.06, 1536: 1.06 1.07;
    //            K = 4: 1280 planes 0.93 0.99, 1536: 0.97 1.01, 2048: 1.05 1.07;
    //   64 x 40, K = 3: 1280 planes 0.93 0.99, 1536: 0.96 1.01, 2048: 1.04 1.06.
    {"plane_per_group64_planes_k2", 1280, "... two sweeps or more, planes smaller than 64 x 64"},
    // Planes whose shorter side fills four fifths of 40, 48, 56 or 64 (pairs_2d_apply), forward in one launch with two
    // lanes a row, both leaving row masks.  N(0, 1), lambda 10^U(-1.3, 0), forward, two lanes a row / a plane per workgroup /
    // pass by pass, us:
    //   K = 2       560 planes    800           1000          1300           2048           4096
    //      33 x 33   55  48  58    55  67  63    55  74  66    70  92  78    102 136 102    166 252 156
    //      40 x 40   46  54  65    46  73  74    46  81  79    72 103  89     91 149 117    161 278 190
    //      44 x 48   68  56  66    68  83  73    68  91  82    86 110  98    130 162 126    215 298 214
    //      50 x 50   80  58  73    80  81  84    81  96  92   126 114 109    154 166 150    271 311 260
    //      56 x 56   64  63  74    65  82  87    72  98  99   105 118 115    132 174 158    232 322 290
    //      60 x 60   97  61  78    99  87  88   110 104 106   149 124 126    185 179 170    321 333 325
    //      64 x 64   76  62  83    77  86  96    79 103 104   118 125 122    149 183 172    260 339 311
    //   K = 10: 36 x 36, 800 planes 194 252 288, 4096: 629 995 722;  47 x 47 237 283 340, 777 1111 1038;
    //      52 x 56 278 295 364, 1300: 441 424 491, 4096: 1003 1163 1127;  63 x 63 330 306 430, 504 441 620, 1150 1229 1666;
    //      64 x 64 274 310 400, 428 444 515, 995 1227 1406.
    //   K = 1: 800 planes 40 x 40 27 43 35, 56 x 56 40 49 44, 64 x 64 46 54 50, 44 x 48 41 47 38, 60 x 60 60 52 46; 1300: 40 59 42,
    //      60 71 59, 67 74 64.
    {"plane_per_group64_full_planes_k2", 560, "... planes of 40 x 40, 48 x 48, 56 x 56 and 64 x 64, two sweeps; two lanes a row beyond"},
    {"plane_per_group64_full_planes_k3", 560, "... three or four sweeps"},
    {"plane_per_group64_full_planes_k5", 560, "... five sweeps or more"},
    {"pair_2d_planes", 704, "2D planes of 33-56 a side that fill four fifths of 40, 48 or 56: two lanes a row beyond this many planes (up to 1024 on sides beyond 48; beyond plane_per_group64_planes_k2 from two to ten sweeps on, by how much of its square a plane fills; one sweep: squares of 40, 48, 56 and 64, up to 1024)"},
    // Beyond plane_per_group64_planes_k2, no squares, forward and forward + reverse sweep, ratio to the better way of the kernels that left
    // pass outputs only (pass by pass beyond 1280 planes, as now with few sweeps):
    //                     two lanes a row                                    pass by pass
    //      K = 2:  1700 planes   3100        9000       1700        3100        9000
    //      36 x 40  1.01 0.95  1.05 1.04  1.05 1.02   1.00 0.97  0.99 1.02  0.98 1.01
    //      41 x 48  1.17 1.06  1.13 1.10  1.12 1.07   0.99 0.97  1.00 1.03  1.04 1.07
    //      47 x 47  0.98 0.86  0.98 0.89  0.92 0.68   0.92 0.87  0.95 0.91  0.95 0.75
    //      49 x 56  1.13 1.05  1.24 1.17  1.10 1.05   0.99 0.96  1.01 1.03  1.03 1.05
    //      60 x 60  1.18 1.02  1.20 1.06  1.09 1.03   1.01 0.98  1.01 0.98  1.01 0.99
    //      63 x 63  0.95 0.86  0.92 0.83  0.86 0.61   0.87 0.89  0.86 0.84  0.87 0.64
    //      K = 3:  36 x 40 0.96 0.92, 0.98 0.98, 0.99 0.98;  41 x 48 1.07 1.01, 1.04 1.03, 1.03 1.01;  33 x 33 0.92 0.80, 0.98 0.85, 1.07 0.83
    //              against 0.91 0.83, 0.91 0.85, 0.94 0.81;  53 x 55 0.91 0.84, 0.90 0.84, 0.85 0.59;  50 x 50 0.97 0.88, 1.02 0.95, 0.94 0.66
    //      K = 4:  41 x 48 0.98 0.95, 0.98 0.99, 1.00 0.99;  50 x 50 0.91 0.84, 0.99 0.90, 0.92 0.63;  49 x 56 1.00 0.96, 1.13 1.08, 1.02 1.00;
    //              60 x 60 1.02 0.92, 1.07 0.94, 0.98 0.92;  64 x 60 0.94 0.85, 1.00 0.90, 0.91 0.87;  60 x 64 1.08 0.91, 1.12 0.97, 1.03 0.95
    //      K = 6:  52 x 56 0.94 0.92, 1.04 1.02;  49 x 56 0.95 0.93, 1.10 1.06;  60 x 60 0.97 0.86, 1.01 0.89;  62 x 64 1.05 0.88, 1.09 0.94
    //      K = 10: 49 x 56 0.90 0.89, 1.05 1.03;  60 x 64 0.99 0.84, 1.05 0.89.
    // A plane per workgroup, 1700 and 2600 planes (K = 2: 57 x 58 1.00 0.90, 1.05 0.97;  60 x 60 1.09 0.96, 1.16 1.03;  63 x 63 0.87 0.80, 0.91 0.85):
    //      K = 3:  57 x 58 0.91 0.84, 0.96 0.88;  60 x 60 0.97 0.87, 1.09 0.94;  58 x 64 1.08 0.91, 1.16 0.94;
    //      K = 4:  57 x 58 0.86 0.81, 0.92 0.84;  60 x 60 0.95 0.87, 1.05 0.92;  58 x 64 1.03 0.89, 1.11 0.92.
    {"pair_2d_many_planes", 2560, "2D planes of 57-64 a side that fill four fifths of 64, no squares: a plane per workgroup up to this many planes (four fifths of it: three sweeps, and rows of 64 with four; plane_per_group64_planes_k2: two sweeps but for ragged rows), two lanes a row beyond (rows of 64 never, others from two to six sweeps on)"},
    // 2D reverse sweep of small batches with a plane per workgroup (tv_plane2d.hpp): both adjoint
    // state tensors of the plane in LDS, 16 x 2 or 8 x 8 threads x samples per row, the segment
    // sums across a row's threads by row shifts.  Against the row-per-lane one-launch kernel (a
    // chain of 32 or 64 samples per lane and pass, one or two waves per CU on such batches),
    // backward call with its lambda reduction, this kernel / that one:
    //   32 x 32, K = 4:  64 planes 14 / 19,  256: 14 / 20,  512: 18 / 22,  768: 23 / 24,  896: 27 / 25;
    //            K = 10: 256 planes 23 / 38;  K = 1: 15 / 15 at every count up to 768 (launches);
    //   28 x 30, K = 2: 512 planes 14 / 21, 1024: 21 / 26;
    // Planes of 33-64 samples a side against two lanes a row (tv2d_bwd_pair_kernel: four planes a CU at
    // once, half the threads of this mapping):
    //   64 x 64, K = 1: 256 planes 13 / 14,  512: 18 / 16,  640: 26 / 19, 2048:  61 /  42, 8192: 230 / 112;
    //            K = 4: 256 planes 33 / 36,  512: 39 / 41,  640: 64 / 44, 1024:  75 /  48, 2048: 163 / 115, 4096: 310 / 180;
    //   48 x 48, K = 2: 256 planes 15 / 17,  512: 21 / 19,  640: 29 / 20, 1024:  37 /  25, 8192: 252 / 132;
    //   40 x 40, K = 4: 256 planes 22 / 24,  512: 30 / 26,  640: 47 / 29, 1024:  56 /  31, 4096: 189 / 108;
    //   52 x 56, K = 4: 576 planes 53 / 42, 1024: 65 / 48, 2048: 121 / 112, 4096: 244 / 173;
    //   64 x 60, K = 4: 640 planes 55 / 55, 1024: 67 / 63, 1536: 100 / 111, 2048: 144 / 153, 3072: 203 / 192, 4096: 268 / 246;
    //   36 x 40, K = 1, against pass by pass from 1024 planes on: 1024: 24 / 18, 1536: 28 / 26, 2048: 33 / 37, 3072: 43 / 34;
    //   rows of no multiple of four samples: 33 x 33, 4096 planes 39 / 42, 47 x 47: 59 / 55, 63 x 63: 106 / 78; 6200: 49 / 56, 92 / 74, 158 / 115.
    // From row masks, K = 10, this mapping / two lanes a row:
    //      560 planes  800       1000      1300        2048        3000        4096
    //   36 x 36  75 / 60  94 / 63   94 / 63  135 / 118  176 / 159  247 / 170  327 / 261
    //   47 x 47  76 / 72  94 / 74   95 / 75  139 / 142  182 / 190  254 / 207  334 / 306
    //   52 x 56  77 / 82  96 / 86   98 / 86  140 / 161  188 / 210  258 / 240  341 / 356
    //   60 x 60  79 / 94  96 / 96   99 / 100 141 / 182  186 / 244  262 / 271  349 / 412
    //   64 x 64  80 / 83  98 / 87  100 / 89  142 / 162  194 / 239  267 / 240  356 / 378
    {"plane_per_group_bwd_planes", 768, "2D reverse sweep, planes of 17-32 a side: a plane per workgroup up to this many planes"},
    {"plane_per_group64_bwd_planes", 512, "2D reverse sweep, planes of 33-64 a side that two lanes a row can take over: a plane per workgroup up to this many planes (half as many again: pass outputs, sides beyond 56 that do not fill 64 x 64; row masks, sides beyond 48: see pairs_2d_bwd)"},
    // ... and against the pass-by-pass reverse sweep (2K launches), which is what other planes of
    // 33-64 samples a side get otherwise: 40 x 48, K = 1: 256 planes 14 / 20, 512: 18 / 22,
    // 1024: 29 / 28, 2048: 53 / 40; K = 3: 256 planes 22 / 44, 1024: 52 / 74, 2048: 95 / 108.
    // K = 4: 1024 planes 63 / 97, 4096: 219 / 245, 8192: 424 / 429; K = 2: 4096 planes 112 / 121,
    // 8192: 242 / 211; 56 x 60, K = 2: 2048 planes 80 / 114, 8192: 293 / 401; 33 x 33, K = 2: 4096
    // planes 103 / 111, 16 384: 418 / 381;  40 x 48, K = 3 again: 5120 planes 216 / 228, 8192: 336 / 323.
    {"plane_per_group64_bwd_ragged_planes", 768, "2D reverse sweep, other planes of 33-64 a side, one sweep: a plane per workgroup up to this many planes"},
    {"plane_per_group64_bwd_ragged_planes_k2", 6144, "... two sweeps or more"},
    // 2D, planes of at most 32 x 32 in one launch: the reverse sweep reads the segment codes of the
    // passes, not their outputs, so the forward kernel writes only the codes and x.  1 = it also
    // writes every pass's output into the workspace, where the pass-by-pass forward leaves them (the
    // tests set it to compare each pass with the oracle's).  Not writing them: 4096 planes of
    // 32 x 32, K = 1 / 4 / 10: 56 -> 52, 156 -> 149, 403 -> 385; 16 384 planes, K = 4: 560 -> 512.
    {"fused_keeps_passes", 0, "2D one-launch forward of planes of at most 32 x 32: 1 = also write every pass's output"},
    // 2D pass by pass, sides of 65-768 samples: chunk codes instead of pass outputs (tv_long.hpp) where the
    // 2K outputs and the two correction tensors take this many bytes or more, that is
    // where they push one another out of the 256 MB last-level cache.  Forming the codes costs a forward pass
    // four instructions a sample and thread, which a call without a reverse sweep does not always get back: it loses up
    // to 3 % on tensors that would stay in that cache by themselves, and wins where they would not.  Pass outputs /
    // codes, lambda 0.1 on images, forward, and forward + reverse sweep:
    //   24 x 512 x 512, K = 10, one lambda (528 MB): 696 / 710, 1197 / 1098;  three lambdas: 607 / 611, 1092 / 995
    //   48 x 512 x 512, K = 4 (480 MB): 553 / 537, 904 / 831;  three: 484 / 463, 814 / 744
    //   24 x 700 x 700, K = 3 (359 MB): 471 / 467, 794 / 725;  three: 434 / 428, 747 / 680
    //   100 x 256 x 256, K = 4 (250 MB): 295 / 298, 505 / 470;  three: 276 / 278, 474 / 439
    //   24 x 512 x 512, K = 4 (240 MB): 309 / 313, 513 / 473;  three: 268 / 270, 465 / 425
    //   512 x 100 x 100, K = 4 (196 MB): 275 / 279, 546 / 472;  three: 272 / 277, 513 / 446
    //   512 x 128 x 128, K = 2 (193 MB): 176 / 176, 340 / 316;  256 of them, K = 4 (160 MB): 205 / 210, 355 / 336
    //   12 x 512 x 512, K = 3 (96 MB), the codes formed in more instructions: 140 / 141, 233 / 221;  128 x 128 x 128, K = 4
    //   (80 MB): 140 / 147, 234 / 226
    // The line is drawn where the pair gains at least three times what the forward call alone can lose.
    {"chunk_codes_bytes", (int64_t)160 << 20, "2D, sides of 65-768 samples: the forward call leaves codes, not pass outputs, from this many bytes of passes on"},
    // Rows of at most 32 samples on the long-row kernels (small 1D batches, see
    // thread_per_sample_1d_rows): 16 threads x 2 samples up to this many rows, 8 x 4 beyond
    // (8192 rows of 32 samples as 256 planes, ten passes each way: 204 -> 180 with 16 x 2).
    {"thread_per_sample_wide_rows", 16384, "short rows on the long-row kernels: 16 threads per row up to this many rows"},
    // 1D calls on rows of 2-16 samples: up to half this many rows eight or sixteen threads per row on the
    // long-row kernels instead of a lane per row, whose few waves are bound by their dependency
    // chains.  Forward, threads per row / lane per row: 12 samples, 32 768 rows 11.8 / 13.5, 49 152: 14.0 /
    // 14.0, 65 536: 17.1 / 15.0;  7 samples, 40 960 rows 11.6 / 11.6, 57 344: 14.9 / 11.4.  Strided rows
    // (columns) of 16 or less, the threads' strided accesses being the worse ones, change over at half of
    // that again: 24 576 columns of 12 14.1 / 13.4, N(0, 1) 0.93 of it, 40 960: 17.6 / 12.9.
    // Rows of 17-32 samples: up to this many (columns of 32: half), and not beyond pair_1d_rows.
    {"thread_per_sample_1d_rows", 81920, "1D rows of at most 32 samples: a few threads per row up to this many rows (half of it: rows of at most 16, columns of 32; a quarter: columns of at most 16)"},
    // 1D calls on rows of 17-32 samples: beyond this many rows, times (m - 12) / 20 for rows of n samples with m the next
    // multiple of four, two lanes a row (tv_pair.hpp) instead of sixteen threads.  The sixteen threads take about
    // the same time for any n; the pairs' chains are half of m long, padding included.  Three quarters of that for strided
    // rows, whose sixteen threads' accesses are the worse ones; twice that for rows of 29-32 that lie apart, which the pairs read
    // sample by sample, a row a lane.  Forward, sixteen threads / two lanes, back to back; N(0, 1) with lambda 1, with 0.3,
    // walks with 2, and N(0, 1) with 64 lambdas of 10^U(-3, 1):
    //   17 samples, 15 300 rows  8.6 /  9.1,  7.2 /  7.2,  9.6 /  8.5,  8.2 /  8.1;  columns, 12 800  8.4 / 8.5, 7.2 / 7.6, 7.4 / 8.2, 8.0 / 8.0
    //   20 samples, 16 300 rows  9.0 /  9.1,  7.1 /  7.3, 10.0 /  9.0,  8.8 /  8.1;  columns, 12 200  8.5 / 9.4, 7.3 / 7.3, 7.5 / 7.7, 8.3 / 8.8
    //   21 samples, 18 400 rows  9.8 / 10.3,  7.8 /  8.7, 11.1 / 10.5, 10.0 / 10.2;  27 600 11.2 / 10.6, 9.0 / 8.9, 12.7 / 10.5, 10.9 / 10.1
    //   24 samples, 24 500 rows 10.8 / 10.8,  7.9 /  7.5, 11.5 / 10.9, 10.0 /  9.8;  columns, 18 400 10.7 / 10.6, 8.3 / 7.5, 9.3 / 9.5, 11.0 / 9.7
    //   25 samples, 26 600 rows 11.9 / 12.8,  9.0 /  9.8, 12.9 / 12.6, 11.0 / 11.7;  33 200 13.1 / 12.9, 9.8 / 9.9, 14.6 / 12.7, 12.1 / 11.8
    //   28 samples, 32 700 rows 11.9 / 12.3,  8.9 /  9.0, 13.4 / 13.5, 11.4 / 11.1;  columns, 24 500 13.0 / 11.9, 10.0 / 8.3, 10.9 / 11.0, 12.9 / 10.7
    //   31 samples, 38 900 rows 14.0 / 15.6, 10.5 / 10.4, 15.6 / 16.5, 13.6 / 13.7;  columns, 29 100 13.3 / 15.1, 10.3 / 10.6, 11.7 / 11.7, 14.0 / 13.5
    //   32 samples, 40 900 rows 14.2 / 15.8, 10.0 /  9.8, 15.1 / 15.0, 13.2 / 13.7;  columns, 30 700 13.9 / 15.1, 10.5 / 10.2, 11.6 / 12.6, 14.3 / 12.8
    //   with 3 samples between them: 29 samples, 52 200 rows 15.9 / 19.4, 11.6 / 16.4, 18.3 / 19.4, 15.5 / 16.9;
    //   32 samples, 40 900 rows 14.5 / 15.9, 10.9 / 12.3, 15.8 / 16.7, 13.6 / 13.5;  81 900: 22.1 / 20.3, 16.2 / 18.1, 25.4 / 21.5, 22.1 / 18.8
    // (Packed rows of 29-32 that start off a 16-byte boundary are read word by word and would do better with a line half as high
    // again, but which kernel runs does not depend on where a caller's buffers lie.)
    {"pair_1d_rows", 40960, "1D rows of 17-32 samples: two lanes a row beyond this many rows x (m - 12) / 20, m the length rounded up to a multiple of four (three quarters of it: strided rows; twice: rows of 29-32 that lie apart)"},
    // 1D calls on rows of 33-64 samples: beyond this many rows, times 1, 2, 3, 8 for rows of up to 40, 48, 56, 64
    // samples, two lanes a row instead of eight threads with
    // 8 or 12 samples each: an elimination takes half the instructions of sums over blocks that cross
    // threads, but a wave holds 32 rows and the longer halves chains of 32.  N(0, 1), lambda 0.3 / 1, forward,
    // eight threads / two lanes:
    //   40 samples, 16 384 rows  10 /  10,  14 /  17,   32 768:  14 /  11,  17 /  18,  524 288: 102 /  51, 148 /  74
    //   48 samples, 32 768 rows  13 /  13,  18 /  19,  131 072:  32 /  25,  46 /  37,  524 288: 105 /  69, 152 /  98
    //   56 samples, 32 768 rows  14 /  15,  19 /  23,  131 072:  32 /  28,  46 /  42,  524 288: 110 /  79, 158 / 113
    //   64 samples, 65 536 rows  20 /  21,  28 /  30,  131 072:  32 /  35,  46 /  50,  524 288: 117 /  99, 165 / 144
    //   60 samples, random walks, lambda 2, the ratio of the two: 98 304 rows 0.92, 131 072: 0.84, 196 608: 0.96, 262 144: 0.99,
    //   524 288: 1.06; its columns 98 304: 1.00, 131 072: 0.91, 196 608: 1.03
    // Unit-stride rows with 3 samples between them, the ratio at 131 072 rows for lambda 0.3 / 1 / walks: 33 samples
    // 0.91 / 1.07 / 1.17, 40: 1.15 / 1.38 / 1.51, 44: 0.84 / 0.95 / 0.99, 52: 0.75 / 0.81 / 0.87, 64: 0.59 / 0.68 / 0.69, and no better with
    // more rows: not beyond 40 samples.
    {"pair_1d_long_rows", 24576, "1D rows of 33-64 samples: two lanes a row beyond this many rows x 1, 2, 3, 8 (up to 40, 48, 56, 64 samples; beyond 40 not where rows lie apart)"},
    // 1D calls on unit-stride rows of 65-256 samples: 32 threads (up to 128 samples) or 64 per row, four samples
    // each, instead of 8-32 threads with 8 or 12.  Few waves are bound by their chains, which follow the samples
    // per thread; many by their instructions, of which the scans across more threads take more.  Forward, N(0, 1)
    // with lambda 1, 8 or 12 samples per thread / four:
    //    65 samples,   64 rows 13.3 /  7.5, 1024: 16.3 / 8.7, 8192: 17.3 / 12.4, 16 384: 20.2 / 18.8, 32 768: 26.1 / 29.3
    //   128 samples,   64 rows 10.0 /  7.6, 1024: 11.1 / 9.3, 8192: 13.8 / 12.6, 12 288: 17.3 / 16.1, 16 384: 18.0 / 19.3
    //   160 samples,   64 rows 14.5 /  7.7, 1024: 14.9 / 8.3, 4096: 15.8 / 12.2
    //   192 samples, 6144 rows 17.2 / 15.0, 8192: 18.4 / 18.4, 12 288: 21.0 / 23.7
    //   256 samples,   64 rows  9.6 /  7.0, 1024: 12.0 / 8.9, 4096: 14.9 / 12.1, 6144: 15.2 / 15.5, 12 288: 22.5 / 24.1
    // At the line, N(0, 1) with lambda 1 and 0.1, walks with 1 and 5, noisy steps with 0.2 and 10^U(-3, 1) a row: 128
    // samples, 9216 rows 1.04-1.12 times as fast, 192, 6144: 1.13-1.25, 256, 6144: 1.01-1.07; nowhere below slower.
    {"wave_per_row_rows", 6144, "1D calls on unit-stride rows of 65-256 samples: four samples a thread up to this many rows (half as many again: up to 128 samples)"},
    // 2D pass by pass with ONE lambda for all planes and three sweeps or more: sides up to this many
    // samples (768 at most, and beyond 64) are solved by tridiagonal elimination (tv_long_tri.hpp), not
    // by block means.  The slower one of the two is kept here for the sake of one number, the
    // gradient of that lambda: a signed sum over all planes that cancels to a few of its terms, and
    // which jumps of the size of the last bit take part is a matter of rounding in either solver.
    // 24 planes of 512 x 512, N(0, 1), lambda 0.1, K = 10, forward: 633 by elimination, 564 by block
    // means.  0: block means everywhere.
    {"one_lambda_tri_side", 768, "2D with one lambda and three sweeps or more: sides of 65 to this many samples (at most 768) by tridiagonal elimination"},
    // Multilevel start of unit-stride rows: from this length on.  8M samples in rows of n, lambda
    // 10^U(-3, 1) per row, cold / multilevel, for random walks, white noise and noisy steps of 64
    // samples: n = 520: 95 / 107, 82 / 103, 79 / 102; 768: 73 / 79, 70 / 78, 59 / 82; 769: 103 / 107,
    // 80 / 101, 83 / 101; 900: 87 / 83, 82 / 85, 72 / 84; 1024: 79 / 76, 80 / 79, 66 / 76; 1100: 150 / 108,
    // 135 / 118, 132 / 107; 1536: 135 / 90, 134 / 94, 116 / 88; 2048: 127 / 82, 125 / 88, 92 / 81; 4096:
    // 135 / 90, 115 / 95, 98 / 88.  So the start wins where a row spans waves, from 1025 samples on, by
    // 10-30 %.  The line at 769 was drawn with an earlier solver, whose cold start took longer: rows of
    // 769-1024 samples come out even on walks and lose up to a quarter on noisy steps, but the size of
    // the workspace hangs on this value, and callers that stored it.
    {"ml_min_length", 769, "multilevel start for unit-stride rows of this many samples or more"},
    // ... and levels are stacked (one at least) until a row has at most this many samples.  One
    // level, solved from the cold start, is what pays: every further level is two more launches,
    // and the cold start of a row of a few thousand samples is cheap next to the fine level.
    // Rows as above, coarsest level at most 256 / 1024 / 4096 samples: n = 2048: 104 / 83 / 82,
    // 111 / 88 / 88, 99 / 81 / 81; 8192 (32M samples): 320 / 308 / 284, 331 / 314 / 290, 307 / 294 / 271;
    // 16 384 (32M): 398 / 385 / 356, 395 / 380 / 352, 389 / 376 / 351.
    {"ml_coarsest", 4096, "coarsest level of the multilevel start"},
    // Backward along few columns of 33-256 samples: half the samples a thread and groups of 16 columns, for shorter chains and more
    // workgroups.  With dL/dlam, this / the mapping for more columns, us:
    //    40 samples, 4096 columns 7.1 / 8.3, 16 384:  8.5 /  9.3, 32 768: 11.9 / 11.2;  128: 7.2 / 8.1, 10.2 / 10.3, 15.3 / 15.5;
    //   160 samples, 4096 columns 8.7 / 9.0, 16 384: 12.4 / 11.5, 32 768: 21.8 / 18.5;  256: 8.2 / 9.5, 14.4 / 14.4, 23.1 / 22.2.
    {"bwd_few_columns", 16384, "backward along columns of 33-256 samples: twice the threads a column up to this many columns"},
};

inline int64_t get(int which) { return table[which].value; }

// The lowest value that chunk_codes_bytes has had: with fewer bytes than that no forward call has left codes, and
// the reverse sweep need not look.  (Looking is a load that everything waits for, and two ways behind a
// branch; it cost reverse sweeps that never find codes up to 1.4 us a pass: 12 x 100 x 100, K = 4, 49 -> 60 us,
// 128 x 128 x 128, K = 4, 83 -> 94.)
inline int64_t chunk_codes_lowest = table[kChunkCodesBytes].value;

// Whether a line that decides which planes of 33-64 a side leave row masks has ever been moved: until then a reverse sweep
// knows from the sizes whether its workspace can hold them.
inline bool mask_lines_moved = false;

inline void set(int which, int64_t value)
{
    if (which >= kPlanePerGroup64Planes && which <= kPair2dManyPlanes && value != table[which].value) mask_lines_moved = true;
    table[which].value = value;
    if (which == kChunkCodesBytes && value < chunk_codes_lowest) chunk_codes_lowest = value;
}

}  // namespace tvd
