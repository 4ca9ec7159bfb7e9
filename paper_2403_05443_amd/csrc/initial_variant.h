#pragma once
// The collide-stream variant a context starts with (all variants give the same
// bits; lb_autotune measures them).  No HIP: a rule on sizes alone.

namespace lbd {

// mb: populations of one buffer in 10^6 bytes; bytes: of one population;
// rows_k: nx / 64 where the row-wave kernel applies (one box, D3Q19, nx = 64, 128
// or 256), else 0; walls: some box has walls.
//
// The times are the kernel's own in real steps, us a launch, a shape's variants
// taken in turns; 0 plain order, 1 row-wave, 3 XCD-chunked, 11 and 12 in place (plain,
// XCD-chunked), 15 XCD-grouped with non-temporal stores.
//  - Two buffers fit the 256 MB last-level cache: 3, each XCD's L2 serves the
//    cache lines its neighbouring tiles share.  96^3 FP32 (67 MB) 21.3 against 22.5 (0)
//    and 21.9 (12); 118^3 FP32 (125 MB) 36.8, 39.8, 37.8; 110^3 FP16 17.6, 20.0,
//    17.8; 24 boxes in FP16 (104 MB) 32.4, 37.8, 33.0.
//  - One buffer fits, or most of it: 12.  128^3 FP32 (159 MB) 46 against 58 (0), 60 (3),
//    66 (1) and 46 (11); 128^3 D3Q27 FP32 (226 MB) 65 against 92 (0); 16 boxes FP32
//    (158 MB) 48, 58 (0); 162^3 FP32 (323 MB) 113, 134 (0), 132 (15); 32 boxes FP32
//    (307 MB) 110, 112 (0).  Past 330 MB what still hits depends on the shape, and the
//    chunked order loses up to a fifth where it does not: 168^3 FP32 (360 MB) 166
//    against 140 (0, 15), 36 boxes FP32 (341 MB) 131, 124 (0), 117 (15), 116^3 D3Q27 FP64
//    (337 MB) 137, 130 (0), 28 boxes D3Q27 (382 MB) 156, 141; though 150^3 D3Q27 FP32
//    (364 MB) takes 139 against 143.  The half formats: 172^3 (193 MB) 53.5 against 77.7 (0)
//    and 75.7 (15), 186^3 (245 MB) 66 against 95 and 94, 192^3 (269 MB) 98 against 99 and
//    96: their line is below the measured one, which lies near 250 MB.
//  - Larger: 15.  256^3 FP16 221 against 231 (0, 11) and 239 (1), FP32 463, 474, 502 (1),
//    FP64 921, 954, 1001; 256 boxes in FP16 411, 423 (0); 164^3 FP32 (335 MB) 122, 129;
//    174^3 FP32 (400 MB) 148, 153.  D3Q27 has no such kernel and takes the plain order: 256^3
//    FP32 686 against 704 (3, 11).  Rows of 64 sites in FP32 far beyond the cache
//    suit the row-wave kernel: 64 x 480 x 512 459 against 481 (15), with walls 445 against 478;
//    64 x 400 x 400 level; FP64 64 x 512 x 512 926 (15), 946 (1).
//  - Walls in the half formats cost the generic kernels arithmetic that the
//    row-wave one decides once a row: 256^3 277 against 334 (15), 128 x 256 x 256 168, 184;
//    256 x 64 x 64 (40 MB) 18.9 against 20.5 (3), but 256 x 32 x 64 (20 MB) 13.8 against
//    12.9, and rows of 64 sites (64 x 512 x 512) 383 against 333 (15).  The in-place kernel
//    beats it where it applies: 256 x 128 x 128 (159 MB) 73 against 83.
//    The in-place kernels pay more for walls than pull, so they win later: 152^3 (133 MB)
//    63 (12) against 55 (3), D3Q27 136^3 (136 MB) 86, 76; 154^3 (139 MB) 65, 75.
inline int initial_variant(int lattice, int bytes, double mb, int rows_k, bool walls) {
    const bool half = bytes == 2, walled_half = half && walls;
    const bool rows = walled_half ? rows_k >= 2 && mb > 25 : bytes == 4 && rows_k == 1 && mb > 800;
    if (mb <= (walled_half ? 136 : 128)) return rows ? 1 : 3;
    if (mb <= (half ? 200 : 330)) return 12;
    if (rows) return 1;
    return lattice == 27 ? 0 : 15;
}

}  // namespace lbd
