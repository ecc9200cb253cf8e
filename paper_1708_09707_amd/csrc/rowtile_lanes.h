// Rules by sizes alone for the row tiles' pieces and passes (host code, no HIP
// types).
#pragma once
#include <cstdint>

namespace hmx {

// Passes of 128 rows (64 lanes of 16-byte units of R rows in FP64, 32 in FP32,
// 16 in BF16), narrower when the largest tile (need units a column) is shorter
inline int rowtile_lanes_tall(int need, int R) {
    int L = 16;
    while (L < need && L * R < 128 && L < 64) L *= 2;
    return L;
}

// Lanes per row group: ntiles tiles of at most need 16-byte units a column, of
// entries of es bytes.
//
// A column that is whole cache lines splits into passes for nothing, so passes
// are 512 bytes wide (256 in BF16) and half of that where it makes no more than
// 4096 workgroups (in BF16 below 512 rows), and 128 bytes for the fewest tiles.
// Columns of other lengths share a line between two passes and leave part of
// the last one idle: there one pass takes the whole column, and narrower ones
// only where they bring idle compute units in (BF16: up to 1024 workgroups, at
// most 32 lanes).  One pass takes FP64 columns of 33 to 63 units as well, where
// that fills the chip.
// Row-tile times in us by lanes 8/16/32/64 (the tall passes above: FP64 64
// lanes past 64 rows, else 32; FP32 32; BF16 16):
//   whole lines  FP64 N = 4096, 64 rows (64 tiles)       17 /  22 /  33 /  42
//                     N = 2^14 3-d, 64 rows (256)        168 / 182 / 189 / 220
//                     the same on a Gaussian mixture     204 / 191 / 205 / 234
//                     N = 2^14, 128 rows (128)           126 / 120 / 124 / 185
//                     N = 2^17, 256 rows (512)          1861 /1601 /1664 /1973
//                     N = 2^19, 256 rows (2048)         7854 /6774 /6223 /6833
//                     48540 3-d, 95 rows (512)          1893 /1581 /1667 /1433 (product)
//                FP32 N = 2^16, 256 rows (256)           451 / 432 / 552 / 591
//                     N = 2^20, 256 rows (4096)         9058 /7792 /7454 /7942
//                BF16 N = 2^20, 64 rows (16384)         5888 /6299 /9553
//                     N = 2^19, 256 rows (2048)         1637 /1723 /1946 /2265
//                     N = 2^20, 256 rows (4096)         3871 /3578 /3868 /4316
//                     N = 2^15 2-d, 512 rows (64)        160 / 176 / 260 / 445
//                     N = 2^15 3-d, 512 rows (64)        333 / 289 / 414 / 707
//   other        FP64 200003, 98 rows (2048)            2158 /1781 /1654 /1441
//                     300007, 147 rows (2048)           4278 /3289 /2979 /3552
//                     10000, 157 rows (64)                97 /  84 / 103 / 159
//                FP32 150000, 147 rows (1024)           1138 / 979 /1054 / 867
//                     6230 3-d, 49 rows (128)             38 /  36 /  47 /  84
//                BF16 150000 2-d, 147 rows (1024)        609 / 620 / 510 / 737
//                     37547, 147 rows (256)              141 / 138 / 175 / 273
//                     102315, 400 rows (256)             723 / 707 / 698 / 891
//                     9000, 71 rows (128)                 45 /  56 /  97
// Over 1358 handles (2-d and 3-d, 27 to 1000 rows, 8 to 16384 tiles) the pick
// takes 1.02 times the best of the four in the geometric mean and 0.80 of the
// tall passes; the worst against those is 256 tiles of 96 FP32 rows, 106 us
// against 94, then 128 tiles of 256 FP32 rows in 3-d, 513 against 474.
inline int rowtile_lanes(int64_t ntiles, int need, int es) {
    const bool bf16 = es == 2, f64 = es == 8;
    const int full = bf16 ? 16 : 32;
    auto works = [&](int L) { return ntiles * ((need + L - 1) / L); };
    int L = 8;
    while (L < need && L < 64) L *= 2;
    if (f64 && need > 32 && need < 64 && works(64) >= 512) return 64;
    if ((int64_t)need * 16 % 128 == 0) {
        if (L > full) L = full;
        if (L == full && works(L) <= 4096 && !(bf16 && need >= 64)) L /= 2;
        if (L == 16 && works(L) <= 128) L = 8;
        return L;
    }
    if (need > 64 || (bf16 && L > 32)) L = 32;
    while (L > 16 && works(L) < (bf16 ? 1024 : 256)) L /= 2;
    if (L == 16 && works(L) < (bf16 ? 129 : 128)) L = 8;
    return L;
}

// Whether a wave fills a piece of a matrix pool (else a workgroup of four): units
// 16-byte units over `pieces` pieces of that kind.  Small pieces are bound by the
// latency of piece, block and offset in turn, so by the pieces in flight; in large
// ones a wave takes the units one after another.  us as a workgroup / a wave:
//   near field  N = 200003 3-d BF16, 49 x 49 (343 units a piece)  3115 / 1240
//               100003 3-d FP32, 49 x 49 (637)                    1180 /  607
//               200000 2-d FP64, 49 x 49 (1225)                   1448 /  976
//               200000 2-d FP32, 98 x 98 (2450)                    628 /  463
//               60000 3-d FP32, 117 x 117 (3510)                   581 /  659
//               60000 3-d BF16, 235 x 235 (7050)                   490 /  531
//               200000 2-d FP64, 196 x 196 (19200)                2831 / 3736
//               4096 2-d FP64, 64 x 64 (2048, 1500 pieces)          20 /   28
//   factors     200003 3-d BF16, 49 rows (below 512)              2397 / 1620
//               200000 2-d FP64, 49 rows (below 512)              1405 / 1107
//               200000 2-d FP64, 196 rows (1024 to 2048)           795 /  943
inline bool piece_by_wave(bool near, int64_t units, int64_t pieces) {
    return pieces >= (near ? 8192 : 1) && units / pieces <= (near ? 3072 : 512);
}

}  // namespace hmx
