// Which tiles a layer product takes, and into how many parts the weight gradient is cut.  Host code without anything of the device, so that the
// tests can ask it where there is none.
#pragma once
#include <algorithm>
#include <cstdint>

namespace csgs {

// What one MFMA of a tile shape costs beside one of the largest shape (conversions per MFMA, tiles per
// wavefront slot), measured on 4096 .. 131072 rows
struct Shape {
    int rt, nt;
    double cost;
};
static constexpr Shape kShapes[] = {{2, 4, 1.0}, {2, 3, 1.01}, {2, 2, 1.05}, {1, 4, 1.06}, {1, 3, 1.1}, {1, 2, 1.17}, {2, 1, 1.22}, {1, 1, 1.33}};
constexpr int CUS = 256;   // compute units; a block has a wavefront for each SIMD

// The shape whose slowest compute unit is done first: blocks per unit, rounded up, times what a block takes.  The larger shapes waste fewer
// conversions, the smaller ones waste fewer columns and leave fewer units idle (4500 x 512 x 100, us: 2x4 33.1, 2x2 19.7, 2x1 14.5, 1x1
// 12.9; 8192 x 256 x 256: 19.8, 20.4, 22.8, 23.1).  Of the two shapes of two instructions a step 1x2 is the quicker where a lane's columns of B
// come in one load (1x2 against 2x1 at 20000 x 481 x 100 46 and 49, 2048 x 602 x 256 14.8 and 17, 4500 x 300 x 512 31 and 33.5), 2x1 for
// dZ, whose B is read along k (5367 x 48 x 460 19.9 and 19.0).
// M is the row bound.  Of a count on the device that lies far below it nothing is known here, and the tiles are then larger than they had best be: 1024
// rows in 8 instances, 100 x 256, 11.9 us with all rows, 10.8 with half of them (blocks of 64 x 64 that staged in LDS 13.2 and 8.9); 8192 rows of
// which 409 are there, 256 x 256, 19.3 (16.2).  Shapes for half the rows would cost the calls that have them all 5 %.
inline Shape pick_shape(int64_t M, int64_t N, int64_t n_inst, bool b_kmajor)
{
    Shape best = kShapes[7];
    double least = 1e300;
    for (const Shape &s : kShapes) {
        if (s.nt > N) continue;   // a lane's NT columns exist
        const int64_t tiles = ((M + 16 * s.rt - 1) / (16 * s.rt)) * ((N + 16 * s.nt - 1) / (16 * s.nt));
        const int64_t per_cu = ((tiles + 3) / 4 * n_inst + CUS - 1) / CUS;
        const double cost = b_kmajor && s.rt == 1 && s.nt == 2 ? 1.25 : s.cost;
        const double c = (double)per_cu * s.rt * s.nt * cost;
        if (c < least) { least = c; best = s; }
    }
    return best;
}

// A row of a matrix this long could put a lane's offset beyond 32 bits
inline bool far_apart(int64_t lda, int64_t ldb) { return lda >= (1 << 24) || ldb >= (1 << 24); }

// ---- the products on the integer matrix cores (digits.hip)
constexpr int DIGIT_CHUNK = 64, DIGIT_WAVES = 8;
constexpr int digit_rows(int kc) { return kc == 1 ? 128 : kc == 2 ? 64 : kc <= 4 ? 32 : 16; }   // of a step

// Tiles of 16 rows that hold one of the `left` rows from a step's first one to the last there is
constexpr int row_tiles(int64_t left, int rows_of_step) { return left <= 0 ? 0 : (int)(((left < rows_of_step ? left : rows_of_step) + 15) / 16); }

// What a block sums again in double.  A wavefront lists the outputs of a tile by themselves up to so many per 16 columns; of more, the tile: an output on its own reads
// a line of B for every k, and that many take as long as the tile.
constexpr int digit_tile_list(int kc) { return kc > 4 ? 8 : 4; }
// Most that a step lists, a tile taken as the outputs that would have stood in its place; and the room: the list is worked off when a step might find too little.  That
// costs the digits of B once more, 10 to 20 us, so there is room for 1024 (131072 x 256 x 256, one output in 750: once in 90 steps).
constexpr int digit_step_list(int kc) { return digit_rows(kc) / 16 * DIGIT_WAVES * digit_tile_list(kc) * (kc > 4 ? 1 : 2); }
constexpr int digit_list(int kc) { return kc == 1 ? 2048 : 1024; }

struct DigitsPlan {
    bool use;
    int kc;              // chunks of k that the kernel is made for
    int cgs, wcs, rgs;   // blocks over the columns, wavefronts of a block side by side over its columns, blocks over the rows
    int64_t few;         // no more rows than these on the device: in double
};

// Microseconds of a product [M x K] [K x N] in double: what the fullest compute unit multiplies and stores, and a launch (131072 rows, us, expected:
// 64 x 256 79, 79; 100 x 256 112, 112; 256 x 256 252, 257; 256 x 47 52, 52; 8192 rows 256 x 256 19.5, 18.9; 4096 rows 512 x 512 34, 34)
inline double double_us(int64_t M, int64_t N, int64_t K, int64_t n_inst, bool b_kmajor)
{
    const Shape s = pick_shape(M, N, n_inst, b_kmajor);
    const int64_t tiles = ((M + 16 * s.rt - 1) / (16 * s.rt)) * ((N + 16 * s.nt - 1) / (16 * s.nt));
    const int64_t per_cu = ((tiles + 3) / 4 * n_inst + CUS - 1) / CUS;
    return 3.0 + (double)per_cu * s.rt * s.nt * ((double)((K + 3) / 4) * 0.029 * s.cost + 0.13);
}

// The digits' form where it is the quicker by 5 %.  Its time is what `begin` says (digits of B to cut, outputs to sum again) and for each step of
// the block with the most of them what `step` says.  Measured against that, us, double / digits (expected): 131072 rows, 256 x 256
// 252 / 148 (149), 256 x 128 128 / 97 (95), 128 x 256 135 / 86 (91), 64 x 256 79 / 60 (62); 65536 rows 512 x 128 126 / 90 (90), 192 x 256 99 / 69 (70);
// 16384 rows 256 x 256 36 / 36 (37), 128 x 256 21 / 22 (23).  Columns for one or two wavefronts: never (131072 rows, 256 x 64 66 / 78, 524288 rows, 64 x 64 79 / 85).
inline DigitsPlan digits_plan(int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, int64_t ldc, int64_t n_inst, bool b_kmajor)
{
    DigitsPlan d{false, 0, 0, 0, 0, 0};
    constexpr int64_t FAR = 1 << 20;   // (a lane's offsets have 32 bits)
    if (K < 16 || K > 512 || N < 16 || N > 4096 || lda >= FAR || ldb >= FAR || ldc >= FAR || (N > K ? N : K) * ldb >= (1 << 29)) return d;
    const int chunks = (int)((K + DIGIT_CHUNK - 1) / DIGIT_CHUNK);
    d.kc = chunks > 5 ? 8 : chunks;
    const int nt = d.kc > 4 ? 1 : 2, tiles = (int)((N + 16 * nt - 1) / (16 * nt));
    d.cgs = (tiles + DIGIT_WAVES - 1) / DIGIT_WAVES;
    d.wcs = (tiles + d.cgs - 1) / d.cgs;
    const int64_t rs = digit_rows(d.kc), steps = (M + rs - 1) / rs * n_inst;
    int64_t rgs = d.cgs <= CUS / 8 ? CUS / 8 / d.cgs * 8 : 8;   // a block per compute unit, those over the same rows on one XCD
    if (rgs > steps) rgs = steps;
    d.rgs = (int)rgs;
    const int64_t turns = (steps + rgs - 1) / rgs;
    if (turns >= 65536) return d;   // (the list of a block's outputs counts its steps in 16 bits)
    if (d.wcs <= 2) return d;
    // us before the first step, and of a step, with columns for up to four and for eight wavefronts
    static constexpr double begin[9][2] = {{}, {11, 9.5}, {14.5, 13}, {15.5, 16}, {19.5, 21}, {12.5, 13.5}, {}, {}, {18.5, 22.5}};
    static constexpr double step[9][2] = {{}, {7.5, 13.2}, {5.4, 9.8}, {4.3, 6.7}, {4.7, 8.0}, {2.9, 3.6}, {}, {}, {3.5, 4.2}};
    const double one = step[d.kc][d.wcs > 4], start = begin[d.kc][d.wcs > 4];
    d.use = start + one * (double)turns < 0.95 * double_us(M, N, K, n_inst, b_kmajor);
    // the rows on the device that are done in double before the digits are cut: three quarters of what takes as long (smaller tiles there)
    const double rate = (double_us(M, N, K, n_inst, b_kmajor) - 3.0) / (double)(M * n_inst), mine = one / (double)(rs * rgs);
    d.few = rate > mine ? (int64_t)(0.75 * (start - 3.0) / (rate - mine)) : 0;
    return d;
}

// Parts of the reduction dimension for dW = Z^T G with `rows` rows that the caller's scratch has room for
inline int dw_max_parts(int rows, int64_t K, int64_t N)
{
    const int64_t tiles = ((K + 127) / 128) * ((N + 31) / 32);
    int64_t want = (512 + tiles - 1) / tiles;
    const int64_t chunks = ((int64_t)rows + 31) / 32;
    if (want > chunks) want = chunks;
    if (want < 1) want = 1;
    int64_t ks = ((rows + want - 1) / want + 31) / 32 * 32;
    if (ks < 32) ks = 32;
    const int64_t parts = (rows + ks - 1) / ks;
    return (int)(parts < 1 ? 1 : parts);
}

// Shape and parts for dW, a block per tile and part: the fewest microseconds by
//  * 29 ns per MFMA for the blocks of the fullest compute unit (28 tiles in 9 parts are 36 blocks for the 32 units of seven XCDs and twice the
//    time of 8 parts), times what the shape costs beside it;
//  * or 0.5 us per chunk of a wavefront where its unit holds too few blocks to multiply meanwhile (the chunk's loads take that long: one
//    block of 1x1 tiles per unit, 8192 rows, 256 x 256, 43 us);
//  * or what the XCDs fetch at 5.6 TB/s: each holds consecutive tiles and reads their columns of Z and G once (65536 rows, 100 x 256, 1x4 in 8
//    parts: seven XCDs read all of G, 97 us; 2x2 in 16 72);
//  * 3.5 us for the kernel that adds several parts and what these take through memory (16 bytes per output and part at about 4 TB/s).
// Measured against that, us: 8192 rows, 256 x 256: 2x2 in 4 / 8 parts 24.4 / 23.9 (24 / 25 expected), 1x2 in 4 24.8 (25), 2x3 in 16 28.6 (28),
// 256 x 47: 1x2 in 8 10.6 (11.2); 4096 rows, 512 x 512: one part of 2x2 37.6 (36), four of 2x4 41 (41), 512 x 100: 1x2 in 2 14.9 (15.6).
inline void dw_split(int rows, int64_t K, int64_t N, Shape *shape, int *parts)
{
    static const Shape shapes[] = {{2, 2, 1.1}, {2, 4, 1.03}, {2, 3, 1.06}, {1, 4, 1.1}, {1, 2, 1.17}, {2, 1, 1.3}, {1, 1, 1.5}};
    constexpr double MFMA_US = 0.029, CHUNK_US = 0.5, FETCH_BYTES_PER_US = 5.6e6, REDUCE_US = 3.5;
    constexpr int64_t RESIDENT = 3;   // blocks that a compute unit holds at once (fitted for all shapes: it is 2 of the largest, whose sums fill 64 KB of LDS, and 4 of the smallest)
    const int64_t chunks = ((int64_t)rows + 31) / 32;
    const int max_parts = dw_max_parts(rows, K, N);
    double least = 1e300;
    *shape = shapes[6];
    *parts = 1;
    for (const Shape &s : shapes) {
        if (s.nt > N || s.rt > K) continue;
        const int64_t tn = (N + 16 * s.nt - 1) / (16 * s.nt), tiles = ((K + 16 * s.rt - 1) / (16 * s.rt)) * tn;
        const int64_t xcd_tiles = (tiles + 7) / 8;   // every part deals its tiles to the XCDs anew
        const int64_t cols_z = (xcd_tiles + tn - 1) / tn * 16 * s.rt, cols_g = (xcd_tiles < tn ? xcd_tiles : tn) * 16 * s.nt;
        const int64_t cols = (tiles + xcd_tiles - 1) / xcd_tiles * ((cols_z < K ? cols_z : K) + (cols_g < N ? cols_g : N));
        const double fetch = (double)cols * rows * 4 / FETCH_BYTES_PER_US;
        for (const int64_t fill : {(int64_t)0, (int64_t)CUS, (int64_t)2 * CUS, (int64_t)4 * CUS}) {
            int64_t p = fill / 8 / xcd_tiles;
            p = p < 1 ? 1 : (p > max_parts ? max_parts : p);
            const int64_t per_cu = (xcd_tiles * p + CUS / 8 - 1) / (CUS / 8), mine = (chunks + 4 * p - 1) / (4 * p);
            const double multiply = (double)(per_cu * mine) * (8 * MFMA_US) * s.rt * s.nt * s.cost;
            const double load = (double)((per_cu + RESIDENT - 1) / RESIDENT * mine) * CHUNK_US;
            const double c = std::max(std::max(multiply, load), fetch) + (p > 1 ? REDUCE_US + (double)(p * K * N) * (16 / 4e6) : 0.0);
            if (c < least) { least = c; *shape = s; *parts = (int)p; }
        }
    }
}

}  // namespace csgs
