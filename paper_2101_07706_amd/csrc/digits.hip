// The layer products on the integer matrix cores, for calls large enough (`digits_plan`).
//
// A number x of a row is taken as the integer round(x 2^39 / R), R a power of two above the row's largest magnitude, in five signed 8-bit digits,
// most significant first: x = R sum_i d_i 2^(-7 - 8 i).  A column of B likewise.  Nineteen of the products of a digit of A by a digit of B, those with
// i + j <= 5, go through v_mfma_i32_16x16x64_i8 into six 32-bit sums, one for each i + j: exact, whatever the order.  Conversions and FMAs
// put them together in double.
//
// The result is the double form's (product_tile), bit for bit, whatever the operands: beside each sum stands the most that it and the double form's sum can
// be apart, and where the floats at both ends of that differ the output is summed again in the double form's own order (product_at).  No average enters
// into it.  In units of 2^-46 R_A R_B an output may be off by
//  * the products that are left out: 2^-9 times the digits 2 .. 4 of the column, their magnitudes added up, for i + j = 6, and 2^-9 K for i + j > 6;
//  * 128 for a number that the digits round, which those of at least 2^-16 R are not (counted by row and by column);
//  * 2^-7 times the column's magnitudes, each as often as the double form rounds after it (v_mfma_f64_16x16x4 is four FMAs in ascending k, each rounded to
//    nearest), with R_A in the place of the row's, for what that form's sum is off, and 1/8 of that for the roundings here;
//  * 1 for what is cut off below.
// Together about 2^-38 R_A R_B for 256 k.  Of normal numbers by uniform weights one output in 6800 is summed again with 64 k, one in 3200 with 256, one in 1400 with
// 512; of features whose scales are log-normal (sigma 1.5) one in 750 with 256.  Rows and columns that hold an infinity, a NaN or nothing but numbers
// beyond 2^-90 .. 2^100, rows so small that results may be denormal and tiles with many such outputs are computed in double.  What is summed again is listed and
// worked off when a block is through or its list full; where it is so much that digits do not pay (known after the first step, if it is so from there on) the block goes on in double.
// (Fifteen products, those with i + j <= 4, and a bound for roundings that are independent of each other, 126 us where this takes 148: off by 2^-19 where values
// repeat along k.)
//
// Why: the instruction does 4.7 POP/s here, 60 times what v_mfma_f64_16x16x4_f64 does, so nineteen products are a third of the time; what counts
// beside them is the vector ALU, at eleven instructions to cut a number and twenty to put an output together.
//  * A block holds the digits of B for its columns in registers (all K, 16 NT columns a wavefront) and walks down the rows of A.  Every number
//    of A is cut once per block, by the wavefront that loaded it (whole rows side by side, so that loads are whole lines and a row's maximum is
//    known at once), and its digits go to LDS, from where all wavefronts read them.  The last digits of B, which two products in nineteen take, wait in
//    LDS too: with them in registers two wavefronts per SIMD do not fit.
//  * Two buffers of rows, one barrier per step.  Half of the wavefronts (one on every SIMD) cut the next step's rows before they multiply, half
//    afterwards, so that the one's vector instructions run beside the other's matrix instructions.
//  * The order of the k within a chunk of 64 is free as long as A and B agree; k = 16 s + 4 g + j for byte 4 s + j of lane group g lets a lane write
//    the digits of the four consecutive k it loaded as one word, and 16 bytes of room after 16 rows spread those words over the banks.
//  * All of a tile's outputs are put together before the first is stored: each is a chain of ten instructions (131072 x 256 x 256 with a row's two outputs
//    at a time 191 against 184).  Registers are full: one value more and the loop waits for a reload behind the loads of A (211 against 191).
// Measured in double / now, us: 131072 rows 256 -> 256 252 / 148, 128 -> 256 135 / 86, 64 -> 256 79 / 60, 65 536 rows 512 -> 128 126 / 90.
// Operands that leave the digits little, in double / now, us: scales of features by exp(1.5 g) 131072 x 256 x 256 255 / 183, 2449029 x 100 x 256 2160 / 1915, 65536 x 512 x 128
// 124 / 120; one feature 300 times the others that no weight looks at (one output in 57) 250 / 287, 2160 / 2286, 124 / 167; infinities everywhere 252 / 281, 2156 / 2274, 124 / 163
// (normal numbers 255 / 148, 2160 / 1475, 126 / 90).  (A list of 512 outputs, and everything of a block that lists more again: 650, 6490, 305, and 6020 for the normal numbers
// of 2449029 rows; a list that is worked off by itself, 16 outputs of a tile of 16 x 16 before all of it is summed again: 501, 4440, 366.)
// A step of 32 rows by 256 columns takes 8 us, of which the matrix instructions 4.4; the rest is the
// wavefronts' own chain (read, multiply, put together, cut, write).
// Tried: digits of B in LDS and every wavefront for itself (64 columns each: A is cut, and read in pieces of 16 bytes, once per 64 columns)
// 165 .. 195 us for 131072 x 256 x 256 with fifteen products, where this form took 126; 16 wavefronts of 16 columns 167 (A's digits are read from LDS twice as often); the
// outputs that are summed again summed at once 236 (the block waits for them at its next barrier).
#include "common.hpp"
#include "gemm_rules.hpp"
#include "product_tile.hpp"
#include "digits.hpp"

namespace csgs {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));

constexpr int DIGITS = 5, SUMS = 6, CHUNK = DIGIT_CHUNK, WPB = DIGIT_WAVES;
constexpr int E_MIN = -90, E_MAX = 100, E_ZERO = -1000, E_BAD = 1000;   // exponents that are used, and what stands for a row of zeros or one that is not

// floor(x + 1/2), one instruction
__device__ inline int round_half_up(float x)
{
    int r;
    asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// The digits of 4 Q numbers, |x scale| < 0.993 2^31: of quad q the digits p in the bytes of d[p][q].  Four digits are the bytes of the rounded integer
// once 0x80 is added to the lower three and taken away again from each byte by itself; the fifth is what the rounding left, in 256ths.
template <int Q, typename D, typename SCALE>   // scale: of quad q
__device__ inline void cut(const float (&x)[4 * Q], SCALE scale, D (&d)[DIGITS])
{
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        uint32_t w[4], low = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float y = x[4 * q + j] * scale(q);
            const int h = round_half_up(y);
            const float r = __builtin_fmaf(y - (float)h, 256.f, 128.f);
            low = __builtin_amdgcn_cvt_pk_u8_f32(r, j, low);
            w[j] = (uint32_t)h + 0x00808080u;
        }
        const uint32_t a = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u), b = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
        const uint32_t c = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u), e = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
        d[0][q] = (int)__builtin_amdgcn_perm(e, c, 0x07060302u);
        d[1][q] = (int)(__builtin_amdgcn_perm(e, c, 0x05040100u) ^ 0x80808080u);
        d[2][q] = (int)(__builtin_amdgcn_perm(b, a, 0x07060302u) ^ 0x80808080u);
        d[3][q] = (int)(__builtin_amdgcn_perm(b, a, 0x05040100u) ^ 0x80808080u);
        d[4][q] = (int)(low ^ 0x80808080u);
    }
}

// The largest magnitude of floats as bits; a NaN counts as the largest of all (a floating-point maximum would drop it)
struct Largest {
    int pos = 0;
    uint32_t neg = 0;
    __device__ void take(float x, float y)
    {
        const int a = __float_as_int(x), b = __float_as_int(y), m = a > b ? a : b;
        const uint32_t n = (uint32_t)a > (uint32_t)b ? (uint32_t)a : (uint32_t)b;
        pos = pos > m ? pos : m;
        neg = neg > n ? neg : n;
    }
    __device__ uint32_t bits() const
    {
        const uint32_t n = neg & 0x7FFFFFFFu;
        return (uint32_t)pos > n ? (uint32_t)pos : n;
    }
};

// e with R = 2^e: every magnitude below 0.993 R, so that the first digit holds what is carried into it
__device__ inline int exponent_of(uint32_t bits) { return bits ? (int)((bits + 0x20000u) >> 23) - 126 : 0; }
__device__ inline bool unusable(uint32_t bits) { return bits && (bits >= 0x7F800000u || exponent_of(bits) < E_MIN || exponent_of(bits) > E_MAX); }
__device__ inline float scale_of(int e) { return __int_as_float((127 + 31 - e) << 23); }
// least magnitude of three (a NaN counts for nothing)
__device__ inline float least_of(float x, float y, float z)
{
    float r;
    asm("v_min3_f32 %0, |%1|, |%2|, |%3|" : "=v"(r) : "v"(x), "v"(y), "v"(z));
    return r;
}
// the least magnitude whose last bit the digits hold
__device__ inline float least_whole(int e) { return __int_as_float((127 - 16 + e) << 23); }

// Of a row of A: its exponent, and what its outputs may be off by for its numbers that the digits only round
struct Row {
    int e;
    float off;
};

// The maximum over L lanes side by side, to all of them; for a whole wavefront as values that it shares
template <int L, int R>
__device__ inline void max_over(uint32_t (&v)[R])
{
    uint32_t o[R];
#define CSGS_MAX_STEP(CTRL, MASK)                                        \
    do {                                                                 \
        _Pragma("unroll") for (int i = 0; i < R; ++i) o[i] = dpp_move<CTRL, MASK>(v[i]); \
        _Pragma("unroll") for (int i = 0; i < R; ++i) v[i] = v[i] > o[i] ? v[i] : o[i];  \
    } while (0)
    CSGS_MAX_STEP(0x128, 0xF);   // row_ror:8
    CSGS_MAX_STEP(0x124, 0xF);
    CSGS_MAX_STEP(0x122, 0xF);
    CSGS_MAX_STEP(0x121, 0xF);
    if constexpr (L == 64) {
        CSGS_MAX_STEP(0x142, 0xA);   // row_bcast:15
        CSGS_MAX_STEP(0x143, 0xC);   // row_bcast:31
#pragma unroll
        for (int i = 0; i < R; ++i) v[i] = (uint32_t)__builtin_amdgcn_readlane((int)v[i], 63);
    } else if constexpr (L == 32) {
#pragma unroll
        for (int i = 0; i < R; ++i) o[i] = (uint32_t)__shfl_xor((int)v[i], 16);
#pragma unroll
        for (int i = 0; i < R; ++i) v[i] = v[i] > o[i] ? v[i] : o[i];
    }
#undef CSGS_MAX_STEP
}

// KC chunks of 64 k (the last of them may be short, or for 8 be missing), NT tiles of 16 columns a wavefront, wcs wavefronts side by side over
// the columns of a block (the wcs - th part of the others takes other rows), cgs blocks over the columns, rgs over the rows.
template <int MODE, int KC, int NT>
__global__ __launch_bounds__(64 * WPB, 1) void gemm_digits_k(
    const float *__restrict__ A, int64_t lda, const float *__restrict__ Bm, int64_t ldb, float *__restrict__ C, int64_t ldc, int M_bound, int N,
    int K, const int32_t *__restrict__ rows_dev, int64_t few, int cgs, int wcs, int rgs, int n_inst, CompStride cs)
{
    constexpr int LPR = KC == 1 ? 16 : (KC == 2 ? 32 : 64);        // lanes of a row
    constexpr int QUADS = 4;                                       // quads (four consecutive k of a row) of a step that a lane cuts
    constexpr int QPR = KC > 4 ? 2 : 1;                            // quads of a row that a lane holds
    constexpr int RW = 64 / LPR * QUADS / QPR, RS = RW * WPB;      // rows of a step that a wavefront cuts, rows of a step
    constexpr int TILES = RS / 16;
    static_assert(RS == digit_rows(KC), "rows of a step");
    constexpr int GS = 272, CS = 4 * GS, PS = KC * CS, TSZ = DIGITS * PS;   // bytes: 16 rows of a lane group, chunk, plane of digits, tile of 16 rows
    __shared__ __align__(16) char digits[2][TILES * TSZ];
    __shared__ __align__(16) char last_digits[WPB * KC * NT * 1024];   // of B, which only one product takes
    __shared__ Row row_of_a[2][RS];
    // Outputs and tiles that are summed again: a step lists no more than STEP_LIST of them, and the list is worked off when it has no room for as many
    constexpr int TILE_LIST = digit_tile_list(KC), STEP_LIST = digit_step_list(KC), LIST = digit_list(KC);
    static_assert(STEP_LIST == TILES * WPB * TILE_LIST * NT, "a tile of every wavefront");
    __shared__ uint32_t again_list[LIST];
    __shared__ uint32_t again;     // entries, and in the upper half the outputs that they stand for
    __shared__ int again_full[2];   // by the step's buffer
    __shared__ int step_end[64];    // of each instance, behind its last step
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, grp = lane >> 4;
    // blocks over the same rows lie on one XCD and share what they read
    const int bid = (int)blockIdx.x, q = bid >> 3;
    const int cg = q % cgs, rg = (q / cgs) * 8 + (bid & 7);
    if (rg >= rgs) return;
    const int wrs = WPB / wcs, wc = wave % wcs, wr = wave / wcs;   // this wavefront's columns and its share of the row tiles
    const int n0 = (cg * wcs + wc) * 16 * NT;
    const bool multiplies = wr < wrs && n0 < N;
    const int kq = K - 4;
    int total;   // steps there are
    auto rows_of = [&](int inst) { return rows_dev ? (const int32_t *)((const char *)rows_dev + inst * cs.adj) : nullptr; };

    // ---- rows of A: quad i of this lane
    auto row_at = [&](int l, int i) { return wave * RW + (QPR == 2 ? i >> 1 : l / LPR + i * (64 / LPR)); };
    auto quad_at = [&](int l, int i) { return l % LPR + (QPR == 2 ? 64 * (i & 1) : 0); };
    auto place = [&](int step, int &inst, int &m0) {   // one instance after the other
        inst = 0;
        m0 = step * RS;
        if (n_inst == 1) return;
        const int end = step_end[here_v(lane)];
        inst = __popcll(__ballot(end <= step));
        m0 = (step - (inst ? __builtin_amdgcn_readlane(end, inst - 1) : 0)) * RS;
    };
    auto load_a = [&](int step, float (&x)[4 * QUADS]) {
        int inst, m0;
        const int l = here_v(lane);
        auto row_of = [&](int i) { return row_at(l, i); };
        auto quad_of = [&](int i) { return quad_at(l, i); };
        place(step < total ? step : total - 1, inst, m0);
        const char *pa = (const char *)(A + (int64_t)m0 * lda) + inst * cs.x;
#pragma unroll
        for (int i = 0; i < QUADS; ++i) {
            const int row = m0 + row_of(i) < M_bound ? row_of(i) : M_bound - 1 - m0, k = 4 * quad_of(i);
            const uint32_t o = (uint32_t)row * (uint32_t)(lda * 4) + 4u * (uint32_t)(k < kq ? k : kq);
            const f32x4u v = *reinterpret_cast<const f32x4u *>(pa + o);
            x[4 * i] = v[0]; x[4 * i + 1] = v[1]; x[4 * i + 2] = v[2]; x[4 * i + 3] = v[3];
        }
    };
    // the rows' exponents and digits into buffer `buf`
    auto put_a = [&](int buf, float (&x)[4 * QUADS]) {
        const int l = here_v(lane);
        auto row_of = [&](int i) { return row_at(l, i); };
        auto quad_of = [&](int i) { return quad_at(l, i); };
        if (K & 3) {   // the piece that holds the last k was read further to the left
#pragma unroll
            for (int i = 0; i < QUADS; ++i) {
                const int sh = 4 * quad_of(i) - kq;
                const float v0 = x[4 * i], v1 = x[4 * i + 1], v2 = x[4 * i + 2], v3 = x[4 * i + 3];
                x[4 * i] = sh == 1 ? v1 : sh == 2 ? v2 : sh == 3 ? v3 : v0;
                x[4 * i + 1] = sh == 1 ? v2 : sh == 2 ? v3 : v1;
                x[4 * i + 2] = sh == 1 ? v3 : v2;
            }
        }
        float sc[QUADS];
        {
            constexpr int ROWS = QUADS / QPR;
            uint32_t b[ROWS];
            float least[ROWS];
#pragma unroll
            for (int i = 0; i < ROWS; ++i) {
                Largest m;
#pragma unroll
                for (int j = 0; j < 4 * QPR; j += 2) m.take(x[4 * QPR * i + j], x[4 * QPR * i + j + 1]);
                b[i] = m.bits();
            }
            max_over<LPR>(b);
#pragma unroll
            for (int i = 0; i < ROWS; ++i) {
                const int e = exponent_of(b[i]);
                least[i] = least_whole(e);
#pragma unroll
                for (int j = 0; j < QPR; ++j) sc[QPR * i + j] = scale_of(e);
            }
            // numbers that the digits only round, few as they are
            bool some = false;
            int rounded[ROWS];
#pragma unroll
            for (int i = 0; i < ROWS; ++i) {
                rounded[i] = 0;
                float m = least_of(x[4 * QPR * i], x[4 * QPR * i + 1], least_of(x[4 * QPR * i + 2], x[4 * QPR * i + 3], INFINITY));
                if (QPR == 2) m = least_of(x[8 * i + 4], x[8 * i + 5], least_of(x[8 * i + 6], x[8 * i + 7], m));
                some |= m < least[i];
            }
            if (__any(some)) {   // (zeros count for nothing: twice the bits less one is largest for them)
                some = false;
#pragma unroll
                for (int i = 0; i < ROWS; ++i) {
                    uint32_t m = ~0u;
#pragma unroll
                    for (int j = 0; j < 4 * QPR; ++j) {
                        const uint32_t v = (uint32_t)__float_as_int(x[4 * QPR * i + j]) * 2u - 1u;
                        m = m < v ? m : v;
                    }
                    some |= m < (uint32_t)__float_as_int(least[i]) * 2u - 1u;
                }
            }
            if (__any(some)) {
#pragma unroll
                for (int i = 0; i < ROWS; ++i)
#pragma unroll
                    for (int j = 0; j < 4 * QPR; ++j) {
                        const float v = x[4 * QPR * i + j];
                        uint64_t w = __ballot(v != 0.f && fabsf(v) < least[i] && 4 * quad_of(QPR * i + j / 4) < K);
                        if (LPR < 64) w = w >> (l & (64 - LPR)) & ((1ull << (LPR & 63)) - 1);
                        rounded[i] += __popcll(w);
                    }
            }
#pragma unroll
            for (int i = 0; i < ROWS; ++i)
                row_of_a[buf][row_of(QPR * i)] = Row{b[i] == 0 ? E_ZERO : unusable(b[i]) ? E_BAD : exponent_of(b[i]), 132.f * (float)rounded[i]};
        }
        int d[DIGITS][QUADS];
        cut<QUADS>(x, [&](int q) { return sc[q]; }, d);
#pragma unroll
        for (int i = 0; i < QUADS; ++i) {
            const int row = row_of(i), kk = quad_of(i);
            char *to = digits[buf] + (row >> 4) * TSZ + (kk >> 4) * CS + (kk & 3) * GS + (row & 15) * 16 + ((kk >> 2) & 3) * 4;
            if (KC == 1 || KC == 2 || KC == 4 || KC == 8 || (kk >> 4) < KC) {
#pragma unroll
                for (int p = 0; p < DIGITS; ++p) *reinterpret_cast<int *>(to + p * PS) = d[p][i];
            }
        }
    };
    // ---- few rows on the device of the many there is room for: in double, the tiles dealt to all wavefronts
    const int my_rows = lane < n_inst ? resolve_count(M_bound, rows_of(lane)) : 0;   // of instance `lane`
    if (rows_dev) {
        int64_t rows = my_rows;
#pragma unroll
        for (int o = 32; o; o >>= 1) rows += __shfl_xor(rows, o);
        if ((int64_t)__builtin_amdgcn_readfirstlane((int)(rows > few)) == 0) {
            const int tn = (N + 31) / 32, waves = cgs * rgs * WPB;
#pragma unroll 1
            for (int inst = 0; inst < n_inst; ++inst) {
                const int tiles = (resolve_count(M_bound, rows_of(inst)) + 15) / 16 * tn;
#pragma unroll 1
                for (int t = ((rg * cgs + cg) * WPB + wave + inst * 97) % waves; t < tiles; t += waves)
                    product_tile<MODE, 1, 2, TAIL_32, uint32_t>((const float *)((const char *)A + inst * cs.x), here(lda), here(Bm), here(ldb),
                                                                (float *)((char *)C + inst * cs.out), here(ldc), nullptr, here(M_bound), here(N),
                                                                here(K), rows_of(inst), t / tn * 16, t % tn * 32);
            }
            return;
        }
    }
    // The steps that hold a row; no other is read.  (us, every step there is room for / these: 131072 x 256 x 256 with 16 384 rows 69 / 40, 65 536 rows 108 / 88, 131072 x 100 x 256
    // with 32 768 rows 47 / 37; eight instances of up to 16 384 rows, 2000 in each 66 / 38 (in double 46), 0 .. 16 384 x 100 x 256 88 / 53 (70).)
    {
        const int incl = wave_inclusive_scan<int32_t>((my_rows + RS - 1) / RS);
        total = __builtin_amdgcn_readlane(incl, 63);
        step_end[lane] = incl;   // (every wavefront writes the same and reads what it wrote)
    }
    if (rg >= total) return;
    float x0[4 * QUADS];
    int step = rg;
    load_a(step, x0);

    uint32_t code = 0;   // names the step in the list
#pragma unroll 1
    for (;;) {   // once, and again after every time that the list is worked off (which leaves no room in the registers for what follows)
        // ---- this wavefront's columns of B: digits of k = 64 c + 16 s + 4 grp + j, columns n0 + NT l16 + t
        i32x4 w[KC][NT][DIGITS - 1];
        char *const last_w = last_digits + (wave * KC * NT) * 1024 + lane * 16;
        bool any_bad;
        int col_e[NT], row_lim;   // exponent of a column's unit, 2^-46 R_A R_B
        float col_off;            // what an output may be off by in that unit, beside its row's share
        {
            // (a lane's offsets lie below 2^32, and what lies beyond the last k reads the last k)
            const float *const b0 = here(Bm);
            const uint32_t ldb4 = (uint32_t)here(ldb) * 4;
            const int l = here_v(lane), l16 = l & 15, grp = l >> 4, ks = here(K);
            auto other = [&](int v, int o) { return __builtin_amdgcn_ds_bpermute((l ^ o) * 4, v); };
            uint32_t ob[NT], ob_max[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const uint32_t n = (uint32_t)(n0 + NT * l16 + t < N ? n0 + NT * l16 + t : N - 1);
                ob[t] = MODE == MODE_DZ ? n * ldb4 + 16u * (uint32_t)grp : n * 4 + (uint32_t)(4 * grp) * ldb4;
                ob_max[t] = MODE == MODE_DZ ? n * ldb4 + 4u * (uint32_t)kq : n * 4 + (uint32_t)(K - 1) * ldb4;
            }
            const uint32_t n2 = (uint32_t)(n0 + NT * l16 < N - 2 ? n0 + NT * l16 : N - 2), ob2 = n2 * 4 + (uint32_t)(4 * grp) * ldb4,
                           ob2_max = n2 * 4 + (uint32_t)(K - 1) * ldb4;
            auto load_b = [&](int c, int t, float (&y)[16]) {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const uint32_t k = (uint32_t)(c * CHUNK + 16 * s);
                    if constexpr (MODE == MODE_DZ) {
                        const uint32_t o = ob[t] + 4 * k;
                        const f32x4u v = *reinterpret_cast<const f32x4u *>((const char *)b0 + (o < ob_max[t] ? o : ob_max[t]));
#pragma unroll
                        for (int j = 0; j < 4; ++j) y[4 * s + j] = v[j];
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const uint32_t o = ob[t] + (k + (uint32_t)j) * ldb4;
                            y[4 * s + j] = *reinterpret_cast<const float *>((const char *)b0 + (o < ob_max[t] ? o : ob_max[t]));
                        }
                    }
                }
            };
            // zeros beyond the last k
            auto end_b = [&](int c, float (&y)[16]) {
                if (c * CHUNK + CHUNK <= K) return;
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const int kb = c * CHUNK + 16 * s + 4 * grp;
                    if constexpr (MODE == MODE_DZ) {
                        const int sh = kb - kq;
                        const float v0 = y[4 * s], v1 = y[4 * s + 1], v2 = y[4 * s + 2], v3 = y[4 * s + 3];
                        y[4 * s] = sh <= 0 ? v0 : sh == 1 ? v1 : sh == 2 ? v2 : sh == 3 ? v3 : 0.f;
                        y[4 * s + 1] = sh <= 0 ? v1 : sh == 1 ? v2 : sh == 2 ? v3 : 0.f;
                        y[4 * s + 2] = sh <= 0 ? v2 : sh == 1 ? v3 : 0.f;
                        y[4 * s + 3] = sh <= 0 ? v3 : 0.f;
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j) y[4 * s + j] = kb + j < K ? y[4 * s + j] : 0.f;
                    }
                }
            };
            float y[KC][NT][16];
#pragma unroll
            for (int c = 0; c < KC; ++c) {
                if constexpr (MODE != MODE_DZ && NT == 2) {   // both columns at once
                    typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));
#pragma unroll
                    for (int s = 0; s < 4; ++s)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const uint32_t o = ob2 + (uint32_t)(c * CHUNK + 16 * s + j) * ldb4;
                            const f32x2u v = *reinterpret_cast<const f32x2u *>((const char *)b0 + (o < ob2_max ? o : ob2_max));
                            y[c][0][4 * s + j] = v[0];
                            y[c][NT - 1][4 * s + j] = v[1];
                        }
                } else {
#pragma unroll
                    for (int t = 0; t < NT; ++t) load_b(c, t, y[c][t]);
                }
            }
            if (MODE != MODE_DZ && NT == 2 && n0 + 32 > N) {   // (read further to the left)
                const bool left = n0 + 2 * l16 >= N - 1;
#pragma unroll
                for (int c = 0; c < KC; ++c)
#pragma unroll
                    for (int j = 0; j < 16; ++j) y[c][0][j] = left ? y[c][NT - 1][j] : y[c][0][j];
            }
            Largest m[NT];
            float later[NT], least[NT];   // sum of the magnitudes, each times the additions that follow on it in the double form; least magnitude
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                later[t] = 0.f;
                least[t] = INFINITY;
            }
#pragma unroll
            for (int c = 0; c < KC; ++c)
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    end_b(c, y[c][t]);
#pragma unroll
                    for (int h = 0; h < 16; h += 8) {   // 32 k, which that form takes together; those of a last piece come first
                        const int k0 = c * CHUNK + 4 * h;
                        float part = 0.f;
#pragma unroll
                        for (int j = h; j < h + 8; j += 2) {
                            m[t].take(y[c][t][j], y[c][t][j + 1]);
                            part += fabsf(y[c][t][j]) + fabsf(y[c][t][j + 1]);
                            least[t] = least_of(y[c][t][j], y[c][t][j + 1], least[t]);
                        }
                        later[t] = __builtin_fmaf(part, (float)(k0 + 32 <= ks ? (ks & ~31) - k0 : ks), later[t]);
                    }
                }
            float sc[NT];
            bool un = false, some = false;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                uint32_t b = m[t].bits(), o = (uint32_t)other((int)b, 16);
                b = b > o ? b : o;
                o = (uint32_t)other((int)b, 32);
                b = b > o ? b : o;
                const int e = exponent_of(b);
                sc[t] = scale_of(e);
                col_e[t] = b == 0 ? E_ZERO : e - 46;
                un |= unusable(b);
                some |= least[t] < least_whole(e);
                least[t] = least_whole(e);
            }
            // bad: a column that the digits do not hold; lim: rows below this may give denormal floats, which round elsewhere
            any_bad = __any(un);
            int el = 0;
#pragma unroll
            for (int t = 0; t < NT; ++t) el = col_e[t] != E_ZERO && col_e[t] < el ? col_e[t] : el;
#pragma unroll
            for (int o = 1; o < 16; o *= 2) {
                const int x = other(el, o);
                el = x < el ? x : el;
            }
            row_lim = __builtin_amdgcn_readfirstlane(-149 - el);
            col_off = 0.f;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                uint32_t dropped = 0;
                int rounded = 0;   // numbers that the digits only round
                if (__any(some)) {
#pragma unroll
                    for (int c = 0; c < KC; ++c)
#pragma unroll
                        for (int j = 0; j < 16; ++j) rounded += y[c][t][j] != 0.f && fabsf(y[c][t][j]) < least[t];
                }
#pragma unroll
                for (int c = 0; c < KC; ++c) {
                    i32x4 d[DIGITS];
                    cut<4>(y[c][t], [&](int) { return sc[t]; }, d);
#pragma unroll
                    for (int p = 2; p < DIGITS; ++p)
#pragma unroll
                        for (int s = 0; s < 4; ++s) dropped = __builtin_amdgcn_sad_u8((uint32_t)d[p][s] ^ 0x80808080u, 0x80808080u, dropped);
#pragma unroll
                    for (int p = 0; p < DIGITS - 1; ++p) {
                        asm volatile("" : "+v"(d[p]));   // (now: left for later, what they are put together from would not fit the registers)
                        w[c][t][p] = d[p];
                    }
                    *reinterpret_cast<i32x4 *>(last_w + (c * NT + t) * 1024) = d[DIGITS - 1];
                    __builtin_amdgcn_sched_barrier(0);
                }
                const float r = __int_as_float((127 - (col_e[t] + 46)) << 23);   // 1 / R
                float off = (float)dropped * 0x1p-9f + later[t] * (0x1.001p-7f + 0x1p-10f) * r + 132.f * (float)rounded;
                off += __int_as_float(other(__float_as_int(off), 16));
                off += __int_as_float(other(__float_as_int(off), 32));
                off = col_e[t] == E_ZERO ? 0.f : off;
                col_off = off > col_off ? off : col_off;
            }
            col_off = (col_off + 1.f + (float)ks * 0x1.1p-9f) * 1.0001f;
        }
        if (wave == 0 && lane == 0) {
            const int none = here_v(0);   // (a constant would be kept, and spilled, outside the loop)
            again = (uint32_t)none;
            again_full[0] = again_full[1] = none;
        }
        put_a(0, x0);
        load_a(step + rgs, x0);
        __syncthreads();

        int buf = 0, steps = 0;
        bool full = false;
#pragma unroll 1
        for (; step < total && !full; step += rgs, buf ^= 1, code += 1u << 15, ++steps) {
            int inst, s0;
            place(step, inst, s0);
            const int32_t *rd = rows_of(inst);
            const int M = resolve_count(M_bound, rd);
            char *pc = (char *)(C + (int64_t)s0 * ldc + n0) + inst * cs.out;
            if (wave >= WPB / 2 && step + rgs < total) {
                put_a(buf ^ 1, x0);
                load_a(step + 2 * rgs, x0);
            }
            if (multiplies) {
#pragma unroll 1
                for (int ti = wr; ti < TILES; ti += wrs) {
                    const int m0 = s0 + 16 * ti;
                    const char *ap = digits[buf] + ti * TSZ + grp * GS + l16 * 16;
                    const int re0 = row_of_a[buf][16 * ti + l16].e;
                    if (m0 >= M) break;
                    // what is listed here is done again in double when the list is full or all steps are through
                    auto list = [&](int n, int outputs) {
                        uint32_t at = 0;
                        if (lane == 0) {
                            at = atomicAdd(&again, (uint32_t)outputs << 16 | (uint32_t)n);
                            const int most = (steps + 1) * (STEP_LIST / 2);
                            if ((int)(at >> 16) + outputs > (most < LIST - STEP_LIST ? most : LIST - STEP_LIST)) again_full[buf] = 1;
                        }
                        return __builtin_amdgcn_readfirstlane((int)at) & 0xFFFF;
                    };
                    auto list_tile = [&]() {
                        const int at = list(1, TILE_LIST * NT);
                        if (lane == 0) again_list[at] = 0x80000000u | code | (uint32_t)((16 * ti) << 8 | wc * 16 * NT);
                    };
                    if (any_bad || __any((re0 == E_BAD || (re0 < row_lim && re0 != E_ZERO)) && m0 + l16 < M)) {
                        list_tile();
                    } else {
                        i32x4 acc[NT][SUMS], a[3], wl[NT];
#pragma unroll
                        for (int t = 0; t < NT; ++t)
#pragma unroll
                            for (int s = 0; s < SUMS; ++s) acc[t][s] = i32x4{0, 0, 0, 0};
                        // A's planes in an order in which two of them take longer than a read from LDS
                        constexpr int order[DIGITS] = {3, 1, 4, 0, 2};
                        auto read_a = [&](int i) { return *reinterpret_cast<const i32x4 *>(ap + (i / DIGITS) * CS + order[i % DIGITS] * PS); };
                        a[0] = read_a(0);
                        a[1] = read_a(1);
#pragma unroll
                        for (int i = 0; i < KC * DIGITS; ++i) {
                            const int c = i / DIGITS, s = order[i % DIGITS];
                            if (i % DIGITS == 0)
#pragma unroll
                                for (int t = 0; t < NT; ++t) wl[t] = *reinterpret_cast<const i32x4 *>(last_w + (c * NT + t) * 1024);
                            if (i + 2 < KC * DIGITS) a[(i + 2) % 3] = read_a(i + 2);
#pragma unroll
                            for (int p = 0; p < DIGITS && s + p < SUMS; ++p)
#pragma unroll
                                for (int t = 0; t < NT; ++t)
                                    acc[t][s + p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i % 3], p < DIGITS - 1 ? w[c][t][p < DIGITS - 1 ? p : 0] : wl[t], acc[t][s + p], 0, 0, 0);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        uint32_t at = ((uint32_t)(16 * ti + 4 * grp) * (uint32_t)ldc + (uint32_t)(NT * l16)) * 4;
                        const int left = N - n0 - NT * l16;
                        uint64_t low[4][NT], any = 0;
                        float v[4][NT];   // (all of them before the first is stored: each is a chain of ten instructions)
                        Row r[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) r[i] = row_of_a[buf][16 * ti + 4 * grp + i];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const double off = (double)(r[i].off + col_off);
#pragma unroll
                            for (int t = 0; t < NT; ++t) {
                                // (within 32 bits for K up to 512: the first digit's magnitude is at most 127; of the last sum only what a unit holds)
                                double d = (double)(int)(((uint32_t)acc[t][0][i] << 8) + (uint32_t)acc[t][1][i]);
                                d = __builtin_fma(d, 256.0, (double)acc[t][2][i]);
                                d = __builtin_fma(d, 256.0, (double)acc[t][3][i]);
                                d = __builtin_fma(d, 256.0, (double)(acc[t][4][i] + (acc[t][5][i] >> 8)));
                                const float most = (float)(d + off);
                                low[i][t] = __ballot(__float_as_int(most) != __float_as_int((float)(d - off)));
                                v[i][t] = __builtin_ldexpf(most, r[i].e + col_e[t]);
                                any |= low[i][t];
                            }
                        }
                        float *p = reinterpret_cast<float *>(pc + at);
                        if (m0 + 16 <= M && n0 + 16 * NT <= N) {
#pragma unroll
                            for (int i = 0; i < 4; ++i, p += ldc) store_floats<NT>(p, v[i]);
                        } else {
#pragma unroll
                            for (int i = 0; i < 4; ++i, p += ldc)
                                if (m0 + 4 * grp + i < M) {
                                    if (left >= NT) store_floats<NT>(p, v[i]);
                                    else if (NT == 2 && left == 1) *p = v[i][0];
                                }
                        }
                        if (any) {
                            int count = 0;
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const int ro = 16 * ti + 4 * grp + i;
                                const bool row_ok = s0 + ro < M && r[i].e != E_ZERO;
#pragma unroll
                                for (int t = 0; t < NT; ++t) {
                                    low[i][t] &= __ballot(row_ok && t < left && col_e[t] != E_ZERO);
                                    count += __popcll(low[i][t]);
                                }
                            }
                            if (count > TILE_LIST * NT) {
                                list_tile();
                            } else if (count > 0) {
                                int at0 = list(count, count);
#pragma unroll
                                for (int i = 0; i < 4; ++i)
#pragma unroll
                                    for (int t = 0; t < NT; ++t) {
                                        const int pos = at0 + __popcll(low[i][t] & (((uint64_t)1 << lane) - 1));
                                        if ((low[i][t] >> lane) & 1)
                                            again_list[pos] = code | (uint32_t)((16 * ti + 4 * grp + i) << 8 | (wc * 16 * NT + NT * l16 + t));
                                        at0 += __popcll(low[i][t]);
                                    }
                            }
                        }
                    }
                }
            }
            if (wave < WPB / 2 && step + rgs < total) {
                put_a(buf ^ 1, x0);
                load_a(step + 2 * rgs, x0);
            }
            __syncthreads();
            full = __builtin_amdgcn_readfirstlane(again_full[buf]) != 0;   // (the next step's go to the other word: the same for all wavefronts)
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // some of the outputs are written again
        __syncthreads();
        const int count = __builtin_amdgcn_readfirstlane((int)again) & 0xFFFF, outputs = __builtin_amdgcn_readfirstlane((int)(again >> 16));
        if (outputs > steps * (STEP_LIST / 2) && step < total) {
            step -= steps * rgs;
            break;
        }
        // tiles, and outputs by themselves, up to sixteen at a time; the wavefronts take them in turn
        const int l = here_v(lane), l16 = l & 15, grp = l >> 4;
#pragma unroll 1
        for (int s = wave; s < count; s += 16 * WPB) {
            const int there = (count - s + WPB - 1) / WPB, some = there < 16 ? there : 16;
            const uint32_t what = again_list[s + WPB * (l16 < some ? l16 : some - 1)];
            const int st = (int)(what >> 15 & 0xFFFF) * rgs + rg;
            int in = 0, before = 0;   // instance, and the steps before its first
            if (n_inst > 1)
#pragma unroll 1
                for (int e = step_end[0]; e <= st; e = step_end[in]) {
                    before = e;
                    ++in;
                }
            const int64_t m = (st - before) * RS + (int)((what >> 8) & 127);
            const int n = cg * wcs * 16 * NT + (int)(what & 255);
            if (__any(!(what >> 31))) {
                const float sum = product_at<MODE, 4>((const float *)((const char *)A + in * cs.x) + m * lda, Bm, MODE == MODE_DZ ? (uint32_t)n * (uint32_t)(ldb * 4) : (uint32_t)n * 4, ldb, K, l);
                if (grp == (l16 & 3) && l16 < some && !(what >> 31)) ((float *)((char *)C + in * cs.out))[m * ldc + n] = sum;
            }
            uint64_t tiles = __ballot(l < some && what >> 31);
#pragma unroll 1
            for (int g = 0; tiles; tiles &= g == NT - 1 ? tiles - 1 : ~0ull, g = g == NT - 1 ? 0 : g + 1) {
                const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)what, __ffsll((unsigned long long)tiles) - 1);
                const int nt = cg * wcs * 16 * NT + (int)(w & 255) + 16 * g;
                if (nt >= N) continue;
                int ig, mg;
                place((int)(w >> 15 & 0xFFFF) * rgs + rg, ig, mg);
                const int32_t *rd = rows_of(ig);
                product_tile<MODE, 1, 1, TAIL_32, uint32_t>((const float *)((const char *)A + ig * cs.x), here(lda), here(Bm), here(ldb),
                                                            (float *)((char *)C + ig * cs.out), here(ldc), nullptr, here(M_bound), here(N),
                                                            here(K), rd, mg + (int)((w >> 8) & 127), nt, l);
            }
        }
        if (step >= total) return;
        __syncthreads();   // (the list is read)
        load_a(step, x0);
    }

    // ---- So many outputs are summed again that digits do not pay (half of what a step may list takes as long as digits save): the steps since the list was last
    // worked off and those that are left, in double, all their tiles dealt to the wavefronts
    constexpr int RT = RS >= 32 ? 2 : 1;
    const int n_first = cg * wcs * 16 * NT, n_end = n_first + wcs * 16 * NT < N ? n_first + wcs * 16 * NT : N;
    const int tn = (n_end - n_first + 63) / 64, each_step = RS / 16 / RT * tn, all = (total - step + rgs - 1) / rgs * each_step;
#pragma unroll 1
    for (int t = wave; t < all; t += WPB) {
        int inst, s0;
        place(step + t / each_step * rgs, inst, s0);
        const int32_t *rd = rows_of(inst);
        const int m0 = s0 + t % each_step / tn * 16 * RT;
        if (m0 >= resolve_count(M_bound, rd)) continue;   // (a tile that starts past the last row would read before the matrix)
        auto tile = [&](auto tail) {
            product_tile<MODE, RT, 4, decltype(tail)::value, uint32_t>((const float *)((const char *)A + inst * cs.x), here(lda), here(Bm), here(ldb),
                                                                       (float *)((char *)C + inst * cs.out), here(ldc), nullptr, here(M_bound),
                                                                       here(n_end), here(K), rd, m0, n_first + t % tn * 64, lane);
        };
        if (K % 32 == 0) tile(std::integral_constant<int, TAIL_NONE>());
        else if (K % 32 <= 8) tile(std::integral_constant<int, TAIL_8>());
        else tile(std::integral_constant<int, TAIL_32>());
    }
}

template <int MODE>
void launch_digits(const DigitsPlan &d, const float *A, int64_t lda, const float *B, int64_t ldb, float *C, int64_t ldc, int M, int N, int K,
                   const int32_t *M_dev, hipStream_t st, const CompInst &ci)
{
    const dim3 grid((unsigned)((d.rgs + 7) / 8 * 8 * d.cgs));
#define CSGS_DIGITS_AS(KID, KC, NT)                                                                                                              \
    CSGS_LAUNCH(KID, (gemm_digits_k<MODE, KC, NT>), grid, dim3(64 * WPB), st, A, lda, B, ldb, C, ldc, M, N, K, M_dev, d.few, d.cgs, d.wcs, d.rgs, \
                ci.n, ci.cs)
#define CSGS_DIGITS(KC, NT)                                         \
    do {                                                            \
        if (MODE == MODE_FWD) CSGS_DIGITS_AS(K_GEMM_DIGITS, KC, NT); \
        else CSGS_DIGITS_AS(K_GEMM_DZ_DIGITS, KC, NT);              \
    } while (0)
    if (d.kc == 1) CSGS_DIGITS(1, 2);
    else if (d.kc == 2) CSGS_DIGITS(2, 2);
    else if (d.kc == 3) CSGS_DIGITS(3, 2);
    else if (d.kc == 4) CSGS_DIGITS(4, 2);
    else if (d.kc == 5) CSGS_DIGITS(5, 1);
    else CSGS_DIGITS(8, 1);
#undef CSGS_DIGITS
#undef CSGS_DIGITS_AS
}
template void launch_digits<MODE_FWD>(const DigitsPlan &, const float *, int64_t, const float *, int64_t, float *, int64_t, int, int, int,
                                      const int32_t *, hipStream_t, const CompInst &);
template void launch_digits<MODE_DZ>(const DigitsPlan &, const float *, int64_t, const float *, int64_t, float *, int64_t, int, int, int,
                                     const int32_t *, hipStream_t, const CompInst &);

}  // namespace csgs
