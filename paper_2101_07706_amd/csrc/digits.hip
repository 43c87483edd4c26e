// The layer products on the integer matrix cores, for calls large enough (`digits_plan`).
//
// A number x of a row is taken as the integer round(x 2^39 / R), R a power of two above the row's largest magnitude, in five signed 8-bit digits,
// most significant first: x = R sum_i d_i 2^(-7 - 8 i).  A column of B likewise.  Fifteen of the products of a digit of A by a digit of B, those with
// i + j <= 4, go through v_mfma_i32_16x16x64_i8 into five 32-bit sums, one for each i + j: exact, whatever the order.  Five conversions and four FMAs
// put them together in double, and one rounding gives the float.
//
// What is left out: a rounding of 2^-40 R per number, and the four products of i + j = 5.  Together an output is off by 2^-40.5 sqrt(K) R_A R_B (one
// standard deviation; R_A, R_B of its row and column).  That is nothing beside the rounding to float unless the output is small against
// its row and column: one that comes out below 2^-16 sqrt(K) R_A R_B (one in four thousand of what a layer sees) is summed again in double, so that no
// output is off by more than 2^-22 of itself (six standard deviations) beside its rounding.  Rows and columns that hold an infinity, a NaN or nothing but
// numbers beyond 2^-90 .. 2^100 are computed in double, and so is a tile with many such outputs, and everything of a block that has too many to list.
// Against 64 bits over 64 .. 131072 rows and 41 .. 512 columns both forms are off by the same 2.53e-8 (2-norm) and 5.96e-8 (largest, of the
// larger of value and root mean square).
//
// Why: the instruction does 4.7 POP/s here, 60 times what v_mfma_f64_16x16x4_f64 does, so fifteen products are a quarter of the time; what counts
// then is the vector ALU, at ten instructions to cut a number and thirteen to put an output together.
//  * A block holds the digits of B for its columns in registers (all K, 16 NT columns a wavefront) and walks down the rows of A.  Every number
//    of A is cut once per block, by the wavefront that loaded it (whole rows side by side, so that loads are whole lines and a row's maximum is
//    known at once), and its digits go to LDS, from where all wavefronts read them.  The last digits of B, which one product in fifteen takes, wait in
//    LDS too: with them in registers two wavefronts per SIMD do not fit.
//  * Two buffers of rows, one barrier per step.  Half of the wavefronts (one on every SIMD) cut the next step's rows before they multiply, half
//    afterwards, so that the one's vector instructions run beside the other's matrix instructions.
//  * The order of the k within a chunk of 64 is free as long as A and B agree; k = 16 s + 4 g + j for byte 4 s + j of lane group g lets a lane write
//    the digits of the four consecutive k it loaded as one word, and 16 bytes of room after 16 rows spread those words over the banks.
// Measured before / now, us: 131072 rows 256 -> 256 252 / 126, 100 -> 256 112 / 79, 65 536 rows 512 -> 256 248 / 129, 58 624 rows 256 -> 256 131 / 72,
// 4096 rows 512 -> 512 35 / 28.  A step of 32 rows by 256 columns takes 7 us, of which the matrix instructions 3.4; the rest is the
// wavefronts' own chain (read, multiply, put together, cut, write).
// Tried: digits of B in LDS and every wavefront for itself (64 columns each: A is cut, and read in pieces of 16 bytes, once per 64 columns)
// 165 .. 195 us for 131072 x 256 x 256; 16 wavefronts of 16 columns 167 (A's digits are read from LDS twice as often); the outputs that are
// summed again summed at once 236 (the block waits for them at its next barrier).
#include "common.hpp"
#include "gemm_rules.hpp"
#include "product_tile.hpp"
#include "digits.hpp"

namespace csgs {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));

constexpr int DIGITS = 5, CHUNK = DIGIT_CHUNK, WPB = DIGIT_WAVES;
constexpr int LIST = 512, TILE_LIST = 32;   // outputs of a block, and of a tile, that are summed again one by one
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

// A value the wavefront shares, as of here: what follows from it is not computed ahead, outside a loop, and kept in registers
template <typename T>
__device__ inline T here(T x)
{
    asm volatile("" : "+s"(x));
    return x;
}

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
    __shared__ int row_e[2][RS];
    __shared__ uint32_t again_list[LIST];
    __shared__ int again_count;
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
    const int steps_inst = (M_bound + RS - 1) / RS, total = steps_inst * n_inst;

    // ---- rows of A: quad i of this lane
    const int lrow = wave * RW + (QPR == 2 ? 0 : lane / LPR), kquad = lane % LPR;
    auto row_of = [&](int i) { return lrow + (QPR == 2 ? i >> 1 : i * (64 / LPR)); };
    auto quad_of = [&](int i) { return kquad + (QPR == 2 ? 64 * (i & 1) : 0); };
    auto place = [&](int step, int &inst, int &m0) {   // the instances in turn
        inst = n_inst == 1 ? 0 : step % n_inst;
        m0 = (n_inst == 1 ? step : step / n_inst) * RS;
    };
    auto load_a = [&](int step, float (&x)[4 * QUADS]) {
        int inst, m0;
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
                row_e[buf][row_of(QPR * i)] = b[i] == 0 ? E_ZERO : unusable(b[i]) ? E_BAD : e;
#pragma unroll
                for (int j = 0; j < QPR; ++j) sc[QPR * i + j] = scale_of(e);
            }
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
    float x0[4 * QUADS];
    load_a(rg, x0);

    // ---- few rows on the device of the many there is room for: in double, the tiles dealt to all wavefronts
    auto rows_of = [&](int inst) { return rows_dev ? (const int32_t *)((const char *)rows_dev + inst * cs.adj) : nullptr; };
    if (rows_dev) {
        int64_t rows = lane < n_inst ? resolve_count(M_bound, rows_of(lane)) : 0;
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

    // ---- this wavefront's columns of B: digits of k = 64 c + 16 s + 4 grp + j, columns n0 + NT l16 + t
    i32x4 w[KC][NT][DIGITS - 1];
    char *const last_w = last_digits + (wave * KC * NT) * 1024 + lane * 16;
    int ce[NT];
    bool col_zero[NT], any_bad;
    {
        // (a lane's offsets lie below 2^32, and what lies beyond the last k reads the last k)
        const uint32_t ldb4 = (uint32_t)ldb * 4;
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
                    const f32x4u v = *reinterpret_cast<const f32x4u *>((const char *)Bm + (o < ob_max[t] ? o : ob_max[t]));
#pragma unroll
                    for (int j = 0; j < 4; ++j) y[4 * s + j] = v[j];
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const uint32_t o = ob[t] + (k + (uint32_t)j) * ldb4;
                        y[4 * s + j] = *reinterpret_cast<const float *>((const char *)Bm + (o < ob_max[t] ? o : ob_max[t]));
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
                        const f32x2u v = *reinterpret_cast<const f32x2u *>((const char *)Bm + (o < ob2_max ? o : ob2_max));
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
#pragma unroll
        for (int c = 0; c < KC; ++c)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int j = 0; j < 16; j += 2) m[t].take(y[c][t][j], y[c][t][j + 1]);
        float sc[NT];
        bool un = false;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            uint32_t b = m[t].bits(), o = (uint32_t)__shfl_xor((int)b, 16);
            b = b > o ? b : o;
            o = (uint32_t)__shfl_xor((int)b, 32);
            b = b > o ? b : o;
            ce[t] = exponent_of(b) - 46;
            sc[t] = scale_of(exponent_of(b));
            col_zero[t] = b == 0;
            un |= unusable(b);
        }
        any_bad = __any(un);
#pragma unroll
        for (int c = 0; c < KC; ++c)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                end_b(c, y[c][t]);
                i32x4 d[DIGITS];
                cut<4>(y[c][t], [&](int) { return sc[t]; }, d);
#pragma unroll
                for (int p = 0; p < DIGITS - 1; ++p) w[c][t][p] = d[p];
                *reinterpret_cast<i32x4 *>(last_w + (c * NT + t) * 1024) = d[DIGITS - 1];
                __builtin_amdgcn_sched_barrier(0);
            }
    }
    if (tid == 0) again_count = 0;
    put_a(0, x0);
    load_a(rg + rgs, x0);
    __syncthreads();

    const double small = 1073741824.0 * sqrt((double)K);   // 2^-16 sqrt(K) R_A R_B in units of the last sum
    int buf = 0;
    uint32_t code = 0;   // names the step in the list
#pragma unroll 1
    for (int step = rg; step < total; step += rgs, buf ^= 1, code += 1u << 15) {
        int inst, s0;
        place(step, inst, s0);
        const int32_t *rd = rows_of(inst);
        const int M = resolve_count(M_bound, rd);
        char *pc = (char *)(C + (int64_t)s0 * ldc + n0) + inst * cs.out;
        if (wave >= WPB / 2) {
            put_a(buf ^ 1, x0);
            load_a(step + 2 * rgs, x0);
        }
        if (multiplies) {
#pragma unroll 1
            for (int ti = wr; ti < TILES; ti += wrs) {
                const int m0 = s0 + 16 * ti;
                const char *ap = digits[buf] + ti * TSZ + grp * GS + l16 * 16;
                const int re0 = row_e[buf][16 * ti + l16];
                if (m0 >= M) break;
                // what is listed here is done again in double when all steps are through
                auto list = [&](int n) {
                    int at = 0;
                    if (lane == 0) at = atomicAdd(&again_count, n);
                    return __builtin_amdgcn_readfirstlane(at);
                };
                auto list_tile = [&]() {
                    const int at = list(1);
                    if (lane == 0 && at < LIST) again_list[at] = 0x80000000u | code | (uint32_t)((16 * ti) << 8 | wc * 16 * NT);
                };
                if (any_bad || __any(re0 == E_BAD && m0 + l16 < M)) {
                    list_tile();
                } else {
                    i32x4 acc[NT][DIGITS], a[3], wl[NT];
#pragma unroll
                    for (int t = 0; t < NT; ++t)
#pragma unroll
                        for (int s = 0; s < DIGITS; ++s) acc[t][s] = i32x4{0, 0, 0, 0};
                    // A's planes in an order in which two of them take longer than a read from LDS
                    constexpr int order[DIGITS] = {1, 4, 0, 3, 2};
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
                        for (int p = 0; s + p < DIGITS; ++p)
#pragma unroll
                            for (int t = 0; t < NT; ++t)
                                acc[t][s + p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i % 3], p < DIGITS - 1 ? w[c][t][p < DIGITS - 1 ? p : 0] : wl[t], acc[t][s + p], 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    uint32_t at = ((uint32_t)(16 * ti + 4 * grp) * (uint32_t)ldc + (uint32_t)(NT * l16)) * 4;
                    const int left = N - n0 - NT * l16;
                    uint64_t low[4][NT], any = 0;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int re = row_e[buf][16 * ti + 4 * grp + i];
                        float v[NT];
#pragma unroll
                        for (int t = 0; t < NT; ++t) {
                            double d = (double)acc[t][0][i];
#pragma unroll
                            for (int s = 1; s < DIGITS; ++s) d = __builtin_fma(d, 256.0, (double)acc[t][s][i]);
                            v[t] = (float)__builtin_amdgcn_ldexp(d, re + ce[t]);
                            low[i][t] = __ballot(fabs(d) < small);
                            any |= low[i][t];
                        }
                        if (m0 + 4 * grp + i < M) {
                            float *p = reinterpret_cast<float *>(pc + (int64_t)i * ldc * 4 + at);
                            if (left >= NT) store_floats<NT>(p, v);
                            else if (NT == 2 && left == 1) *p = v[0];
                        }
                    }
                    if (any) {
                        int count = 0;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int ro = 16 * ti + 4 * grp + i;
                            const bool row_ok = s0 + ro < M && row_e[buf][ro] != E_ZERO;
#pragma unroll
                            for (int t = 0; t < NT; ++t) {
                                low[i][t] &= __ballot(row_ok && t < left && !col_zero[t]);
                                count += __popcll(low[i][t]);
                            }
                        }
                        if (count > TILE_LIST) {
                            list_tile();
                        } else if (count > 0) {
                            int at0 = list(count);
#pragma unroll
                            for (int i = 0; i < 4; ++i)
#pragma unroll
                                for (int t = 0; t < NT; ++t) {
                                    const int pos = at0 + __popcll(low[i][t] & (((uint64_t)1 << lane) - 1));
                                    if (((low[i][t] >> lane) & 1) && pos < LIST)
                                        again_list[pos] = code | (uint32_t)((16 * ti + 4 * grp + i) << 8 | (wc * 16 * NT + NT * l16 + t));
                                    at0 += __popcll(low[i][t]);
                                }
                        }
                    }
                }
            }
        }
        if (wave < WPB / 2) {
            put_a(buf ^ 1, x0);
            load_a(step + 2 * rgs, x0);
        }
        __syncthreads();
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // some of the outputs are written again
    __syncthreads();
    const int count = __builtin_amdgcn_readfirstlane(again_count);
    if (count > LIST) {   // more than the list holds: everything
#pragma unroll 1
        for (int step = rg; step < total; step += rgs) {
            const int inst = step % n_inst, s0 = step / n_inst * RS;
            const int32_t *rd = rows_of(inst);
            if (!multiplies) break;
            const int end = NT * row_tiles(resolve_count(M_bound, rd) - s0, RS);   // (a tile that starts past the last row would read before the matrix)
#pragma unroll 1
            for (int ti = wr * NT; ti < end; ti += ti % NT == NT - 1 ? (wrs - 1) * NT + 1 : 1)
                if (n0 + 16 * (ti % NT) < N)
                    product_tile<MODE, 1, 1, TAIL_32, uint32_t>((const float *)((const char *)A + inst * cs.x), here(lda), here(Bm), here(ldb),
                                                                (float *)((char *)C + inst * cs.out), here(ldc), nullptr, here(M_bound), here(N),
                                                                here(K), rd, s0 + 16 * (ti / NT), n0 + 16 * (ti % NT));
        }
        return;
    }
    // tiles, and outputs that came out small against their row's and column's maxima: four at a time
#pragma unroll 1
    for (int s = 4 * wave; s < count; s += 4 * WPB) {
        const uint32_t what = again_list[s + grp < count ? s + grp : count - 1];
        const bool is = s + grp < count && !(what >> 31);
        const int st = (int)(what >> 15 & 0xFFFF) * rgs + rg, in = st % n_inst;
        const int64_t m = st / n_inst * RS + (int)((what >> 8) & 127);
        const int n = cg * wcs * 16 * NT + (int)(what & 255);
        const float *pa = (const float *)((const char *)A + in * cs.x) + m * lda;
        const float *pb = MODE == MODE_DZ ? Bm + (int64_t)n * ldb : Bm + n;
        const int64_t bs = MODE == MODE_DZ ? 1 : ldb;
        double sum = 0.0;
        for (int k0 = l16; k0 < K; k0 += 256) {
            float va[16], vb[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int k = k0 + 16 * u < K ? k0 + 16 * u : K - 1;
                va[u] = pa[k];
                vb[u] = pb[k * bs];
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) sum = __builtin_fma((double)va[u], k0 + 16 * u < K ? (double)vb[u] : 0.0, sum);
        }
#pragma unroll
        for (int o = 8; o; o >>= 1) sum += __shfl_xor(sum, o);
        if (l16 == 0 && is) ((float *)((char *)C + in * cs.out))[m * ldc + n] = (float)sum;
        const int tiles = __popcll(__ballot(l16 == 0 && s + grp < count && what >> 31));
#pragma unroll 1
        for (int g = 0; tiles && g < 4 * NT; ++g) {
            const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)what, 16 * (g / NT));
            const int nt = cg * wcs * 16 * NT + (int)(w & 255) + 16 * (g % NT);
            if (s + g / NT >= count || !(w >> 31) || nt >= N) continue;
            const int sg = (int)(w >> 15 & 0xFFFF) * rgs + rg, ig = sg % n_inst;
            const int32_t *rd = rows_of(ig);
            product_tile<MODE, 1, 1, TAIL_32, uint32_t>((const float *)((const char *)A + ig * cs.x), here(lda), here(Bm), here(ldb),
                                                        (float *)((char *)C + ig * cs.out), here(ldc), nullptr, here(M_bound), here(N),
                                                        here(K), rd, sg / n_inst * RS + (int)((w >> 8) & 127), nt);
        }
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
        if (MODE == MODE_FWD) CSGS_DIGITS_AS(K_GEMM, KC, NT);       \
        else CSGS_DIGITS_AS(K_GEMM_DZ, KC, NT);                     \
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
