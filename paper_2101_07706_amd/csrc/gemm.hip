// csgs_layer_gemm: H = Z W (Section 3, Eq. 1), fp32 in, fp32 out, fp64 matrix-core accumulation, and the two gradient
// products of a layer.
//
// Why double: sampled rows carry 1/p_j discounts that compound over the layers, so the products
// z*w of a near-cancelling output reach magnitude 10 and more while the tolerance is 1e-5
// absolute.  fp32 MFMA with double master accumulators over runs of 32 k was measured to miss it
// (5.9e-5 against 3.5e-5 allowed on one output of the largest configuration).  The operands are
// widened to double (exact), products of two 24-bit mantissas are exact in
// double, and v_mfma_f64_16x16x4_f64 accumulates in double, so the only rounding is the final
// conversion to float.
//
// What bounds it, and why it has this form: v_mfma_f64_16x16x4_f64 occupies a SIMD for 29 ns (72 TFLOP/s over the device), and
// the vector ALU stands still meanwhile: every vector instruction, of any wavefront, adds its own 1.8 ns (measured with adds,
// conversions and FMAs beside the MFMAs, one and two wavefronts per SIMD).  So what counts is vector instructions per MFMA,
// and the time until all SIMDs multiply.
//  * A wavefront works for itself on a tile of 16 RT x 16 NT outputs: no LDS, no barrier.  Its operands come straight
//    from L1 / L2 (16 bytes a cycle and compute unit), the next 32 k on their way while the current ones are multiplied.
//  * The lane group l / 16 = g feeds k = 8 g + s at step s, for both operands alike, which leaves the sum unchanged.  A
//    lane then needs 8 consecutive k of a row where the k lie side by side (two 16-byte loads), and NT (RT for Z^T)
//    consecutive columns of 8 rows where the columns do (8 loads of up to 16 bytes); its NT results of a row go out in one store.
//  * All addresses are an offset that a lane keeps from the start plus scalar arithmetic, so the only vector instructions in the loop are
//    the conversions: RT + NT per RT * NT MFMAs.
//  * Rows and columns that do not exist read the nearest ones that do and are not stored, so no operand needs a mask; a K that is no
//    multiple of 32 takes its last k first, in steps of four.
// With blocks of four wavefronts that staged 64 or 128 x 64 tiles in LDS (conversions by every wavefront, addresses in vector
// registers, a barrier per 32 k) before: 4096 x 512 x 512 46 -> 37 us, 4096 x 300 x 512 36 -> 25, 4500 x 512 x 100 29 -> 13,
// 8192 x 256 x 256 25 -> 20, 8192 x 256 x 47 12.2 -> 7.7, 2048 x 602 x 256 27 -> 15.5, 1024 x 256 x 256 9.5 -> 5.9,
// 131072 x 256 x 256 278 -> 262, odd sizes (20000 x 301 x 201) 85 -> 53.
//
// Block ids are remapped so that consecutive tiles (same rows of Z, neighbouring column tiles)
// land on the same XCD and share its L2.
#include <type_traits>
#include "common.hpp"

#include "gemm_rules.hpp"

namespace csgs {

// The same kernel serves the layer's forward product and its two gradient products; they differ in
// how the operands lie in memory and in where the result goes:
//   FWD  H  = Z W        A(m,k) = Z[m][k]           B(k,n) = W[k][n]      C float [M x N]
//   DZ   dZ = G W^T      A(m,k) = G[m][k]           B(k,n) = W[n][k]      C float [M x N]
//   DW   dW = Z^T G      A(m,k) = Z[k][m]           B(k,n) = G[k][n]      the reduction dimension (the rows of the
//        sampled layer) is dealt to the four wavefronts of a block, whose sums are added in LDS, and over blockIdx.y; the
//        parts go out in double and a second kernel adds them in a fixed order (one part: float, no second kernel).
enum { MODE_FWD = 0, MODE_DZ = 1, MODE_DW = 2 };

// MFMA steps (of four k) that a kernel has for the K % 32 k behind the whole chunks
enum { TAIL_NONE = 0, TAIL_8 = 2, TAIL_32 = 8 };

// N consecutive floats at a byte offset from an address the whole wavefront shares.  Four bytes of alignment are
// enough for any width of global load on this part.
template <int N, typename OFF>
__device__ inline void load_floats(const char *base, OFF off, float *out)
{
    typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
    typedef float f2 __attribute__((ext_vector_type(2), aligned(4)));
    const char *p = base + off;
    if constexpr (N == 4) {
        const f4 x = *reinterpret_cast<const f4 *>(p);
        out[0] = x[0]; out[1] = x[1]; out[2] = x[2]; out[3] = x[3];
    } else if constexpr (N >= 2) {
        const f2 x = *reinterpret_cast<const f2 *>(p);
        out[0] = x[0]; out[1] = x[1];
        if constexpr (N == 3) out[2] = *reinterpret_cast<const float *>(p + 8);
    } else {
        out[0] = *reinterpret_cast<const float *>(p);
    }
}
template <int N>
__device__ inline void store_floats(float *p, const float *v)
{
    typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
    typedef float f2 __attribute__((ext_vector_type(2), aligned(4)));
    if constexpr (N == 4) {
        *reinterpret_cast<f4 *>(p) = f4{v[0], v[1], v[2], v[3]};
    } else if constexpr (N >= 2) {
        *reinterpret_cast<f2 *>(p) = f2{v[0], v[1]};
        if constexpr (N == 3) p[2] = v[2];
    } else {
        *p = v[0];
    }
}

// OFF: a lane's byte offsets; 64 bits only where rows lie 2^24 floats apart or more.
// Registers: two sets of operands (16 (RT + NT) in all) and 8 RT NT of sums; 230 for 2 x 4, 135 for 2 x 2.
template <int MODE, int RT, int NT, int TAIL, typename OFF>
__global__ __launch_bounds__(256, RT * NT >= 6 ? 2 : (RT * NT >= 4 ? 3 : 4)) void gemm_wave_k(
    const float *__restrict__ A, int64_t lda, const float *__restrict__ Bm, int64_t ldb, float *__restrict__ C, int64_t ldc,
    double *__restrict__ partial, int M_bound, int N, int K_bound, const int32_t *__restrict__ rows_dev, int tiles_n, int n_tiles,
    int n_blocks, CompStride cs)
{
    constexpr bool DW = MODE == MODE_DW, B_KMAJOR = MODE == MODE_DZ;
    constexpr int BM = 16 * RT, BN = 16 * NT;
    A = comp_ptr(A, cs.x); C = comp_ptr(C, cs.out); rows_dev = comp_ptr(rows_dev, cs.adj);   // B (the weights) is shared
    const int lane = (int)(threadIdx.x & 63), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int grp = lane >> 4, l16 = lane & 15;
    // XCD-aware tile order: hardware deals consecutive block ids round-robin to the 8 XCDs
    const int bid = (int)blockIdx.x;
    const int per_xcd = (n_blocks + 7) / 8;
    // (rotated by the instance: the row tiles beyond a mini-batch's row count are the last ones, and with the
    // same order for every instance they would all fall to the same XCD, which then idles)
    const int blk = (((bid & 7) + (int)blockIdx.z) & 7) * per_xcd + (bid >> 3);
    const int tile = DW ? blk : blk * 4 + wave;
    if (blk >= n_blocks || tile >= n_tiles) return;   // for dW the whole block
    const int m0 = (tile / tiles_n) * BM, n0 = (tile % tiles_n) * BN;
    const int m_dev = (!DW && rows_dev) ? *rows_dev : M_bound;
    const int K = DW ? __builtin_amdgcn_readfirstlane(resolve_count(K_bound, rows_dev)) : K_bound;

    // ---- where this lane's operands lie: bytes from addresses that the whole wavefront shares
    OFF offa[DW ? 1 : RT], offb[B_KMAJOR ? NT : 1];
    const char *pa, *pb;
    if constexpr (DW) {
        const int m = m0 + RT * l16 < M_bound - RT ? m0 + RT * l16 : M_bound - RT;
        offa[0] = (OFF)(8 * grp) * (OFF)(lda * 4) + (OFF)m * 4;
        pa = reinterpret_cast<const char *>(A);
    } else {
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const int row = m0 + 16 * r + l16 < M_bound ? 16 * r + l16 : M_bound - 1 - m0;
            offa[r] = (OFF)row * (OFF)(lda * 4) + (OFF)(32 * grp);
        }
        pa = reinterpret_cast<const char *>(A + (int64_t)m0 * lda);
    }
    const int col0 = n0 + NT * l16 < N - NT ? n0 + NT * l16 : N - NT;   // this lane's first column
    if constexpr (B_KMAJOR) {
        const int nb = n0 < N - NT ? n0 : N - NT;
#pragma unroll
        for (int t = 0; t < NT; ++t) offb[t] = (OFF)(col0 - nb + t) * (OFF)(ldb * 4) + (OFF)(32 * grp);
        pb = reinterpret_cast<const char *>(Bm + (int64_t)nb * ldb);
    } else {
        offb[0] = (OFF)(8 * grp) * (OFF)(ldb * 4) + (OFF)col0 * 4;
        pb = reinterpret_cast<const char *>(Bm);
    }

    struct Set {
        float a[8][RT], b[8][NT];
    };
    const int64_t lda4 = lda * 4, ldb4 = ldb * 4;
    // the chunk whose first k stands at ca, cb
    auto load = [&](Set &x, const char *ca, const char *cb) {
        // (the offsets are kept apart from the shared address by hand: left alone the compiler adds the two in every lane)
#pragma unroll
        for (auto &o : offa) asm volatile("" : "+v"(o));
#pragma unroll
        for (auto &o : offb) asm volatile("" : "+v"(o));
        if constexpr (DW) {
#pragma unroll
            for (int s = 0; s < 8; ++s, ca += lda4) load_floats<RT>(ca, offa[0], x.a[s]);
        } else {
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                float v[8];
                load_floats<4>(ca, offa[r], v);
                load_floats<4>(ca + 16, offa[r], v + 4);
#pragma unroll
                for (int s = 0; s < 8; ++s) x.a[s][r] = v[s];
            }
        }
        if constexpr (B_KMAJOR) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                float v[8];
                load_floats<4>(cb, offb[t], v);
                load_floats<4>(cb + 16, offb[t], v + 4);
#pragma unroll
                for (int s = 0; s < 8; ++s) x.b[s][t] = v[s];
            }
        } else {
#pragma unroll
            for (int s = 0; s < 8; ++s, cb += ldb4) load_floats<NT>(cb, offb[0], x.b[s]);
        }
    };
    doublex4 acc[RT][NT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[r][t] = doublex4{0.0, 0.0, 0.0, 0.0};
    auto step = [&](const float *av, const float *bv) {
        double a[RT], b[NT];
#pragma unroll
        for (int r = 0; r < RT; ++r) a[r] = (double)av[r];
#pragma unroll
        for (int t = 0; t < NT; ++t) b[t] = (double)bv[t];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < RT; ++r) acc[r][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[r], b[t], acc[r][t], 0, 0, 0);
    };
    auto multiply = [&](const Set &x) {
#pragma unroll
        for (int s = 0; s < 8; ++s) step(x.a[s], x.b[s]);
    };
    // the last K % 32 k: lane group g feeds k = kt + 4 s + g, so no step multiplies more than three k that do not exist
    constexpr int TS = DW ? TAIL_32 : TAIL;
    struct Tail {
        float a[TS > 0 ? TS : 1][RT], b[TS > 0 ? TS : 1][NT];
    };
    const int kt = K & ~31, tail = K & 31;
    auto load_tail = [&](Tail &x) {
        const char *ta = pa + (DW ? kt * lda4 : (int64_t)kt * 4), *tb = pb + (B_KMAJOR ? (int64_t)kt * 4 : kt * ldb4);
#pragma unroll
        for (int s = 0; s < TS; ++s) {
            const int kb = 4 * s < tail - 1 ? 4 * s : (tail > 0 ? tail - 1 : -1);   // (without a tail the last k stands in)
            const int g = kb + grp < tail - 1 ? grp : tail - 1 - kb;
            if constexpr (DW) {
                load_floats<RT>(ta + kb * lda4, offa[0] - (OFF)(8 * grp) * (OFF)lda4 + (OFF)g * (OFF)lda4, x.a[s]);
            } else {
#pragma unroll
                for (int r = 0; r < RT; ++r) load_floats<1>(ta + kb * 4, offa[r] - (OFF)(32 * grp) + (OFF)(4 * g), &x.a[s][r]);
            }
            if constexpr (B_KMAJOR) {
#pragma unroll
                for (int t = 0; t < NT; ++t) load_floats<1>(tb + kb * 4, offb[t] - (OFF)(32 * grp) + (OFF)(4 * g), &x.b[s][t]);
            } else {
                load_floats<NT>(tb + kb * ldb4, (OFF)g * (OFF)ldb4 + (OFF)col0 * 4, x.b[s]);
            }
        }
    };
    auto multiply_tail = [&](Tail &x) {
#pragma unroll
        for (int s = 0; s < TS; ++s) {
            if (4 * s >= tail) break;
            if (4 * s + 4 > tail) {
                const bool ok = 4 * s + grp < tail;
#pragma unroll
                for (int r = 0; r < RT; ++r) x.a[s][r] = ok ? x.a[s][r] : 0.f;
#pragma unroll
                for (int t = 0; t < NT; ++t) x.b[s][t] = ok ? x.b[s][t] : 0.f;
            }
            step(x.a[s], x.b[s]);
        }
    };

    // ---- chunks of 32 k, `stride` apart: lane group g feeds k = 8 g + s at step s
    int c0 = 0, n_chunks = K >> 5;
    int64_t sa = 128, sb = B_KMAJOR ? 128 : 32 * ldb4;   // bytes from one chunk of this wavefront to its next
    bool own_tail = true;
    if constexpr (DW) {   // this block's chunks, dealt to its four wavefronts in turn
        const int all = (K + 31) >> 5, per = (all + (int)gridDim.y - 1) / (int)gridDim.y;
        const int first = (int)blockIdx.y * per + wave, end = first - wave + per < all ? first - wave + per : all;
        const int whole_end = end < n_chunks ? end : n_chunks;
        own_tail = tail && end == all && first < all && ((all - 1 - first) & 3) == 0 && first <= all - 1;
        c0 = first * 32;
        sa = 128 * lda4;
        sb = 128 * ldb4;
        n_chunks = whole_end > first ? (whole_end - first + 3) >> 2 : 0;
    }
    Set s0, s1;
    Tail tl;
    if constexpr (!DW && TAIL != TAIL_NONE) load_tail(tl);
    const char *ca = pa, *cb = pb;
    if constexpr (DW) {
        ca += c0 * lda4;
        cb += c0 * ldb4;
    }
    if (n_chunks > 0) load(s0, ca, cb);
    if constexpr (!DW) {
        // a row count on the device is needed only now that loads are on their way
        if (m0 >= (m_dev < M_bound ? m_dev : M_bound)) return;
        if constexpr (TAIL != TAIL_NONE) multiply_tail(tl);
    }
    if (n_chunks > 0) {
        // The next chunk is asked for before this one is multiplied, and no load sits under a condition of its own: the
        // compiler then waits for exactly the chunk it needs
        int c = 0;
        for (; c + 2 < n_chunks; c += 2) {
            load(s1, ca += sa, cb += sb);
            multiply(s0);
            load(s0, ca += sa, cb += sb);
            multiply(s1);
        }
        if (c + 2 == n_chunks) {
            load(s1, ca += sa, cb += sb);
            multiply(s0);
            multiply(s1);
        } else {
            multiply(s0);
        }
    }
    if constexpr (DW) {
        if (own_tail) {
            load_tail(tl);
            multiply_tail(tl);
        }
    }

    // ---- accumulator element i of lane (g, l) belongs to row g + 4 i of operand A's 16 and to column l of B's
    const bool col_ok = n0 + NT * l16 < N;
    if constexpr (!DW) {
        const int M = m_dev < M_bound ? m_dev : M_bound;
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = m0 + 16 * r + grp + 4 * i;
                float v[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) v[t] = (float)acc[r][t][i];
                if (row < M && col_ok) store_floats<NT>(C + (int64_t)row * ldc + col0, v);
            }
    } else {
        // the four wavefronts' sums, added in wavefront order
        constexpr int E = RT * NT * 4;
        __shared__ double red[4][E][64];
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) red[wave][(r * 4 + i) * NT + t][lane] = acc[r][t][i];
        __syncthreads();
        static_assert(E % (4 * NT) == 0 && (E / 4) % NT == 0, "whole rows per wavefront");
#pragma unroll
        for (int j = 0; j < RT; ++j) {
            const int ri = wave * RT + j, r = ri >> 2, i = ri & 3;
            const int ma = m0 + RT * (grp + 4 * i);
            const int row = (ma < M_bound - RT ? ma : M_bound - RT) + r;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int e = ri * NT + t;
                const double s = ((red[0][e][lane] + red[1][e][lane]) + red[2][e][lane]) + red[3][e][lane];
                if (ma < M_bound && col_ok) {
                    if (C) C[(int64_t)row * ldc + col0 + t] = (float)s;   // the only part
                    else partial[((int64_t)blockIdx.y * M_bound + row) * N + col0 + t] = s;
                }
            }
        }
    }
}
// dW[i] = sum over the K parts, in ascending part order (fixed: the result does not depend on timing)
__global__ __launch_bounds__(256) void gemm_reduce_parts(const double *__restrict__ partial, int parts, int64_t count,
                                                         int N, float *__restrict__ C, int64_t ldc)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    double s = 0.0;
    int p = 0;
    for (; p + 8 <= parts; p += 8) {   // eight loads in flight, added in ascending part order
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = partial[(int64_t)(p + u) * count + i];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; p < parts; ++p) s += partial[(int64_t)p * count + i];
    C[(i / N) * ldc + (i % N)] = (float)s;
}

template <int MODE>
static void launch_product(const float *A, int64_t lda, const float *B, int64_t ldb, float *C, int64_t ldc, int M, int N, int K,
                           const int32_t *M_dev, hipStream_t st, const CompInst &ci)
{
    const bool far = far_apart(lda, ldb);
    const Shape s = far ? Shape{1, 1, 0.0} : pick_shape(M, N, ci.n, MODE == MODE_DZ);
    const int tm = (int)(((int64_t)M + 16 * s.rt - 1) / (16 * s.rt)), tn = (int)(((int64_t)N + 16 * s.nt - 1) / (16 * s.nt));
    const int n_tiles = tm * tn, n_blocks = (n_tiles + 3) / 4;
    const dim3 grid((unsigned)((n_blocks + 7) / 8 * 8), 1, (unsigned)ci.n);
    double *none = nullptr;
    constexpr int STAGE = MODE;   // (names the launch in the profile)
#define CSGS_PRODUCT(RT, NT, TAIL, OFF)                                                                                                       \
    do {                                                                                                                                      \
        if (STAGE == MODE_FWD)                                                                                                                \
            CSGS_LAUNCH(K_GEMM, (gemm_wave_k<MODE, RT, NT, TAIL, OFF>), grid, dim3(256), st, A, lda, B, ldb, C, ldc, none, M, N, K, M_dev,    \
                        tn, n_tiles, n_blocks, ci.cs);                                                                                        \
        else                                                                                                                                  \
            CSGS_LAUNCH(K_GEMM_DZ, (gemm_wave_k<MODE, RT, NT, TAIL, OFF>), grid, dim3(256), st, A, lda, B, ldb, C, ldc, none, M, N, K, M_dev, \
                        tn, n_tiles, n_blocks, ci.cs);                                                                                        \
    } while (0)
#define CSGS_SHAPE(RT, NT)                                                  \
    if (s.rt == RT && s.nt == NT) {                                         \
        if (K % 32 == 0) CSGS_PRODUCT(RT, NT, TAIL_NONE, uint32_t);         \
        else if (K % 32 <= 8) CSGS_PRODUCT(RT, NT, TAIL_8, uint32_t);       \
        else CSGS_PRODUCT(RT, NT, TAIL_32, uint32_t);                       \
    }
    if (far) {
        CSGS_PRODUCT(1, 1, TAIL_32, uint64_t);
        return;
    }
    CSGS_SHAPE(2, 4) CSGS_SHAPE(2, 3) CSGS_SHAPE(2, 2) CSGS_SHAPE(2, 1) CSGS_SHAPE(1, 4) CSGS_SHAPE(1, 3) CSGS_SHAPE(1, 2) CSGS_SHAPE(1, 1)
#undef CSGS_SHAPE
#undef CSGS_PRODUCT
}

}  // namespace csgs

using namespace csgs;

static bool too_many_tiles(int64_t M, int64_t N) { return ((M + 127) / 128) * ((N + 31) / 32) > 0x3FFFFFFF; }

extern "C" int csgs_layer_gemm(const float *Z, int64_t ldz, int32_t M, const int32_t *M_dev, int32_t K, const float *W, int64_t ldw,
                               int32_t Nout, float *H, int64_t ldh, void *stream)
{
    return csgs_layer_gemm_n(nullptr, Z, ldz, M, M_dev, K, W, ldw, Nout, H, ldh, stream);
}

extern "C" int csgs_layer_gemm_n(const csgs_inst_strides *inst, const float *Z, int64_t ldz, int32_t M, const int32_t *M_dev,
                                 int32_t K, const float *W, int64_t ldw, int32_t Nout, float *H, int64_t ldh, void *stream)
{
    if (!Z || !W || !H || M <= 0 || K <= 0 || Nout <= 0 || ldz < K || ldw < Nout || ldh < Nout) return CSGS_EINVAL;
    CompInst ci;
    if (open_instances(inst, &ci) != CSGS_OK) return CSGS_EINVAL;
    if (too_many_tiles(M, Nout)) return CSGS_EUNSUPPORTED;
    launch_product<MODE_FWD>(Z, ldz, W, ldw, H, ldh, M, Nout, K, M_dev, (hipStream_t)stream, ci);
    CSGS_LAUNCH_CHECK();
    return CSGS_OK;
}

extern "C" int csgs_layer_gemm_grad_z(const float *G, int64_t ldg, int32_t M, const int32_t *M_dev, int32_t Nout, const float *W,
                                      int64_t ldw, int32_t K, float *dZ, int64_t lddz, void *stream)
{
    if (!G || !W || !dZ || M <= 0 || K <= 0 || Nout <= 0 || ldg < Nout || ldw < Nout || lddz < K) return CSGS_EINVAL;
    if (too_many_tiles(M, K)) return CSGS_EUNSUPPORTED;
    // output [M x K]; the reduction runs over the Nout columns of G
    launch_product<MODE_DZ>(G, ldg, W, ldw, dZ, lddz, M, K, Nout, M_dev, (hipStream_t)stream, CompInst{});
    CSGS_LAUNCH_CHECK();
    return CSGS_OK;
}

extern "C" size_t csgs_layer_gemm_grad_w_scratch_bytes(int32_t M, int32_t K, int32_t Nout)
{
    if (M <= 0 || K <= 0 || Nout <= 0) return 0;
    return (size_t)dw_max_parts(M, K, Nout) * (size_t)K * (size_t)Nout * sizeof(double);
}

// dW = Z^T G with the partial sums in `parts` (device, at least csgs_layer_gemm_grad_w_scratch_bytes bytes)
static int grad_w_launch(const float *Z, int64_t ldz, const float *G, int64_t ldg, int32_t M, const int32_t *M_dev, int32_t K,
                         int32_t Nout, float *dW, int64_t lddw, double *parts_buf, hipStream_t st)
{
    // kernel terms: output [K x Nout], reduction over the M rows (their count may live on the device)
    Shape s;
    int parts;
    dw_split(M, K, Nout, &s, &parts);
    const bool far = far_apart(ldz, ldg);
    if (far) s = Shape{1, 1, 0.0};
    const int tm = (int)(((int64_t)K + 16 * s.rt - 1) / (16 * s.rt)), tn = (int)(((int64_t)Nout + 16 * s.nt - 1) / (16 * s.nt));
    const int n_tiles = tm * tn;
    const dim3 grid((unsigned)((n_tiles + 7) / 8 * 8), (unsigned)parts);
    float *out = parts == 1 ? dW : nullptr;
#define CSGS_DW(RT, NT, OFF)                                                                                                                \
    CSGS_LAUNCH(K_GEMM_DW, (gemm_wave_k<MODE_DW, RT, NT, TAIL_32, OFF>), grid, dim3(256), st, Z, ldz, G, ldg, out, lddw, parts_buf, K, Nout, \
                M, M_dev, tn, n_tiles, n_tiles, CompStride{0, 0, 0, 0})
    if (far) CSGS_DW(1, 1, uint64_t);
    else if (s.nt == 3) CSGS_DW(2, 3, uint32_t);
    else if (s.rt == 2 && s.nt == 4) CSGS_DW(2, 4, uint32_t);
    else if (s.rt == 2 && s.nt == 2) CSGS_DW(2, 2, uint32_t);
    else if (s.rt == 2) CSGS_DW(2, 1, uint32_t);
    else if (s.nt == 4) CSGS_DW(1, 4, uint32_t);
    else if (s.nt == 2) CSGS_DW(1, 2, uint32_t);
    else CSGS_DW(1, 1, uint32_t);
#undef CSGS_DW
    CSGS_LAUNCH_CHECK();
    if (parts == 1) return CSGS_OK;
    const int64_t count = (int64_t)K * Nout;
    CSGS_LAUNCH(K_GEMM_DW_REDUCE, gemm_reduce_parts, dim3((unsigned)((count + 255) / 256)), dim3(256), st,
                (const double *)parts_buf, parts, count, Nout, dW, lddw);
    CSGS_LAUNCH_CHECK();
    return CSGS_OK;
}

extern "C" int csgs_layer_gemm_grad_w(const float *Z, int64_t ldz, const float *G, int64_t ldg, int32_t M, const int32_t *M_dev,
                                      int32_t K, int32_t Nout, float *dW, int64_t lddw, void *scratch, size_t scratch_bytes,
                                      void *stream)
{
    if (!Z || !G || !dW || M <= 0 || K <= 0 || Nout <= 0 || ldz < K || ldg < Nout || lddw < Nout || !scratch ||
        ((uintptr_t)scratch & 7))
        return CSGS_EINVAL;
    if (scratch_bytes < csgs_layer_gemm_grad_w_scratch_bytes(M, K, Nout)) return CSGS_EWORKSPACE;
    return grad_w_launch(Z, ldz, G, ldg, M, M_dev, K, Nout, dW, lddw, (double *)scratch, (hipStream_t)stream);
}

// ---------------------------------------------------------------- the same without any allocation
// The partial sums of csgs_layer_gemm_grad_w_static live in this array, which is part of the library's
// device image: every device the library runs on holds its own copy, at its own address, until the
// process ends.  Host code never uses the array's name as an address; the address on the current
// device is looked up once per device and kept.
static __device__ __align__(256) unsigned char scratch[CSGS_GRAD_W_STATIC_BYTES];
static std::atomic<void *> g_static_scratch[64];   // per device; null = not looked up yet (zero-initialised)

// Address of `scratch` on the current device, or null.
static void *static_scratch_ptr()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    void *p = g_static_scratch[dev].load(std::memory_order_acquire);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
        g_static_scratch[dev].store(p, std::memory_order_release);   // every thread would store the same address
    }
    return p;
}

extern "C" int csgs_layer_gemm_grad_w_static(const float *Z, int64_t ldz, const float *G, int64_t ldg, int32_t M,
                                             const int32_t *M_dev, int32_t K, int32_t Nout, float *dW, int64_t lddw, void *stream)
{
    if (!Z || !G || !dW || M <= 0 || K <= 0 || Nout <= 0 || ldz < K || ldg < Nout || lddw < Nout) return CSGS_EINVAL;
    if (csgs_layer_gemm_grad_w_scratch_bytes(M, K, Nout) > (size_t)CSGS_GRAD_W_STATIC_BYTES) return CSGS_EWORKSPACE;
    void *parts_buf = static_scratch_ptr();
    if (!parts_buf) return CSGS_ELAUNCH;
    // every part that the reduction reads is written by the product kernel of the same call: nothing to clear
    return grad_w_launch(Z, ldz, G, ldg, M, M_dev, K, Nout, dW, lddw, (double *)parts_buf, (hipStream_t)stream);
}

static const char *const kErr[] = {"ok",
                                   "invalid argument",
                                   "workspace too small",
                                   "unsupported dtype or dimension",
                                   "fixed-point format out of range",
                                   "kernel launch failed"};

extern "C" const char *csgs_strerror(int code)
{
    const int i = -code;
    return (i >= 0 && i < (int)(sizeof(kErr) / sizeof(kErr[0]))) ? kErr[i] : "unknown error";
}
