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
// Large Z W and G W^T leave these kernels for sums of 8-bit digits on the integer matrix cores, where digits_plan (gemm_rules.hpp)
// expects those to be done first: digits.hip, 131072 x 256 x 256 252 -> 126 us.  The figures above are for these kernels.
//
// Block ids are remapped so that consecutive tiles (same rows of Z, neighbouring column tiles)
// land on the same XCD and share its L2.
#include <type_traits>
#include "common.hpp"
#include "gemm_rules.hpp"
#include "product_tile.hpp"
#include "digits.hpp"

namespace csgs {

template <int MODE, int RT, int NT, int TAIL, typename OFF>
__global__ __launch_bounds__(256, RT * NT >= 6 ? 2 : (RT * NT >= 4 ? 3 : 4)) void gemm_wave_k(
    const float *__restrict__ A, int64_t lda, const float *__restrict__ Bm, int64_t ldb, float *__restrict__ C, int64_t ldc,
    double *__restrict__ partial, int M_bound, int N, int K_bound, const int32_t *__restrict__ rows_dev, int tiles_n, int n_tiles,
    int n_blocks, CompStride cs)
{
    constexpr bool DW = MODE == MODE_DW;
    constexpr int BM = 16 * RT, BN = 16 * NT;
    A = comp_ptr(A, cs.x); C = comp_ptr(C, cs.out); rows_dev = comp_ptr(rows_dev, cs.adj);   // B (the weights) is shared
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    // XCD-aware tile order: hardware deals consecutive block ids round-robin to the 8 XCDs
    const int bid = (int)blockIdx.x;
    const int per_xcd = (n_blocks + 7) / 8;
    // (rotated by the instance: the row tiles beyond a mini-batch's row count are the last ones, and with the
    // same order for every instance they would all fall to the same XCD, which then idles)
    const int blk = (((bid & 7) + (int)blockIdx.z) & 7) * per_xcd + (bid >> 3);
    const int tile = DW ? blk : blk * 4 + wave;
    if (blk >= n_blocks || tile >= n_tiles) return;   // for dW the whole block
    product_tile<MODE, RT, NT, TAIL, OFF>(A, lda, Bm, ldb, C, ldc, partial, M_bound, N, K_bound, rows_dev, (tile / tiles_n) * BM,
                                          (tile % tiles_n) * BN);
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
    const DigitsPlan digits = digits_plan(M, N, K, lda, ldb, ldc, ci.n, MODE == MODE_DZ);
    if (digits.use) {
        launch_digits<MODE>(digits, A, lda, B, ldb, C, ldc, M, N, K, M_dev, st, ci);
        return;
    }
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
