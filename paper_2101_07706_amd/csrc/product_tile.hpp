// The layer products on the fp64 matrix cores: one wavefront's tile (what bounds it and why it has this form: gemm.hip).
#pragma once
#include "common.hpp"

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

// A value the wavefront shares, as of here: what follows from it is not computed ahead, outside a loop, and kept in registers
template <typename T>
__device__ inline T here(T x)
{
    asm volatile("" : "+s"(x));
    return x;
}

template <typename T>
__device__ inline T here_v(T x)   // the same for a lane's own
{
    asm volatile("" : "+v"(x));
    return x;
}

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

// One wavefront's tile (for dW: a block's), output rows m0 .. m0 + 16 RT - 1 and columns n0 .. n0 + 16 NT - 1.
// OFF: a lane's byte offsets; 64 bits only where rows lie 2^24 floats apart or more.
// Registers: two sets of operands (16 (RT + NT) in all) and 8 RT NT of sums; 230 for 2 x 4, 135 for 2 x 2.
template <int MODE, int RT, int NT, int TAIL, typename OFF>
__device__ inline __attribute__((always_inline)) void product_tile(
    const float *__restrict__ A, int64_t lda, const float *__restrict__ Bm, int64_t ldb, float *__restrict__ C, int64_t ldc,
    double *__restrict__ partial, int M_bound, int N, int K_bound, const int32_t *__restrict__ rows_dev, int m0, int n0,
    const int lane = (int)(threadIdx.x & 63))
{
    constexpr bool DW = MODE == MODE_DW, B_KMAJOR = MODE == MODE_DZ;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int grp = lane >> 4, l16 = lane & 15;
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

// Sixteen outputs that lie anywhere, summed in the order of product_tile: lane l gives the row (pa) and the column's offset in B (ob, bytes) of output l % 16, and its
// sum is the result in lane 16 (l % 4) + l (l < 16): of four small tiles (v_mfma_f64_4x4x4, which adds like the large one) the diagonals.
// CHUNKS of 32 k are on their way at once.
template <int MODE, int CHUNKS>
__device__ inline float product_at(const float *pa, const float *Bm, uint32_t ob, int64_t ldb, int K, int lane)
{
    const int grp = lane >> 4, l16 = lane & 15;
    const int64_t bs = MODE == MODE_DZ ? 4 : ldb * 4;   // bytes from one k to the next
    const uint32_t og = ob + (uint32_t)(8 * grp) * (uint32_t)bs;
    double acc = 0.0;
    auto step = [&](float a, float b) { acc = __builtin_amdgcn_mfma_f64_4x4x4f64((double)a, (double)b, acc, 0, 0, 0); };
    const int kt = K & ~31;
    struct Set {
        float a[8], b[8];
    };
    auto load = [&](Set &x, int c) {   // (beyond the last chunk that one again)
        c = c < kt ? c : kt - 32;
        const char *ca = (const char *)(pa + 8 * grp) + (int64_t)c * 4, *cb = (const char *)here(Bm) + c * here(bs);
        load_floats<4>(ca, 0, x.a);
        load_floats<4>(ca, 16, x.a + 4);
        if constexpr (MODE == MODE_DZ) {
            load_floats<4>(cb, og, x.b);
            load_floats<4>(cb + 16, og, x.b + 4);
        } else {
#pragma unroll
            for (int s = 0; s < 8; ++s, cb += bs) load_floats<1>(cb, og, &x.b[s]);
        }
    };
    Set x[CHUNKS];
    if (kt) {
#pragma unroll
        for (int u = 0; u < CHUNKS; ++u) load(x[u], 32 * u);
    }
    for (int k0 = kt; k0 < K; k0 += 4) {
        const int k = k0 + grp < K ? k0 + grp : K - 1;
        float a = pa[k], b;
        load_floats<1>((const char *)Bm, ob + (uint32_t)k * (uint32_t)bs, &b);
        step(k0 + grp < K ? a : 0.f, k0 + grp < K ? b : 0.f);
    }
#pragma unroll 1
    for (int c = 0; c < kt; c += 32 * CHUNKS) {
#pragma unroll
        for (int u = 0; u < CHUNKS; ++u) {
            if (c + 32 * u >= kt) break;
#pragma unroll
            for (int s = 0; s < 8; ++s) step(x[u].a[s], x[u].b[s]);
            load(x[u], c + 32 * (CHUNKS + u));
        }
    }
    return (float)acc;
}

}  // namespace csgs
