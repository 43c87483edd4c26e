// csgs_aggregate: Z = P~ sigma?(X)  (Section 3, Eq. 1 with the sampled operator P~).
//
// A wavefront takes a tile of output rows, resolves their edges into LDS, and its groups of G lanes (4 .. 64, spread over the
// features of a slice with V-element vector loads) stream through equal shares of them.  Products are accumulated in double,
// in ascending edge order, and rounded to float once: sampled rows carry 1/p_j discounts of 10^2..10^3, so near-cancelling
// outputs would lose the 1e-5 absolute tolerance with a float accumulator.  Bound by vector instructions where rows are
// many (a widening and a double add per element, the staging per slice, a row's end in most steps), by latency where they are
// few.  Rows with many kept edges (hubs) are taken by all wavefronts of the block that owns them, after its ordinary rows.
//
// Also here: csgs_gather_rows (staging of the sampled remote feature rows) and csgs_aggregate_grad
// (dH_prev = (P~^T dZ) .* [H_prev > 0]: the same kernel on a per-call transpose of P~).
#include "common.hpp"
#include "aggregate_tile.hpp"

namespace csgs {


// Block b of the grid: row block b / n_slices (four tiles of tr consecutive output rows, one per wavefront) and
// feature slice b % n_slices (G * V features).  The hardware deals consecutive blocks round-robin to the 8 XCDs, so with 2, 4
// or 8 slices all blocks of slice s run on XCDs s, s + n_slices, ...: such an XCD's L2 sees only slice s of the gathered
// table, a quarter of it for rows of 1 KB, and a row that several output rows refer to is fetched from memory less often.
template <typename T, int V, int G, bool RELU>
__global__ __launch_bounds__(AGG_BLOCK) void aggregate_k(const int32_t *__restrict__ adj_rowptr,
                                                         const int32_t *__restrict__ adj_col,
                                                         const float *__restrict__ adj_val, int32_t nS_bound,
                                                         const int32_t *__restrict__ nS_dev,
                                                         const int32_t *__restrict__ n_cols_p,
                                                         const T *__restrict__ Xl, int64_t ldl, int64_t rows_l,
                                                         const T *__restrict__ Xr, int64_t ldr, int64_t rows_r,
                                                         const int32_t *__restrict__ src_row, int32_t F,
                                                         float *__restrict__ Z, int64_t ldz,
                                                         const float *__restrict__ mask, int64_t ldm,
                                                         int32_t n_slices, int32_t tr, CompStride cs)
{
    __shared__ WaveStage<tile_rows(G)> stage[AGG_WAVES];
    __shared__ double heads[AGG_WAVES][WAVE * V], carries[AGG_WAVES][2 * G * V];
    const int32_t slice = (int32_t)(blockIdx.x % (unsigned)n_slices);
    const int64_t block_row0 = (int64_t)(blockIdx.x / (unsigned)n_slices) * (AGG_WAVES * tr);
    adj_rowptr = comp_ptr(adj_rowptr, cs.adj); adj_col = comp_ptr(adj_col, cs.adj); adj_val = comp_ptr(adj_val, cs.adj);
    nS_dev = comp_ptr(nS_dev, cs.adj); n_cols_p = comp_ptr(n_cols_p, cs.adj); src_row = comp_ptr(src_row, cs.adj);
    Xl = comp_ptr(Xl, cs.x); Xr = comp_ptr(Xr, cs.xr); Z = comp_ptr(Z, cs.out);
    // the two counts that may live on the device are asked for together; a count that is not given is read from a
    // stand-in address and dropped
    const int32_t nS_raw = *(nS_dev ? nS_dev : adj_rowptr);
    const int32_t n_cols_raw = *(n_cols_p ? n_cols_p : adj_rowptr);
    const int32_t nS = !nS_dev ? nS_bound : (nS_raw < 0 ? 0 : (nS_raw < nS_bound ? nS_raw : nS_bound));
    const int64_t n_cols = n_cols_p ? (int64_t)n_cols_raw : (src_row ? 0x7FFFFFFFll : rows_l);
    if (block_row0 >= nS) return;
    const int tid = (int)threadIdx.x;
    const int wave = tid >> 6;
    // V is at most F, and where F is no multiple of it the last V features of a row are taken together: those among them that
    // another lane (or slice) has too are written twice, the same.  Lanes past the row read the slice's start and store nothing
    const int32_t slice0 = slice * G * V < F - V ? slice * G * V : F - V;
    const int32_t lane_f = slice0 + (tid % G) * V;
    const int32_t f = lane_f < F - V ? lane_f : F - V;
    const bool active = lane_f < F;
    const bool is_long = aggregate_tile<T, V, G, RELU>(stage[wave], tr, heads[wave], carries[wave], block_row0 + (int64_t)wave * tr, 0, slice0, f,
                                                       active, adj_rowptr, adj_col, adj_val, nS_bound, nS, n_cols, Xl, ldl, rows_l,
                                                       Xr, ldr, rows_r, src_row, Z, ldz, mask, ldm);
    if (__syncthreads_or(is_long ? 1 : 0))
        aggregate_long_rows<T, V, G, RELU>(&heads[0][0], tr, block_row0, 0, is_long, slice0, f, active, adj_rowptr, adj_col, adj_val, n_cols, Xl, ldl,
                                           rows_l, Xr, ldr, rows_r, src_row, Z, ldz, mask, ldm);
}

template <typename T, int V, int G>
static int launch_agg(const int32_t *rp, const int32_t *col, const float *val, int32_t nS, const int32_t *nsd, const int32_t *ncp, const void *Xl,
                      int64_t ldl, int64_t rl, const void *Xr, int64_t ldr, int64_t rr, const int32_t *src_row, int32_t F, int relu, float *Z, int64_t ldz,
                      const float *mask, int64_t ldm, int kid, hipStream_t st, const CompInst &ci = CompInst{})
{
    const int64_t n_slices = (F + G * V - 1) / (G * V);
    // Rows per wavefront.  A full tile (8 rows per lane group) shares the cost of its set-up among the most rows, but a
    // launch for one mini-batch then has too few wavefronts: each walks through its tile's edges alone.  Tiles are
    // halved until the launch has 512 blocks, two per compute unit (us per launch, full / this rule, one mini-batch:
    // 2048 rows of 27 edges, F = 256, 81 / 24; 8192 x 2.8, F = 256, 21 / 17; 4096 x 1.6, F = 512, 13 / 9; 256 x 2,
    // F = 64, 12 / 7).  Not further: at 1024 blocks the set-up dominates (8192 x 2.8: 22; 4096 x 1.6: 13), as it does
    // with less than half a row per lane group (1024 x 2.2, F = 256: 4 rows per wavefront 8.6, 8 rows 7.6).
    int tr = tile_rows(G);
    constexpr int tr_min = WAVE / G / 2 > 2 ? WAVE / G / 2 : 2;
    auto blocks_of = [&](int r) { return ((int64_t)nS + AGG_WAVES * r - 1) / (AGG_WAVES * r); };
    while (tr > tr_min && blocks_of(tr) * n_slices * ci.n < 512) tr >>= 1;
    const int64_t row_blocks = blocks_of(tr);
    if (row_blocks * n_slices > 0x7FFFFFFFll) return CSGS_EUNSUPPORTED;
    const dim3 grid((unsigned)(row_blocks * n_slices), 1, (unsigned)ci.n);
#define CSGS_AGG_LAUNCH(RELU)                                                                                                     \
    CSGS_LAUNCH_ID(kid, (aggregate_k<T, V, G, RELU>), grid, dim3(AGG_BLOCK), st, rp, col, val, nS, nsd, ncp, (const T *)Xl, ldl, rl, \
                   (const T *)Xr, ldr, rr, src_row, F, Z, ldz, mask, ldm, (int32_t)n_slices, (int32_t)tr, ci.cs)
    if (relu) CSGS_AGG_LAUNCH(true); else CSGS_AGG_LAUNCH(false);
#undef CSGS_AGG_LAUNCH
    CSGS_LAUNCH_CHECK();
    return CSGS_OK;
}

// Lanes per row and slice.  Rows of 1 KB and more are cut into (about) four slices; shorter rows are taken whole by the
// smallest group of lanes that covers them.  Eight slices, one per XCD, keep more of the table in the L2s but stage every edge
// eight times and end a row every few steps, and the kernel is bound by vector instructions where rows are many (us, eight /
// four / two slices, F = 256: 83 K rows of 21 kept edges 228 / 200 / 207, 131 K of 22 353 / 305 / 321, 2048 of 26 22 / 19 /
// 18, 7.3 K of 2.9 17 / 14 / 16, eight of those 51 / 53 / 51).
template <typename T, int V>
static int pick_group(const int32_t *rp, const int32_t *col, const float *val, int32_t nS, const int32_t *nsd, const int32_t *ncp, const void *Xl,
                      int64_t ldl, int64_t rl, const void *Xr, int64_t ldr, int64_t rr, const int32_t *src_row, int32_t F, int relu, float *Z, int64_t ldz,
                      const float *mask, int64_t ldm, int kid, hipStream_t st, const CompInst &ci = CompInst{})
{
    const int64_t vecs = (F + V - 1) / V;
    const int64_t want = (int64_t)F * (int64_t)sizeof(T) >= 1024 ? (vecs + 3) / 4 : vecs;
#define CSGS_AGG_G(GG) launch_agg<T, V, GG>(rp, col, val, nS, nsd, ncp, Xl, ldl, rl, Xr, ldr, rr, src_row, F, relu, Z, ldz, mask, ldm, kid, st, ci)
    if (want <= 4) return CSGS_AGG_G(4);
    if (want <= 8) return CSGS_AGG_G(8);
    if (want <= 16) return CSGS_AGG_G(16);
    if (want <= 32) return CSGS_AGG_G(32);
    return CSGS_AGG_G(64);
#undef CSGS_AGG_G
}

// Tables whose rows start anywhere, or whose rows are no whole number of four-element pieces: the same wide loads, which take any
// address, the last V features of a row together (they overlap the lane's before).  A piece then lies across two cache lines more
// often and a slice's edge in the middle of one, so slices are fewer and wider here, of 256 features (us, an element or a pair per lane
// and four slices / this: 2048 rows of 27 edges, F = 602, 36 / 25; 20000 of 6, F = 481, 54 / 47, bf16 56 / 37, F = 201 31 / 24; 3000 of 8,
// F = 333, 19 / 14, bf16 18 / 15; 68536 of 4.5, F = 481, 146 / 111).  Up to 128 features by how many rows there are:
//  * 65 .. 128: many rows are taken whole (two slices / one: 131 K rows of 13, F = 65, 129 / 95, F = 127 176 / 157), from ODD_WIDE_ROWS on by
//    16 lanes with eight features each (3000 rows of 0.6 edges, F = 82, 7.0 / 6.2, of 27, F = 127, 9.5 / 9.0; 777 rows of 100, F = 127, 12.2 / 13.4).
//  * 33 .. 64: 16 lanes with four each.  What rows of an edge or two pay for the share of a row that every group may hold (777 rows of 0.6,
//    F = 63, an element per lane 5.2, this 5.9; 3000, 5.5 / 6.4) longer ones get back (777 of 27, F = 65, 10.2 / 7.6, of 100, F = 63, 21.6 / 12.0).
//  * 17 .. 32: 16 lanes with a pair each (32 with an element / eight with four / this: 100 rows of 100, F = 17, 14.0 / 14.8 / 10.1; 2048 of 27,
//    F = 31, 8.5 / 8.3 / 7.1), beyond ODD_GROUPS_FROM rows, which fill the device with fewer lanes each, eight with four (20000 of 27, F = 31, 20.6 / 15.1 / 15.9).
//  * 9 .. 16, between ODD_GROUPS_FROM and ODD_GROUPS_TO rows: eight lanes with a pair (16 with an element / this: 60000 of 27, F = 15, 27.9 / 24.5).
// The others keep an element per lane, or a pair where rows begin on one and hold whole pairs:
//  * fewer features: four lanes with four each let a tile be twice as many rows that a wavefront walks through alone (100 rows of 100,
//    F = 15, 9.9 / 23.4; 2048 of 100, F = 5, 14.1 / 23.8; 12000 of 27, F = 5, 8.8 / 11.7; 131072 of 13, F = 15, 41 / 45);
//  * float rows of 257 to 320 features in pairs, where a second slice of 256 is nearly empty, if they are many (pairs / two slices: F = 258, 8192 rows of
//    27, 37.9 / 44.3, of 0.6, F = 270, 9.2 / 9.8; 60000 of 13, F = 262, 156 / 189; 2048 of 100, F = 258, 35.8 / 29.7);
//  * a handful of rows, a row per wavefront, which has no shares to put together (16 rows of 3, F = 31, 4.9 / 5.4, F = 63 4.9 / 5.2; 64 of
//    3 5.3 / 5.6, 5.1 / 5.5).
constexpr int32_t ODD_FEW_ROWS = 64, ODD_WIDE_ROWS = 1024, ODD_WHOLE_ROWS = 4096, ODD_GROUPS_FROM = 8192, ODD_GROUPS_TO = 65536, ODD_PAIRS = 320;
template <typename T>
static int pick_odd(const int32_t *rp, const int32_t *col, const float *val, int32_t nS, const int32_t *nsd, const int32_t *ncp, const void *Xl,
                    int64_t ldl, int64_t rl, const void *Xr, int64_t ldr, int64_t rr, const int32_t *src_row, int32_t F, int relu, float *Z, int64_t ldz,
                    const float *mask, int64_t ldm, int kid, hipStream_t st, const CompInst &ci)
{
#define CSGS_AGG_VG(V, G) launch_agg<T, V, G>(rp, col, val, nS, nsd, ncp, Xl, ldl, rl, Xr, ldr, rr, src_row, F, relu, Z, ldz, mask, ldm, kid, st, ci)
    const int64_t rows = (int64_t)nS * ci.n;
    if (F > 128) return CSGS_AGG_VG(8, 32);
    if (F > 64 && rows > ODD_WHOLE_ROWS) return CSGS_AGG_VG(4, 32);
    if (F > 64 && rows > ODD_WIDE_ROWS) return CSGS_AGG_VG(8, 16);
    if (F > 32) return CSGS_AGG_VG(4, 16);
    if (F > 16) return rows > ODD_GROUPS_FROM ? CSGS_AGG_VG(4, 8) : CSGS_AGG_VG(2, 16);
    return CSGS_AGG_VG(2, 8);
#undef CSGS_AGG_VG
}

template <typename T>
static int pick_vec(const int32_t *rp, const int32_t *col, const float *val, int32_t nS, const int32_t *nsd, const int32_t *ncp, const void *Xl,
                    int64_t ldl, int64_t rl, const void *Xr, int64_t ldr, int64_t rr, const int32_t *src_row, int32_t F, int relu, float *Z, int64_t ldz,
                    const float *mask, int64_t ldm, int kid, hipStream_t st, const CompInst &ci = CompInst{})
{
    // rows of whole pieces that every row starts on a multiple of (8 floats are read as two pieces of 4)
    auto whole = [&](int v) {
        const int piece = (v == 8 && sizeof(T) == 4) ? 4 : v;
        const uintptr_t bytes = (uintptr_t)piece * sizeof(T);
        const int zpiece = v == 8 ? 4 : v;
        return F % v == 0 && (!Xl || (ldl % piece == 0 && ((uintptr_t)Xl % bytes) == 0)) &&
               (!Xr || (ldr % piece == 0 && ((uintptr_t)Xr % bytes) == 0)) && ldz % zpiece == 0 &&
               ((uintptr_t)Z % ((uintptr_t)zpiece * sizeof(float))) == 0;
    };
    if (whole(8)) return pick_group<T, 8>(rp, col, val, nS, nsd, ncp, Xl, ldl, rl, Xr, ldr, rr, src_row, F, relu, Z, ldz, mask, ldm, kid, st, ci);
    if (whole(4)) return pick_group<T, 4>(rp, col, val, nS, nsd, ncp, Xl, ldl, rl, Xr, ldr, rr, src_row, F, relu, Z, ldz, mask, ldm, kid, st, ci);
    const int64_t rows = (int64_t)nS * ci.n;
    const bool narrow = F <= 8 || (F <= 16 && (rows <= ODD_GROUPS_FROM || rows > ODD_GROUPS_TO));
    const bool pairs = sizeof(T) == 4 && F > 256 && F <= ODD_PAIRS && rows > ODD_WHOLE_ROWS && whole(2);
    if (narrow || pairs || rows <= ODD_FEW_ROWS) {
        if (whole(2)) return pick_group<T, 2>(rp, col, val, nS, nsd, ncp, Xl, ldl, rl, Xr, ldr, rr, src_row, F, relu, Z, ldz, mask, ldm, kid, st, ci);
        return pick_group<T, 1>(rp, col, val, nS, nsd, ncp, Xl, ldl, rl, Xr, ldr, rr, src_row, F, relu, Z, ldz, mask, ldm, kid, st, ci);
    }
    return pick_odd<T>(rp, col, val, nS, nsd, ncp, Xl, ldl, rl, Xr, ldr, rr, src_row, F, relu, Z, ldz, mask, ldm, kid, st, ci);
}

// ------------------------------------------------------------------ gradient of the aggregation
// dH_prev = (P~^T dZ) .* [H_prev > 0].  P~ is held by rows; its transpose is built per call in the
// caller's scratch: entries per column counted with integer atomics, a prefix sum turns the
// counts into column offsets, a second pass drops every entry into its column in arrival order,
// and a third puts each column's entries into ascending row order (ranks by counting inside a
// wavefront for columns of up to 64 entries, through a bitmap over the rows in LDS for longer ones).
// Then the forward kernel runs on the transposed structure with dZ as the gathered table and the
// ReLU derivative as an output mask.  Every column is summed in ascending row order, in double, with
// one rounding: the result does not depend on timing.

// one wavefront per row of P~: counts[c] += 1 for every entry of the row
__global__ __launch_bounds__(256) void adjT_count(const int32_t *__restrict__ adj_rowptr,
                                                  const int32_t *__restrict__ adj_col, int32_t nS_bound,
                                                  const int32_t *__restrict__ nS_dev, int32_t n_cols_bound,
                                                  const int32_t *__restrict__ n_cols_dev, int64_t cap,
                                                  int32_t *__restrict__ counts)
{
    const int32_t nS = resolve_count(nS_bound, nS_dev), n_cols = resolve_count(n_cols_bound, n_cols_dev);
    const int lane = lane_id();
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t n_waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t r = wave; r < nS; r += n_waves) {
        const int32_t beg = adj_rowptr[r] < 0 ? 0 : adj_rowptr[r];
        const int32_t end = adj_rowptr[r + 1] < cap ? adj_rowptr[r + 1] : (int32_t)cap;   // stay inside adj_col whatever the pointers say
        for (int32_t e = beg + lane; e < end; e += WAVE) {
            const int32_t c = adj_col[e];
            if (c >= 0 && c < n_cols) atomicAdd(&counts[c], 1);
        }
    }
}

// colptr = exclusive prefix of counts.  A block takes `rounds` times PREFIX_COLS columns and adds up all counts before them
// itself (4 bytes per column, from the L2s): nobody waits, and 4 K columns are two blocks instead of one that goes round by 8192
// (7.2 -> 4.2 us; 131 K columns 167 -> 18).  Blocks re-read what lies before them, so there are PREFIX_GRID of them at most and
// each takes several rounds (64 M columns, one block / a block per 2048 columns / this: 88 / 551 / 13 ms).
constexpr int PREFIX_COLS = 2048;
constexpr int64_t PREFIX_GRID = 512;
__global__ __launch_bounds__(256) void adjT_prefix(const int32_t *__restrict__ counts, int32_t n_cols_bound,
                                                   const int32_t *__restrict__ n_cols_dev, int32_t *__restrict__ colptr, int32_t rounds)
{
    __shared__ int32_t lds[17];
    __shared__ int32_t s_before[4];
    const int32_t n_cols = resolve_count(n_cols_bound, n_cols_dev);
    const int tid = (int)threadIdx.x;
    const int64_t first = (int64_t)blockIdx.x * rounds * PREFIX_COLS;
    if (first >= n_cols) {
        if (first == 0 && tid == 0) colptr[0] = 0;
        return;
    }
    int32_t sum_before = 0;
    {
        const int4 *__restrict__ c4 = reinterpret_cast<const int4 *>(counts);
        const int64_t n4 = first / 4;
        int64_t i = tid;
        for (; i + 3 * 256 < n4; i += 4 * 256) {   // four loads on their way at a time
            const int4 p = c4[i], q = c4[i + 256], r = c4[i + 512], t = c4[i + 768];
            sum_before += (p.x + p.y + p.z + p.w) + (q.x + q.y + q.z + q.w) + (r.x + r.y + r.z + r.w) + (t.x + t.y + t.z + t.w);
        }
        for (; i < n4; i += 256) {
            const int4 p = c4[i];
            sum_before += p.x + p.y + p.z + p.w;
        }
    }
    sum_before = wave_sum(sum_before);
    if ((tid & (WAVE - 1)) == 0) s_before[tid >> 6] = sum_before;
    int32_t base = 0;   // of the round's first column
    for (int32_t round = 0; round < rounds; ++round) {
        const int64_t c0 = first + (int64_t)round * PREFIX_COLS + tid * 8;
        if (c0 - tid * 8 >= n_cols) break;   // the whole block
        int32_t v[8], sum = 0;
        if (c0 + 8 <= n_cols) {
            const int4 p = *reinterpret_cast<const int4 *>(counts + c0), q = *reinterpret_cast<const int4 *>(counts + c0 + 4);
            v[0] = p.x; v[1] = p.y; v[2] = p.z; v[3] = p.w;
            v[4] = q.x; v[5] = q.y; v[6] = q.z; v[7] = q.w;
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = c0 + k < n_cols ? counts[c0 + k] : 0;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) sum += v[k];
        int32_t total;
        int32_t ex = block_exclusive_scan<int32_t>(sum, lds, &total);   // (its barriers are behind the stores of s_before)
        if (round == 0) base = s_before[0] + s_before[1] + s_before[2] + s_before[3];
        ex += base;
        base += total;
        if (c0 + 8 <= n_cols) {
            int32_t o[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) { o[k] = ex; ex += v[k]; }
            *reinterpret_cast<int4 *>(colptr + c0) = make_int4(o[0], o[1], o[2], o[3]);
            *reinterpret_cast<int4 *>(colptr + c0 + 4) = make_int4(o[4], o[5], o[6], o[7]);
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (c0 + k < n_cols) colptr[c0 + k] = ex;
                ex += v[k];
            }
        }
        if (c0 < n_cols && c0 + 8 >= n_cols) colptr[n_cols] = ex;   // the thread of the last column
    }
}

// one wavefront per row of P~: entry (r, c, v) goes to slot colptr[c] + --left[c] of the unordered list
// (left: the counts, which nobody needs any more)
__global__ __launch_bounds__(256) void adjT_fill(const int32_t *__restrict__ adj_rowptr,
                                                 const int32_t *__restrict__ adj_col, const float *__restrict__ adj_val,
                                                 int32_t nS_bound, const int32_t *__restrict__ nS_dev,
                                                 int32_t n_cols_bound, const int32_t *__restrict__ n_cols_dev,
                                                 const int32_t *__restrict__ colptr, int32_t *__restrict__ left,
                                                 uint2 *__restrict__ unordered, int64_t cap)
{
    const int32_t nS = resolve_count(nS_bound, nS_dev), n_cols = resolve_count(n_cols_bound, n_cols_dev);
    const int lane = lane_id();
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t n_waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t r = wave; r < nS; r += n_waves) {
        const int32_t beg = adj_rowptr[r] < 0 ? 0 : adj_rowptr[r];
        const int32_t end = adj_rowptr[r + 1] < cap ? adj_rowptr[r + 1] : (int32_t)cap;
        for (int32_t e = beg + lane; e < end; e += WAVE) {
            const int32_t c = adj_col[e];
            if (c >= 0 && c < n_cols) {
                const int64_t slot = (int64_t)colptr[c] + atomicSub(&left[c], 1) - 1;
                if (slot >= 0 && slot < cap) unordered[slot] = make_uint2((uint32_t)r, __float_as_uint(adj_val[e]));
            }
        }
    }
}

// Puts the entries of every column into ascending row order: (row, value) from the unordered list into
// rowT / valT.  A block owns ORD_COLS consecutive columns.  Columns of up to 64 entries are taken by one
// wavefront each, an entry's place being the number of entries of its column with a smaller row (rows are
// distinct inside a column).  Longer columns (hubs among the sampled nodes) are then taken by the whole
// block one at a time: the rows present are marked in a bitmap in LDS, ORD_TILE_ROWS rows at a time, and an
// entry's place is the number of marked rows below its own.
constexpr int ORD_COLS = 16, ORD_PER_WAVE = ORD_COLS / AGG_WAVES;
constexpr int ORD_TILE_ROWS = 65536;
constexpr int ORD_TILE_WORDS = ORD_TILE_ROWS / 32;

__global__ __launch_bounds__(256) void adjT_order(const int32_t *__restrict__ colptr, int32_t n_cols_bound,
                                                  const int32_t *__restrict__ n_cols_dev, int32_t nS_bound,
                                                  const int32_t *__restrict__ nS_dev, const uint2 *__restrict__ unordered,
                                                  int32_t *__restrict__ rowT, float *__restrict__ valT, int64_t cap)
{
    __shared__ uint32_t bm[ORD_TILE_WORDS];
    __shared__ int32_t below[ORD_TILE_WORDS];   // marked rows in the words before this one
    __shared__ int32_t long_cols[ORD_COLS];
    __shared__ int32_t n_long;
    __shared__ int32_t scan_lds[17];
    const int32_t n_cols = resolve_count(n_cols_bound, n_cols_dev), nS = resolve_count(nS_bound, nS_dev);
    const int tid = (int)threadIdx.x, lane = tid & (WAVE - 1), wave = tid >> 6;
    if (tid == 0) n_long = 0;
    __syncthreads();
    auto extent = [&](int32_t c, int32_t *beg, int32_t *end) {   // stays inside the lists whatever the offsets say
        const int32_t b = colptr[c], e = colptr[c + 1];
        *beg = b < 0 ? 0 : b;
        *end = e < cap ? e : (int32_t)cap;
    };
    {   // the extents of the wavefront's columns in one load, then their entries together
        const int64_t col0 = (int64_t)blockIdx.x * ORD_COLS + wave * ORD_PER_WAVE;
        const int64_t at = col0 + lane < n_cols ? col0 + lane : n_cols;
        const int32_t edge = (lane <= ORD_PER_WAVE && col0 < n_cols) ? colptr[at] : 0;
        int32_t beg[ORD_PER_WAVE], len[ORD_PER_WAVE];
        uint2 v[ORD_PER_WAVE];
#pragma unroll
        for (int k = 0; k < ORD_PER_WAVE; ++k) {
            const int32_t b = __builtin_amdgcn_readlane(edge, k), e = __builtin_amdgcn_readlane(edge, k + 1);
            beg[k] = b < 0 ? 0 : b;                                        // stays inside the lists whatever the offsets say
            len[k] = (e < cap ? e : (int32_t)cap) - beg[k];                // (a column past the last one is empty)
            if (len[k] > WAVE) {
                if (lane == 0) long_cols[atomicAdd(&n_long, 1)] = (int32_t)(col0 + k);   // in any order: the columns do not meet
                len[k] = 0;
            }
        }
#pragma unroll
        for (int k = 0; k < ORD_PER_WAVE; ++k) v[k] = lane < len[k] ? unordered[beg[k] + lane] : make_uint2(0xFFFFFFFFu, 0u);
#pragma unroll
        for (int k = 0; k < ORD_PER_WAVE; ++k) {
            int32_t place = 0;
            for (int32_t j = 0; j < len[k]; ++j) place += (uint32_t)__builtin_amdgcn_readlane((int)v[k].x, j) < v[k].x ? 1 : 0;
            if (lane < len[k]) {
                rowT[beg[k] + place] = (int32_t)v[k].x;
                valT[beg[k] + place] = __uint_as_float(v[k].y);
            }
        }
    }
    __syncthreads();
    const int32_t cnt = n_long;
    for (int32_t li = 0; li < cnt; ++li) {
        int32_t beg, end;
        extent(long_cols[li], &beg, &end);
        int32_t base = 0;   // entries of this column with rows below the tile
        for (int64_t lo = 0; lo < nS; lo += ORD_TILE_ROWS) {
            const int32_t words = (int32_t)((nS - lo + 31) / 32 < ORD_TILE_WORDS ? (nS - lo + 31) / 32 : ORD_TILE_WORDS);
            for (int32_t w = tid; w < words; w += AGG_BLOCK) bm[w] = 0u;
            __syncthreads();
            for (int32_t e = beg + tid; e < end; e += AGG_BLOCK) {
                const int64_t d = (int64_t)unordered[e].x - lo;
                if (d >= 0 && d < (int64_t)words * 32) atomicOr(&bm[d >> 5], 1u << (d & 31));
            }
            __syncthreads();
            int32_t pc[ORD_TILE_WORDS / AGG_BLOCK], sum = 0;
#pragma unroll
            for (int k = 0; k < ORD_TILE_WORDS / AGG_BLOCK; ++k) {
                const int32_t w = tid * (ORD_TILE_WORDS / AGG_BLOCK) + k;
                pc[k] = w < words ? __popc(bm[w]) : 0;
                sum += pc[k];
            }
            int32_t total;
            int32_t ex = block_exclusive_scan<int32_t>(sum, scan_lds, &total);
#pragma unroll
            for (int k = 0; k < ORD_TILE_WORDS / AGG_BLOCK; ++k) {
                below[tid * (ORD_TILE_WORDS / AGG_BLOCK) + k] = ex;
                ex += pc[k];
            }
            __syncthreads();
            for (int32_t e = beg + tid; e < end; e += AGG_BLOCK) {
                const uint2 v = unordered[e];
                const int64_t d = (int64_t)v.x - lo;
                if (d >= 0 && d < (int64_t)words * 32) {
                    const int32_t place = base + below[d >> 5] + __popc(bm[d >> 5] & ((1u << (d & 31)) - 1u));
                    if (place < end - beg) {
                        rowT[beg + place] = (int32_t)v.x;
                        valT[beg + place] = __uint_as_float(v.y);
                    }
                }
            }
            base += total;
            __syncthreads();   // the bitmap is cleared for the next tile or column
        }
    }
}

// The same in one launch for few entries: a block owns consecutive columns and looks at the columns of all entries itself (4 bytes each, from the
// L2s), so that nothing has to be cleared, counted with atomics or waited for between launches.  Its wavefronts take consecutive shares of the
// entries (ascending entries have ascending rows): each counts those of the block's columns by column and lists them in LDS, in order, so that after
// one prefix over columns and wavefronts an entry's place is the next one of its wavefront and column -- linear in the entries, however
// long a column is.  Wavefronts of a block whose lists outgrow LDS read their shares again.  An entry's row is searched for in the row pointers.
// Bound by latency up to 20 K entries, from 100 K on by the instructions that look at every entry in every block.  (us of csgs_aggregate_grad with 8
// features, several launches / this: 2 K entries of 8192 columns 22 / 13.5, 20 K 22 / 15.5, 131 K 36.6 / 32; 20 K and a column of 257
// 31 / 19, of 2049 79 / 33, of 8192 248 / 67, of 60 K 1704 / 423; comparing the entries of a column with each other for their places made those
// 23, 107, 391 and 6740.)
constexpr int ONE_BLOCK = 1024, ONE_WAVES = ONE_BLOCK / WAVE, ONE_GRID = 256;
constexpr int ONE_CHUNKS = 192;   // pieces of 64 entries that LDS holds; a wavefront chains as many as it needs
constexpr int32_t ONE_COLS = 65536;   // most columns
constexpr int ONE_OWN = ONE_COLS / ONE_GRID;
// Most entries, as the caller bounds them (the spare room of its arrays costs nothing).  With arrays that are full (us as above): 262 K entries of 256 columns
// 684 / 159, of 8192 54.7 / 53.5, of 65536 59.6 / 51.3; 520 K 1299 / 287, 104 / 97 and 88.5 / 96; 1.04 M 2107 / 483, 160 / 181, 148 / 180.  More columns
// than ONE_WIDE hold few entries each, which the several launches order well.
constexpr int64_t ONE_ENTRIES = 1ll << 19, ONE_ENTRIES_WIDE = 3ll << 17;
constexpr int32_t ONE_WIDE = 8192;
static_assert(ONE_OWN == 256 && ONE_ENTRIES <= 1 << 24, "an entry and its column in 32 bits");

// The row of an entry: last r with adj_rowptr[r] <= e, by eighths (the loads of a round together).  nS > 0.
__device__ inline int32_t entry_row(const int32_t *__restrict__ adj_rowptr, int32_t nS, int32_t e)
{
    int32_t lo = 0, hi = nS;   // adj_rowptr[lo] <= e < adj_rowptr[hi]
    while (hi - lo > 1) {
        const int32_t span = hi - lo;
        int32_t p[7];
#pragma unroll
        for (int k = 0; k < 7; ++k) p[k] = adj_rowptr[lo + (int32_t)((int64_t)span * (k + 1) / 8)];
        int below = 0;
#pragma unroll
        for (int k = 0; k < 7; ++k) below += p[k] <= e ? 1 : 0;
        const int32_t new_lo = lo + (int32_t)((int64_t)span * below / 8);
        hi = below < 7 ? lo + (int32_t)((int64_t)span * (below + 1) / 8) : hi;
        lo = new_lo;
    }
    return lo;
}

__global__ __launch_bounds__(ONE_BLOCK) void adjT_one(const int32_t *__restrict__ adj_rowptr, const int32_t *__restrict__ adj_col,
                                                      const float *__restrict__ adj_val, int32_t nS_bound, const int32_t *__restrict__ nS_dev,
                                                      int32_t n_cols_bound, const int32_t *__restrict__ n_cols_dev, int64_t cap,
                                                      int32_t *__restrict__ colptr, int32_t *__restrict__ rowT, float *__restrict__ valT)
{
    constexpr int U = 8;                                 // entries on their way per lane
    __shared__ uint32_t l_e[ONE_CHUNKS * WAVE];          // an entry (from the first one) << 8 | its column (from the block's first)
    __shared__ uint16_t l_next[ONE_CHUNKS];              // the wavefront's piece after this one
    __shared__ int32_t l_s[ONE_CHUNKS * WAVE];           // the entries in their places
    __shared__ int32_t at[ONE_WAVES][ONE_OWN];           // entries of a wavefront's share by column, then their next place
    __shared__ int32_t n_pieces, s_before[ONE_WAVES], s_own[ONE_OWN / WAVE];   // of entries: before the block's columns, by wavefront; in 64 of them
    const int32_t nS = resolve_count(nS_bound, nS_dev), n_cols = resolve_count(n_cols_bound, n_cols_dev);
    const int tid = (int)threadIdx.x, lane = tid & (WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t own = (n_cols + ONE_GRID - 1) / ONE_GRID;   // at most ONE_OWN
    const int32_t c0 = (int32_t)blockIdx.x * own, c1 = c0 + own < n_cols ? c0 + own : n_cols;
    if (c0 >= n_cols) {
        if (n_cols == 0 && blockIdx.x == 0 && tid == 0) colptr[0] = 0;
        return;
    }
    // entries of the rows (inside the arrays whatever the pointers say)
    int32_t e_beg = nS > 0 ? adj_rowptr[0] : 0, e_end = nS > 0 ? adj_rowptr[nS] : 0;
    if (e_beg < 0) e_beg = 0;
    if (e_end > cap) e_end = (int32_t)cap;
    if (e_end < e_beg) e_end = e_beg;
    for (int i = tid; i < ONE_WAVES * ONE_OWN; i += ONE_BLOCK) (&at[0][0])[i] = 0;
    if (tid == 0) n_pieces = ONE_WAVES;   // a wavefront's first piece is its own
    __syncthreads();
    // the wavefront's share (blocks begin at different ones, so that they don't ask the same pieces of an L2 for the same lines at once)
    const int part = (wave + (int)blockIdx.x) % ONE_WAVES;
    const int32_t share = (e_end - e_beg + ONE_BLOCK - 1) / ONE_BLOCK * WAVE;
    const int32_t w0 = e_beg + part * share < e_end ? e_beg + part * share : e_end, w1 = w0 + share < e_end ? w0 + share : e_end;
    const uint64_t lanes_below = (1ull << lane) - 1ull;
    const uint32_t n_mine = (uint32_t)(c1 - c0);
    int32_t before = 0, n_listed = 0, piece = part, used = 0;   // entries of columns before the block's (lane by lane); of its own, listed
    bool listed = true;
    int32_t c[U], next_c[U];
    auto wide = [&](int32_t e) {   // (entries start anywhere)
#pragma unroll
        for (int u = 0; u < U; u += 4) {
            const u32x4 v = load_global<u32x4, 4>(adj_col + e + u);
            next_c[u] = (int32_t)v.x; next_c[u + 1] = (int32_t)v.y; next_c[u + 2] = (int32_t)v.z; next_c[u + 3] = (int32_t)v.w;
        }
    };
    for (int32_t from = w0;; from += U * WAVE) {   // asks for the entries from here on, looks at the ones before; a lane's U lie side by side
        const int32_t e = from + lane * U;
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = next_c[u];
        if (from + U * WAVE <= w1) {
            wide(e);
        } else if (from < w1) {
#pragma unroll
            for (int u = 0; u < U; ++u) next_c[u] = -1;   // (a negative column is nobody's)
            if (e + U <= w1) wide(e);
            else
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (e + u < w1) next_c[u] = adj_col[e + u];
        }
        if (from > w0) {
            uint32_t mine = 0;   // which of the lane's entries are of the block's columns
#pragma unroll
            for (int u = 0; u < U; ++u) {
                before += (uint32_t)c[u] < (uint32_t)c0 ? 1 : 0;
                mine |= (uint32_t)(c[u] - c0) < n_mine ? 1u << u : 0u;
            }
            if (__any(mine)) {
                const int32_t n = __popc(mine), incl = wave_inclusive_scan<int32_t>(n), total = __builtin_amdgcn_readlane(incl, WAVE - 1);
                const int32_t fresh = (used + total - 1) / WAVE;   // pieces begun
                int32_t next = piece, i = used + incl - n;
                if (listed && fresh) {
                    if (lane == 0) next = atomicAdd(&n_pieces, fresh);
                    next = __builtin_amdgcn_readfirstlane(next);
                    listed = next + fresh <= ONE_CHUNKS;
                    if (listed && lane < fresh) l_next[lane ? next + lane - 1 : piece] = (uint16_t)(next + lane);
                }
                for (uint32_t m = mine; m; m &= m - 1u, ++i) {
                    const int u = __ffs((int)m) - 1;
                    int32_t d = c[0];
#pragma unroll
                    for (int k = 1; k < U; ++k) d = u == k ? c[k] : d;
                    d -= c0;
                    atomicAdd(&at[part][d], 1);
                    if (listed) l_e[i < WAVE ? piece * WAVE + i : next * WAVE + i - WAVE] = (uint32_t)(e - U * WAVE + u - e_beg) << 8 | (uint32_t)d;
                }
                used += total - fresh * WAVE;
                piece = fresh ? next + fresh - 1 : piece;
                n_listed += total;
            }
        }
        if (from >= w1) break;
    }
    before = wave_sum(before);
    if (lane == 0) s_before[wave] = before;
    __syncthreads();
    // a thread per column: where it begins, and each share's entries of it
    int32_t n_col[ONE_WAVES], sum = 0, end = 0;
    if (tid < ONE_OWN) {
#pragma unroll
        for (int w = 0; w < ONE_WAVES; ++w) {
            n_col[w] = at[w][tid];
            sum += n_col[w];
        }
        end = wave_inclusive_scan<int32_t>(sum);
        if (lane == WAVE - 1) s_own[wave] = end;
    }
    __syncthreads();
    const int32_t base = wave_sum(lane < ONE_WAVES ? s_before[lane] : 0), n_own = wave_sum(lane < ONE_OWN / WAVE ? s_own[lane] : 0);
    if (tid < ONE_OWN) {
        end += base + wave_sum(lane < wave ? s_own[lane] : 0);
        int32_t place = end - sum;
        if (tid < c1 - c0) colptr[c0 + tid] = place;
        if (tid == c1 - c0 - 1 && c1 == n_cols) colptr[n_cols] = end;
#pragma unroll
        for (int w = 0; w < ONE_WAVES; ++w) {
            at[w][tid] = place;
            place += n_col[w];
        }
    }
    __syncthreads();
    // places of a wavefront's next 64 entries (lanes that `have` one), in order: lanes of the same column find each other bit by bit
    const int bits = own > 1 ? 32 - __clz(own - 1) : 0;
    auto place = [&](bool have, int32_t d) {
        uint64_t same = __ballot(have);
        for (int b = 0; b < bits; ++b) {
            const uint64_t set = __ballot((d >> b) & 1);
            same &= (d >> b) & 1 ? set : ~set;
        }
        const int32_t rank = __popcll(same & lanes_below);
        int32_t p = 0;
        if (have && rank == 0) p = atomicAdd(&at[part][d], __popcll(same));
        __builtin_amdgcn_wave_barrier();   // (the wavefront's next 64 come after these)
        return __shfl(p, have ? __ffsll((long long)same) - 1 : lane, WAVE) + rank;
    };
    auto put = [&](int32_t p, int32_t row, float v) {
        if (p < cap) {
            rowT[p] = row;
            valT[p] = v;
        }
    };
    if (n_pieces <= ONE_CHUNKS) {   // (so all wavefronts have listed theirs)
        for (int32_t left = n_listed, piece = part; left > 0; left -= WAVE) {
            const bool have = lane < left;
            const uint32_t v = have ? l_e[piece * WAVE + lane] : 0u;
            if (left > WAVE) piece = l_next[piece];
            const int32_t p = place(have, (int32_t)(v & 255u)) - base;
            if (have) l_s[p] = e_beg + (int32_t)(v >> 8);   // p < n_own <= listed entries
        }
        __syncthreads();
        // a thread per place (few threads search where there are few entries)
        for (int32_t i = tid; i < n_own; i += ONE_BLOCK) {
            const int32_t e = l_s[i];
            const float v = adj_val[e];
            put(base + i, entry_row(adj_rowptr, nS, e), v);
        }
        return;
    }
    for (int32_t e0 = w0; e0 < w1; e0 += WAVE) {
        const int32_t e = e0 + lane < w1 ? e0 + lane : w1 - 1, d = adj_col[e] - c0;
        const bool have = e0 + lane < w1 && (uint32_t)d < n_mine;
        if (!__any(have)) continue;
        const float v = adj_val[e];
        const int32_t p = place(have, d);
        if (have) put(p, entry_row(adj_rowptr, nS, e), v);
    }
}

__global__ void fill_zero_i32(int32_t *p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = 0;
}

struct GradScratch {
    int32_t *counts, *colptr, *rowT;
    float *valT;
    uint2 *unordered;   // (row, value bits) of every entry, grouped by column, in arrival order inside a column
    size_t bytes;
};

__host__ inline GradScratch carve_grad(void *base, int32_t n_cols_cap, int64_t adj_cap)
{
    GradScratch g;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = align_up(off + bytes, 256);
        return (char *)base + o;
    };
    g.counts = (int32_t *)take((size_t)n_cols_cap * 4);
    g.colptr = (int32_t *)take(((size_t)n_cols_cap + 1) * 4);
    g.rowT = (int32_t *)take((size_t)adj_cap * 4);
    g.valT = (float *)take((size_t)adj_cap * 4);
    g.unordered = (uint2 *)take((size_t)adj_cap * 8);
    g.bytes = off;
    return g;
}

// out[k, :] = X[ids[k], :]; one wavefront per row, rows strided over the grid.  An id outside the table gives a zero row.
// WHOLE: rows of whole pieces of U that start on a multiple of it, everything counted in pieces.  Else everything is counted in bytes, the
// pieces are taken from any address, and the last one of a row (of at least one piece) ends with it and may overlap the one before.
template <typename U, bool WHOLE>
__global__ __launch_bounds__(256) void gather_rows_k(const U *__restrict__ X, int64_t ld, int64_t rows, int64_t row,
                                                     const int32_t *__restrict__ ids, int64_t cap,
                                                     const int64_t *__restrict__ n_dev, U *__restrict__ out,
                                                     int64_t ldo, CompStride cs)
{
    constexpr int32_t SIZE = (int32_t)sizeof(U);
    X = comp_ptr(X, cs.x); ids = comp_ptr(ids, cs.adj); n_dev = comp_ptr(n_dev, cs.adj); out = comp_ptr(out, cs.out);
    int64_t n = cap;
    if (n_dev) {
        const int64_t d = *n_dev;
        n = d < 0 ? 0 : (d < cap ? d : cap);
    }
    const int lane = lane_id();
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t n_waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t k = wave; k < n; k += n_waves) {
        const int64_t id = ids[k];
        const bool ok = id >= 0 && id < rows;
        if constexpr (WHOLE) {
            for (int32_t f = lane; f < (int32_t)row; f += WAVE) out[k * ldo + f] = ok ? X[id * ld + f] : U{};
        } else {
            for (int64_t f = lane * SIZE; f < row; f += WAVE * SIZE) {
                const int64_t at = f < row - SIZE ? f : row - SIZE;
                store_global<U, 2>((char *)out + k * ldo + at, ok ? load_global<U, 2>((const char *)X + id * ld + at) : U{});
            }
        }
    }
}

template <typename U, bool WHOLE>
static void launch_gather(const void *X, int64_t ld_b, int64_t rows, int64_t row_b, const int32_t *ids, int64_t cap,
                          const int64_t *n_dev, void *out, int64_t ldo_b, hipStream_t st, const CompInst &ci)
{
    const int64_t waves = cap < 8192 ? cap : 8192;
    const unsigned blocks = (unsigned)((waves + 3) / 4);
    constexpr int64_t UNIT = WHOLE ? (int64_t)sizeof(U) : 1;
    CSGS_LAUNCH(K_GATHER_ROWS, (gather_rows_k<U, WHOLE>), dim3(blocks, 1, (unsigned)ci.n), dim3(256), st, (const U *)X, ld_b / UNIT, rows,
                row_b / UNIT, ids, cap, n_dev, (U *)out, ldo_b / UNIT, ci.cs);
}

}  // namespace csgs

using namespace csgs;

extern "C" int csgs_gather_rows_n(const csgs_inst_strides *inst, const void *X, int64_t ld, int64_t rows, int32_t F, int dtype,
                                  const int32_t *ids, int64_t cap, const int64_t *n_dev, void *out, int64_t ldo, void *stream)
{
    if (!X || !ids || !out || rows <= 0 || F <= 0 || ld < F || ldo < F || cap <= 0) return CSGS_EINVAL;
    CompInst ci;
    if (open_instances(inst, &ci) != CSGS_OK) return CSGS_EINVAL;
    if (dtype != CSGS_F32 && dtype != CSGS_BF16) return CSGS_EUNSUPPORTED;
    const int64_t elt = dtype == CSGS_F32 ? 4 : 2;
    const int64_t row_b = (int64_t)F * elt, ld_b = ld * elt, ldo_b = ldo * elt;
    hipStream_t st = (hipStream_t)stream;
    auto whole = [&](int64_t a) {
        return row_b % a == 0 && ld_b % a == 0 && ldo_b % a == 0 && ((uintptr_t)X % (uintptr_t)a) == 0 &&
               ((uintptr_t)out % (uintptr_t)a) == 0;
    };
    const int64_t piece = whole(16) ? 16 : (whole(4) ? 4 : 2);
    // Rows that the wavefront's lanes cover at once go in whole pieces; longer ones that are no whole 16-byte pieces in 16 bytes from any
    // address (us, 131 K rows, 16 bytes from any address / whole pieces: 9 bf16 values 14.1 / 10.3, 5 floats 12.9 / 10.8, 31 floats 16.2 /
    // 15.7, 133 floats 22.7 / 28.1, 333 bf16 values 26.9 / 42.7; 75 bf16 values 16.5 / 20.8, of 30 K rows 5.7 / 5.3).  No pieces of 8: the same
    // in pieces of 4 is quicker (12 bf16 values 13.5 / 12.0, 2 floats 11.8 / 9.1).
    if (piece == 16) launch_gather<u32x4, true>(X, ld_b, rows, row_b, ids, cap, n_dev, out, ldo_b, st, ci);
    else if (row_b > WAVE * piece) launch_gather<u32x4, false>(X, ld_b, rows, row_b, ids, cap, n_dev, out, ldo_b, st, ci);
    else if (piece == 4) launch_gather<uint32_t, true>(X, ld_b, rows, row_b, ids, cap, n_dev, out, ldo_b, st, ci);
    else launch_gather<uint16_t, true>(X, ld_b, rows, row_b, ids, cap, n_dev, out, ldo_b, st, ci);
    CSGS_LAUNCH_CHECK();
    return CSGS_OK;
}

extern "C" int csgs_gather_rows(const void *X, int64_t ld, int64_t rows, int32_t F, int dtype, const int32_t *ids,
                                int64_t cap, const int64_t *n_dev, void *out, int64_t ldo, void *stream)
{
    return csgs_gather_rows_n(nullptr, X, ld, rows, F, dtype, ids, cap, n_dev, out, ldo, stream);
}

extern "C" int csgs_aggregate(const int32_t *adj_rowptr, const int32_t *adj_col, const float *adj_val, int32_t nS,
                              const int32_t *nS_dev, const int32_t *n_next, const void *X_local, int64_t ld_local, int64_t rows_local,
                              const void *X_remote, int64_t ld_remote, int64_t rows_remote, const int32_t *src_row,
                              int32_t F, int dtype, int relu_on_input, float *Z, int64_t ldz, void *stream)
{
    return csgs_aggregate_n(nullptr, adj_rowptr, adj_col, adj_val, nS, nS_dev, n_next, X_local, ld_local, rows_local, X_remote,
                            ld_remote, rows_remote, src_row, F, dtype, relu_on_input, Z, ldz, stream);
}

extern "C" int csgs_aggregate_n(const csgs_inst_strides *inst, const int32_t *adj_rowptr, const int32_t *adj_col,
                                const float *adj_val, int32_t nS, const int32_t *nS_dev, const int32_t *n_next,
                                const void *X_local, int64_t ld_local, int64_t rows_local, const void *X_remote,
                                int64_t ld_remote, int64_t rows_remote, const int32_t *src_row, int32_t F, int dtype,
                                int relu_on_input, float *Z, int64_t ldz, void *stream)
{
    CompInst ci;
    if (open_instances(inst, &ci) != CSGS_OK) return CSGS_EINVAL;
    if (!adj_rowptr || !adj_col || !adj_val || nS <= 0 || F <= 0 || rows_local < 0 || (rows_local > 0 && !X_local) ||
        (X_local && ld_local < F) || !Z || ldz < F || (X_remote && (ld_remote < F || rows_remote < 0)))
        return CSGS_EINVAL;
    if (!X_remote) rows_remote = 0;
    if (!X_local || rows_local == 0) { X_local = nullptr; rows_local = 0; ld_local = F; }
    if (dtype != CSGS_F32 && dtype != CSGS_BF16) return CSGS_EUNSUPPORTED;
    if (rows_remote > 0x7FFFFFFEll) return CSGS_EUNSUPPORTED;   // staged rows are addressed as -1 - row in 32 bits
    hipStream_t st = (hipStream_t)stream;
    if (dtype == CSGS_F32)
        return pick_vec<float>(adj_rowptr, adj_col, adj_val, nS, nS_dev, n_next, X_local, ld_local, rows_local, X_remote,
                               ld_remote, rows_remote, src_row, F, relu_on_input, Z, ldz, nullptr, 0, prof::K_AGGREGATE, st, ci);
    return pick_vec<uint16_t>(adj_rowptr, adj_col, adj_val, nS, nS_dev, n_next, X_local, ld_local, rows_local, X_remote,
                              ld_remote, rows_remote, src_row, F, relu_on_input, Z, ldz, nullptr, 0, prof::K_AGGREGATE, st, ci);
}

extern "C" size_t csgs_aggregate_grad_scratch_bytes(int32_t n_cols, int64_t adj_cap)
{
    if (n_cols <= 0 || adj_cap <= 0) return 0;
    return carve_grad(nullptr, n_cols, adj_cap).bytes;
}

extern "C" int csgs_aggregate_grad(const int32_t *adj_rowptr, const int32_t *adj_col, const float *adj_val, int64_t adj_cap,
                                   int32_t nS, const int32_t *nS_dev, int32_t n_cols, const int32_t *n_cols_dev, const float *dZ,
                                   int64_t lddz, int32_t F, const float *H_prev, int64_t ldh, float *dH_prev, int64_t ldd,
                                   void *scratch, size_t scratch_bytes, void *stream)
{
    if (!adj_rowptr || !adj_col || !adj_val || adj_cap <= 0 || adj_cap > 0x7FFFFFFFll || nS <= 0 || n_cols <= 0 || !dZ ||
        lddz < F || F <= 0 || (H_prev && ldh < F) || !dH_prev || ldd < F || !scratch || ((uintptr_t)scratch & 255))
        return CSGS_EINVAL;
    const GradScratch g = carve_grad(scratch, n_cols, adj_cap);
    if (scratch_bytes < g.bytes) return CSGS_EWORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    if (adj_cap <= (n_cols <= ONE_WIDE ? ONE_ENTRIES : ONE_ENTRIES_WIDE) && n_cols <= ONE_COLS) {
        CSGS_LAUNCH(K_ADJT_ORDER, adjT_one, dim3(ONE_GRID), dim3(ONE_BLOCK), st, adj_rowptr, adj_col, adj_val, nS, nS_dev, n_cols, n_cols_dev, adj_cap,
                    g.colptr, g.rowT, g.valT);
        CSGS_LAUNCH_CHECK();
    } else {
        const unsigned zb = (unsigned)(((int64_t)n_cols + 255) / 256 < 1024 ? ((int64_t)n_cols + 255) / 256 : 1024);
        CSGS_LAUNCH(K_FILL_ZERO, fill_zero_i32, dim3(zb), dim3(256), st, g.counts, (int64_t)n_cols);
        CSGS_LAUNCH_CHECK();
        const unsigned rb = (unsigned)(((int64_t)nS + 3) / 4 < 4096 ? ((int64_t)nS + 3) / 4 : 4096);   // 4 rows (wavefronts) per block
        CSGS_LAUNCH(K_ADJT_COUNT, adjT_count, dim3(rb), dim3(256), st, adj_rowptr, adj_col, nS, nS_dev, n_cols, n_cols_dev, adj_cap, g.counts);
        CSGS_LAUNCH_CHECK();
        const int64_t pieces = ((int64_t)n_cols + PREFIX_COLS - 1) / PREFIX_COLS, rounds = (pieces + PREFIX_GRID - 1) / PREFIX_GRID;
        CSGS_LAUNCH(K_ADJT_PREFIX, adjT_prefix, dim3((unsigned)((pieces + rounds - 1) / rounds)), dim3(256), st, (const int32_t *)g.counts, n_cols, n_cols_dev,
                    g.colptr, (int32_t)rounds);
        CSGS_LAUNCH_CHECK();
        CSGS_LAUNCH(K_ADJT_FILL, adjT_fill, dim3(rb), dim3(256), st, adj_rowptr, adj_col, adj_val, nS, nS_dev, n_cols, n_cols_dev,
                    (const int32_t *)g.colptr, g.counts, g.unordered, adj_cap);
        CSGS_LAUNCH_CHECK();
        const unsigned ob = (unsigned)(((int64_t)n_cols + ORD_COLS - 1) / ORD_COLS);
        CSGS_LAUNCH(K_ADJT_ORDER, adjT_order, dim3(ob), dim3(AGG_BLOCK), st, (const int32_t *)g.colptr, n_cols, n_cols_dev, nS, nS_dev,
                    (const uint2 *)g.unordered, g.rowT, g.valT, adj_cap);
        CSGS_LAUNCH_CHECK();
    }
    // the forward kernel on the transposed structure: rows = columns of P~, gathered table = dZ
    // (its rows are bounded by the row count of P~), output mask = [H_prev > 0]
    return pick_vec<float>(g.colptr, g.rowT, g.valT, n_cols, n_cols_dev, nS_dev, dZ, lddz, (int64_t)nS, nullptr, (int64_t)F, 0,
                           nullptr, F, 0, dH_prev, ldd, H_prev, ldh, prof::K_AGGREGATE_GRAD, st);
}
